// Variance estimate (Section 2): the temporal variance of the luminance
// moments where the history is long enough, a depth- and normal-weighted
// spatial estimate where it is not.  The second moment arrives as the
// central moment m2c = E[L^2] - E[L]^2, so neither branch cancels.
//
// Pass 1 (pointwise) writes the temporal estimate and lists the pixels
// whose history is short, except in tiles that hold many of them; pass 2
// computes the spatial estimate of the listed pixels, eight lanes per pixel,
// spread over every CU, and of the dense tiles from LDS.  (Where the temporal
// step has written the first part, it has listed every short pixel.)
#include <algorithm>
#include <mutex>

#include "sv_internal.h"

namespace sv {

constexpr int kSpatialBlocks = 1024;  // pass-2 grid (grid-stride over the list)

struct VarianceArgs {
    const float *m1, *m2c;
    const uint8_t *n;
    const void *z, *dzdx, *dzdy, *nx, *ny, *nz;
    float *var;
    VarWork *work;
    uint32_t cap;  // entries per sublist
    int w, h, pitch;
    float sigma_z, eps_z;
    NormalCoef nc;
    int min_hist;
};

// This thread's pixel of tile `tile` (-1: a padding workgroup, which still
// takes the barriers); true if it needs the spatial estimate, else its
// pointwise one is stored.
template <typename T>
__device__ __forceinline__ bool variance_point_px(const VarianceArgs &a, int tile, int bxt,
                                                  int byt, int &x, int &y) {
    x = bxt * kVX + (threadIdx.x & 63), y = byt * kVY + (threadIdx.x >> 6);
    const bool inside = tile >= 0 && x < a.w && y < a.h;
    const uint32_t o = vofs(inside ? (uint32_t)y * (uint32_t)a.pitch + (uint32_t)x : 0u);
    // all three loads issued together (the address is in the image)
    const int nn = a.n[o];
    const float zp = ldo<T>(a.z, o), m2 = ldf(a.m2c, o);
    const int n = inside ? nn : 0;
    const bool live = inside && n >= 1 && !empty_px(zp);
    const bool spatial = live && n < a.min_hist;
    if (inside && !spatial) stf(a.var, o, live ? fmaxf(0.f, m2) : 0.f);
    return spatial;
}

// Depth scale of an offset: the same for (dx, dy) and (-dx, -dy), bit for bit.
__device__ __forceinline__ float spatial_depth_scale(const VarianceArgs &a, float gx, float gy,
                                                     int dx, int dy) {
    const float den =
        fmaf(a.sigma_z, fabsf(grad_offset(gx, gy, (float)dx, (float)dy)), a.eps_z);
    return kLog2e / den;
}

// Weight of a tap (not the centre) from its depth difference, depth scale
// and squared normal chord.
__device__ __forceinline__ float spatial_weight(const VarianceArgs &a, float dz, float kz,
                                                float s2) {
    return __builtin_amdgcn_exp2f(add_normal_term(-fabsf(dz) * kz, s2, a.nc));
}

// ---- dense tiles ---------------------------------------------------------------
//
// A tile with at least kDenseTile short pixels is computed by one workgroup:
// its window, (64 + 2 R) x (4 + 2 R) pixels of depth, normal and moments, is
// staged once in LDS, and the short pixels are packed onto the threads.  Every
// value is then loaded about 2.7 times (R = 3) where the listed form gathers
// it 49 times.  The sums run in the listed form's order (eight partial sums of
// taps sub, sub + 8, ..., joined as its butterfly joins them), so a pixel's
// result does not depend on which form computed it.  An empty or outside pixel
// is staged with an infinite depth, which marks it: its weight is 0.
// A quarter of a tile: below it the list is as fast, and its pixels spread over
// the whole chip.  Measured at 1920x1080, binary32, the call with its short
// pixels in 16x16 patches (everything listed -> dense tiles): 2 % short 23 ->
// 24 us, 20 % 126 -> 90, 50 % 245 -> 115, all 415 -> 155 (there the pointwise
// pass went from 79 to 8 us: a listing tile takes an atomic, and those of a
// sublist run one after the other).
constexpr uint32_t kDenseTile = 65;
constexpr int kDenseBlocks = 768;  // workgroups that share the dense tiles

// The pointwise pass leaves one word per tile, dense or not, at the end of the
// tile's sublist (tile % 8), where no entry of it can be: a sublist has 256
// words per tile, and a tile lists fewer than kDenseTile pixels.
__device__ __forceinline__ uint32_t flag_word(uint32_t cap, int tile) {
    return (uint32_t)tile % kXCD * cap + cap - 1u - (uint32_t)tile / kXCD;
}

template <int R>
struct DenseShape {
    static constexpr int COLS = kVX + 2 * R, ROWS = kVY + 2 * R, N = COLS * ROWS;
    static constexpr int D = 2 * R + 1, NT = D * D, CTR = R * D + R;
};

// Four lanes per pixel, lane q taking taps q, q + 4, ...: the listed form's
// partial sums q and q + 4, joined first as its butterfly joins them.
template <int R>
__device__ __forceinline__ float dense_estimate(const VarianceArgs &a, const float4 *s_g,
                                                 const float2 *s_m, int ci, float gx, float gy,
                                                 int q) {
    using S = DenseShape<R>;
    constexpr int D = S::D, NT = S::NT, CTR = S::CTR, PER = (NT + 3) / 4;
    const float4 pg = s_g[ci];
    float w[PER], m1[PER], sw[2] = {0.f, 0.f}, s1[2] = {0.f, 0.f}, sm[2] = {0.f, 0.f};
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        const int t = q + 4 * j;
        const int dx = t % D - R, dy = t / D - R;
        // past the window: the empty entry after the tile's
        const int i = t < NT ? ci + dy * S::COLS + dx : S::N;
        const float2 m = s_m[i];
        const float4 g = s_g[i];
        const float v =
            spatial_weight(a, pg.x - g.x, spatial_depth_scale(a, gx, gy, dx, dy),
                           chord2(pg.y, pg.z, pg.w, g.y, g.z, g.w));
        // an empty tap's -0 adds nothing, and marks it for the second loop
        w[j] = t == CTR ? 1.f : g.x < INFINITY ? v : -0.f;
        m1[j] = m.x;
        sw[j & 1] += w[j];
        s1[j & 1] = fmaf(w[j], m.x, s1[j & 1]);
        sm[j & 1] = fmaf(w[j], m.y, sm[j & 1]);
    }
    auto join = [](const float (&v)[2]) {
        float s = v[0] + v[1];
        s += __shfl_xor(s, 2, 64);
        return s + __shfl_xor(s, 1, 64);
    };
    const float sum = join(sw), mean1 = join(s1) / sum, mom = join(sm);
    s1[0] = s1[1] = 0.f;
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        const float d = m1[j] - mean1;  // may be infinite: not to be times a 0
        s1[j & 1] = signbit(w[j]) ? s1[j & 1] : fmaf(w[j] * d, d, s1[j & 1]);
    }
    return fmaxf(0.f, (mom + join(s1)) / sum);
}

// One dense tile (its short pixels found as the pointwise pass found them);
// every thread of the workgroup calls it.
template <typename T, int R>
__device__ __forceinline__ void variance_dense_tile(const VarianceArgs &a, int tile, float4 *s_g,
                                                    float2 *s_m, float2 *s_d, uint8_t *s_px,
                                                    uint32_t *wave_n) {
    using S = DenseShape<R>;
    const int gxt = (a.w + kVX - 1) / kVX;
    const int byt = tile / gxt, bxt = tile - byt * gxt;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int x = bxt * kVX + lane, y = byt * kVY + wave;
    const bool inside = x < a.w && y < a.h;
    const uint32_t po = vofs(inside ? (uint32_t)y * (uint32_t)a.pitch + (uint32_t)x : 0u);
    const int n = a.n[po];
    const float gx = ldo<T>(a.dzdx, po), gy = ldo<T>(a.dzdy, po);
#pragma unroll
    for (int it = 0; it < (S::N + 255) / 256; ++it) {
        const int i = threadIdx.x + it * 256;
        const int r = i / S::COLS, c = i - r * S::COLS;
        const int qx = bxt * kVX - R + c, qy = byt * kVY - R + r;
        const bool in = i < S::N && qx >= 0 && qx < a.w && qy >= 0 && qy < a.h;
        const uint32_t q = vofs(in ? (uint32_t)qy * (uint32_t)a.pitch + (uint32_t)qx : 0u);
        const float z = ldo<T>(a.z, q), nx = ldo<T>(a.nx, q), ny = ldo<T>(a.ny, q),
                    nz = ldo<T>(a.nz, q), m1 = ldf(a.m1, q), m2 = ldf(a.m2c, q);
        const bool ok = in && !empty_px(z);
        if (i < S::N) {
            s_g[i] = ok ? make_float4(z, nx, ny, nz) : make_float4(INFINITY, 0.f, 0.f, 0.f);
            s_m[i] = ok ? make_float2(m1, m2) : make_float2(0.f, 0.f);
        }
    }
    if (threadIdx.x == 0) {
        s_g[S::N] = make_float4(INFINITY, 0.f, 0.f, 0.f);
        s_m[S::N] = make_float2(0.f, 0.f);
    }
    s_d[threadIdx.x] = make_float2(gx, gy);
    __syncthreads();
    const bool spatial = inside && n >= 1 && n < a.min_hist &&
                         s_g[(wave + R) * S::COLS + lane + R].x < INFINITY;
    const uint64_t mask = __ballot(spatial);
    if (lane == 0) wave_n[wave] = (uint32_t)__popcll(mask);
    __syncthreads();
    const uint32_t n0 = wave_n[0], n1 = wave_n[1], n2 = wave_n[2], total = n0 + n1 + n2 + wave_n[3];
    const uint32_t before = (wave > 0 ? n0 : 0u) + (wave > 1 ? n1 : 0u) + (wave > 2 ? n2 : 0u);
    if (spatial)
        s_px[before + (uint32_t)__popcll(mask & ((1ull << lane) - 1ull))] = (uint8_t)threadIdx.x;
    __syncthreads();
    const int q = threadIdx.x & 3;
    for (uint32_t k = threadIdx.x / 4; k < total; k += 64) {  // whole groups of four
        const int px = s_px[k], lx = px & 63, ly = px >> 6;
        const float2 d = s_d[px];
        const float v = dense_estimate<R>(a, s_g, s_m, (ly + R) * S::COLS + lx + R, d.x, d.y, q);
        if (q == 0)
            stf(a.var, (uint32_t)(byt * kVY + ly) * (uint32_t)a.pitch + (uint32_t)(bxt * kVX + lx),
                v);
    }
}

// The pointwise pass.  Dense tiles are marked, the short pixels of the others
// listed.
template <typename T>
__global__ __launch_bounds__(256) void variance_point_k(VarianceArgs a) {
    __shared__ uint32_t wave_n[4], base_sh;
    const int gxt = (a.w + kVX - 1) / kVX;
    const int tile = xcd_tile(gxt * ((a.h + kVY - 1) / kVY));
    int x, y;
    const bool spatial = variance_point_px<T>(a, tile, tile % gxt, tile / gxt, x, y);
    const bool dense = (uint32_t)__syncthreads_count(spatial) >= kDenseTile;  // uniform
    if (tile >= 0 && threadIdx.x == 0) a.work->list[flag_word(a.cap, tile)] = dense ? 1u : 0u;
    list_short_pixel(a.work, a.cap, tile, spatial && !dense, x, y, wave_n, base_sh);
}

template <typename T>
__global__ __launch_bounds__(256) void variance_point_batch_k(const VarianceArgs *args,
                                                              const int *prefix, int n, int total) {
    __shared__ uint32_t wave_n[4], base_sh;
    int s = 0;
    const int lt = batch_tile(prefix, n, total, s);
    if (lt < 0) return;
    const VarianceArgs a = args[s];
    const int gxt = (a.w + kVX - 1) / kVX;
    int x, y;
    const bool spatial = variance_point_px<T>(a, lt, lt % gxt, lt / gxt, x, y);
    list_short_pixel(a.work, a.cap, lt, spatial, x, y, wave_n, base_sh);
}

// Zero state of a workspace's counters (the allocation-free entry point's
// shared array, which another call may have left in any state).
__global__ __launch_bounds__(64) void variance_reset_k(VarWork *w) {
    if (threadIdx.x < kXCD) {
        w->count[threadIdx.x * kLines + kCount] = 0;
        w->count[threadIdx.x * kLines + kBase] = 0;
        w->count[threadIdx.x * kLines + kNext] = 0;
    }
}

// Sum over the 8 lanes of an aligned lane group (butterfly: a fixed order,
// so the result is the same on every run).
__device__ __forceinline__ float group8_sum(float v) {
    v += __shfl_xor(v, 4, 64);
    v += __shfl_xor(v, 2, 64);
    v += __shfl_xor(v, 1, 64);
    return v;
}

// Window of radius R, eight lanes per listed pixel: lane `sub` takes taps
// sub, sub + 8, ...  Every tap's loads are issued before any weight is
// formed, and the weights and m1 stay in registers for the second pass.
template <typename T, int R>
__device__ __forceinline__ void variance_spatial_stream(const VarianceArgs &a, uint32_t b, uint32_t blocks) {
    constexpr int D = 2 * R + 1, NT = D * D, PER = (NT + 7) / 8, CTR = R * D + R;
    uint32_t pre[kXCD + 1];
    pre[0] = 0;
#pragma unroll
    for (int k = 0; k < kXCD; ++k)
        pre[k + 1] = pre[k] + min(a.work->count[k * kLines + kCount] -
                                      a.work->count[k * kLines + kBase],
                                  a.cap);
    const uint32_t count = pre[kXCD];
    // the list is consumed: the next appending pass starts after it (no
    // workgroup of this pass reads kNext)
    if (b == 0 && threadIdx.x < kXCD)
        a.work->count[threadIdx.x * kLines + kNext] = a.work->count[threadIdx.x * kLines + kCount];
    const int sub = threadIdx.x & 7;
    const uint32_t groups = blocks * (blockDim.x / 8);
    for (uint32_t e = b * (blockDim.x / 8) + (threadIdx.x >> 3); e < count; e += groups) {
        int k = 0;
#pragma unroll
        for (int j = 1; j < kXCD; ++j) k += e >= pre[j] ? 1 : 0;
        const uint32_t packed = a.work->list[k * a.cap + (e - pre[k])];
        const int x = (int)(packed & 32767u), y = (int)(packed >> 15);
        if (x >= a.w || y >= a.h) continue;  // only a stale entry can be outside
        const uint32_t po = (uint32_t)y * (uint32_t)a.pitch + (uint32_t)x;
        const float zc = ldo<T>(a.z, po), gx = ldo<T>(a.dzdx, po), gy = ldo<T>(a.dzdy, po);
        const float nxp = ldo<T>(a.nx, po), nyp = ldo<T>(a.ny, po), nzp = ldo<T>(a.nz, po);
        float zq[PER], qx_[PER], qy_[PER], qz_[PER], m1q[PER], m2q[PER];
        bool ok[PER];
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            const int t = sub + 8 * j;
            const int dx = t % D - R, dy = t / D - R;
            const int qx = x + dx, qy = y + dy;
            ok[j] = t < NT && qx >= 0 && qx < a.w && qy >= 0 && qy < a.h;
            const uint32_t q = vofs(ok[j] ? (uint32_t)qy * (uint32_t)a.pitch + (uint32_t)qx : po);
            zq[j] = ldo<T>(a.z, q);
            qx_[j] = ldo<T>(a.nx, q);
            qy_[j] = ldo<T>(a.ny, q);
            qz_[j] = ldo<T>(a.nz, q);
            m1q[j] = ldf(a.m1, q);
            m2q[j] = ldf(a.m2c, q);
        }
        // pass 1: weights and weighted sums of m1 and m2c
        float wt[PER];
        float sw = 0.f, s1 = 0.f, sm = 0.f;
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            const int t = sub + 8 * j;
            const int dx = t % D - R, dy = t / D - R;
            // an empty pixel enters no sum, whatever moments it holds
            ok[j] = ok[j] && (t == CTR || !empty_px(zq[j]));
            float w;
            if (t == CTR) {
                w = 1.f;
            } else {
                const float s2 = chord2(nxp, nyp, nzp, qx_[j], qy_[j], qz_[j]);
                const float kz = spatial_depth_scale(a, gx, gy, dx, dy);
                w = spatial_weight(a, zc - zq[j], kz, s2);
            }
            wt[j] = w;
            if (ok[j]) {
                sw += w;
                s1 = fmaf(w, m1q[j], s1);
                sm = fmaf(w, m2q[j], sm);
            }
        }
        sw = group8_sum(sw);
        s1 = group8_sum(s1);
        sm = group8_sum(sm);
        const float mean1 = s1 / sw;
        // pass 2: spread of m1 about its weighted mean
        float spread = 0.f;
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            const float d = m1q[j] - mean1;
            if (ok[j]) spread = fmaf(wt[j] * d, d, spread);
        }
        spread = group8_sum(spread);
        if (sub == 0) stf(a.var, po, fmaxf(0.f, (sm + spread) / sw));
    }
}

template <typename T, int R>
__global__ __launch_bounds__(256) void variance_spatial_k(VarianceArgs a) {
    variance_spatial_stream<T, R>(a, blockIdx.x, gridDim.x);
}

// One row of workgroups per stream.
template <typename T, int R>
__global__ __launch_bounds__(256) void variance_spatial_batch_k(const VarianceArgs *args) {
    const VarianceArgs a = args[blockIdx.y];
    variance_spatial_stream<T, R>(a, blockIdx.x, gridDim.x);
}

// The second pass after variance_point_k: the workgroups of the dense tiles
// and the list's, side by side, so that few dense tiles hide behind the list.
// (Within the pointwise pass their latency came on top of the list's: 27 us
// instead of 22 with 2 % of the pixels short.)  A dense workgroup walks a
// strided run of its XCD's contiguous range of tiles, their marks read 256 at
// a time.
template <typename T, int R>
__global__ __launch_bounds__(256, 4) void variance_short_k(VarianceArgs a, int dense) {
    __shared__ float4 s_g[DenseShape<R>::N + 1];
    __shared__ float2 s_m[DenseShape<R>::N + 1], s_d[256];
    __shared__ uint8_t s_px[256], s_flag[256];
    __shared__ uint32_t wave_n[4];
    const int b = (int)blockIdx.x, nslot = dense / kXCD;
    if (b >= dense) {
        variance_spatial_stream<T, R>(a, (uint32_t)(b - dense), kSpatialBlocks);
        return;
    }
    const int tiles = ((a.w + kVX - 1) / kVX) * ((a.h + kVY - 1) / kVY);
    const int per = (tiles + kXCD - 1) / kXCD;
    const int first = b % kXCD * per, last = min(tiles, first + per);
    for (int base = first + b / kXCD; base < last; base += 256 * nslot) {
        const int mine = base + (int)threadIdx.x * nslot;
        const bool flag = mine < last && a.work->list[flag_word(a.cap, mine)] != 0u;
        if (!__syncthreads_or(flag)) continue;  // uniform
        s_flag[threadIdx.x] = flag;
        __syncthreads();
        for (int k = 0; k < 256 && base + k * nslot < last; ++k) {
            if (!s_flag[k]) continue;  // uniform
            variance_dense_tile<T, R>(a, base + k * nslot, s_g, s_m, s_d, s_px, wave_n);
            __syncthreads();  // the next tile stages over this one
        }
        __syncthreads();
    }
}

template <typename T>
static void point_batch_launch(const void *args, const int *prefix, int n, int total,
                               hipStream_t s) {
    hipLaunchKernelGGL(variance_point_batch_k<T>, dim3(xcd_grid(total)), dim3(256), 0, s,
                       (const VarianceArgs *)args, prefix, n, total);
}

template <typename T, int R>
static void spatial_batch_launch(const void *args, const int *, int n, int, hipStream_t s) {
    // every stream's list at once: walked one stream after the other, each
    // paid its own chain of loads (twelve streams of 640..2560 columns: 77 us,
    // now 52 us)
    const int blocks = std::max(128, kSpatialBlocks / n);
    hipLaunchKernelGGL((variance_spatial_batch_k<T, R>), dim3(blocks, n), dim3(256), 0, s,
                       (const VarianceArgs *)args);
}

template <typename T, int R>
void launch_radius(const VarianceArgs &a, unsigned grid, bool listed, hipStream_t s) {
    const int tiles = ((a.w + kVX - 1) / kVX) * ((a.h + kVY - 1) / kVY);
    if (!listed && !record_pass(&point_batch_launch<T>, a, tiles)) {
        hipLaunchKernelGGL(variance_point_k<T>, dim3(grid), dim3(256), 0, s, a);
        // (grid, one workgroup per tile, and kDenseBlocks are multiples of kXCD)
        const int dense = (int)std::min<unsigned>(grid, kDenseBlocks);
        hipLaunchKernelGGL((variance_short_k<T, R>), dim3(dense + kSpatialBlocks), dim3(256), 0,
                           s, a, dense);
        return;
    }
    if (record_pass(&spatial_batch_launch<T, R>, a, 0)) return;
    hipLaunchKernelGGL((variance_spatial_k<T, R>), dim3(kSpatialBlocks), dim3(256), 0, s, a);
}

template <typename T>
void launch_variance(const VarianceArgs &a, unsigned grid, int radius, bool listed,
                     hipStream_t s) {
    switch (radius) {
    case 0: launch_radius<T, 0>(a, grid, listed, s); break;
    case 1: launch_radius<T, 1>(a, grid, listed, s); break;
    case 2: launch_radius<T, 2>(a, grid, listed, s); break;
    case 3: launch_radius<T, 3>(a, grid, listed, s); break;
    case 4: launch_radius<T, 4>(a, grid, listed, s); break;
    case 5: launch_radius<T, 5>(a, grid, listed, s); break;
    case 6: launch_radius<T, 6>(a, grid, listed, s); break;
    default: launch_radius<T, 7>(a, grid, listed, s); break;
    }
}

}  // namespace sv

// ---- the variance estimate without a caller workspace -------------------------
//
// For callers that cannot allocate (code under graph capture, tight serving
// loops): the workspace is one file-scope device array, kNoAllocBytes
// long, which each GPU holds for the life of the process.  Host code never
// passes the array's name to a kernel (in host code it is a stand-in, not a
// device address): the device address comes from hipGetSymbolAddress, taken
// once per device with that device current, and only that address is used.

namespace sv {

// 32 MiB: the eight counters and the pixel list of a 3840x2160 frame
// (sv_variance_work_bytes gives 33,178,624 bytes there).
constexpr size_t kNoAllocBytes = size_t(32) << 20;
constexpr int kMaxDevices = 64;

static __device__ __align__(256) unsigned char scratch[kNoAllocBytes];

static std::mutex g_scratch_lock;
static void *g_scratch_ptr[kMaxDevices];

// This device's address of the array, looked up on the first call on the
// device (with the device current); nullptr on failure.
static void *scratch_ptr(int dev) {
    std::lock_guard<std::mutex> lk(g_scratch_lock);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return nullptr;
        g_scratch_ptr[dev] = p;
    }
    return g_scratch_ptr[dev];
}

}  // namespace sv

extern "C" int sv_variance_noalloc(const float *m1, const float *m2c, const uint8_t *n,
                                   const sv_gbuf *g, float *var, sv_dims d, sv_dtype t,
                                   const sv_variance_params *p, sv_stream stream) {
    using namespace sv;
    if (!valid_dtype(t)) return SV_EDTYPE;
    const int dc = check_dims(d);
    if (dc < 0 || !p) return SV_EINVAL;
    if (p->flags & SV_V_LISTED) return SV_EINVAL;  // a list lives in the caller's workspace
    if (dc == 1) return SV_OK;
    if (sv_variance_work_bytes(d) > kNoAllocBytes) return SV_ETOOBIG;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return SV_EHIP;
    void *work = scratch_ptr(dev);
    if (!work) return SV_EHIP;
    // every call shares this device's array and finds what the last call
    // left there: its counters are cleared first (a kernel, not a memset,
    // so that a captured graph holds kernel nodes only)
    hipLaunchKernelGGL(variance_reset_k, dim3(1), dim3(64), 0, as_stream(stream),
                       (VarWork *)work);
    const int rc = hip_status(hipGetLastError());
    if (rc != SV_OK) return rc;
    return sv_variance(m1, m2c, n, g, var, work, d, t, p, stream);
}

extern "C" size_t sv_variance_work_bytes(sv_dims d) {
    if (sv::check_dims(d) < 0) return 0;
    return offsetof(sv::VarWork, list) + sizeof(uint32_t) * 256 * (size_t)sv::point_grid(d);
}

extern "C" int sv_variance(const float *m1, const float *m2c, const uint8_t *n, const sv_gbuf *g,
                           float *var, void *work, sv_dims d, sv_dtype t,
                           const sv_variance_params *p, sv_stream stream) {
    using namespace sv;
    if (!valid_dtype(t)) return SV_EDTYPE;
    int dc = check_dims(d);
    if (dc < 0 || !g || !p) return SV_EINVAL;
    if (p->radius < 0 || p->radius > 7 || p->min_hist < 0) return SV_EINVAL;
    if (!(p->sigma_n >= 0.f)) return SV_EINVAL;
    if (dc == 1) return SV_OK;
    if (!m1 || !m2c || !n || !var || !work || !g->z || !g->dzdx || !g->dzdy || !g->nx || !g->ny ||
        !g->nz)
        return SV_EINVAL;
    const size_t es = elem_size(t);
    const span ins[] = {plane_span(m1, d, 4), plane_span(m2c, d, 4), plane_span(n, d, 1),
                        plane_span(g->z, d, es), plane_span(g->dzdx, d, es),
                        plane_span(g->dzdy, d, es), plane_span(g->nx, d, es),
                        plane_span(g->ny, d, es), plane_span(g->nz, d, es)};
    const span so = plane_span(var, d, 4);
    const span sw{(uintptr_t)work, (uintptr_t)work + sv_variance_work_bytes(d)};
    for (const span &si : ins)
        if (overlaps(so, si) || overlaps(sw, si)) return SV_EALIAS;
    if (overlaps(so, sw)) return SV_EALIAS;
    const unsigned grid = point_grid(d);
    VarianceArgs a{m1, m2c, n, g->z, g->dzdx, g->dzdy, g->nx, g->ny, g->nz, var,
                   (VarWork *)work, (grid / kXCD) * 256u, d.w, d.h, d.pitch, p->sigma_z,
                   p->eps_z, make_normal_coef(p->sigma_n), p->min_hist};
    hipStream_t s = as_stream(stream);
    const bool listed = (p->flags & SV_V_LISTED) != 0;
    if (t == SV_F32)
        launch_variance<float>(a, grid, p->radius, listed, s);
    else
        launch_variance<half_t>(a, grid, p->radius, listed, s);
    return hip_status(hipGetLastError());
}
