// Variance estimate (Section 2): the temporal variance of the luminance
// moments where the history is long enough, a depth- and normal-weighted
// spatial estimate where it is not.  The second moment arrives as the
// central moment m2c = E[L^2] - E[L]^2, so neither branch cancels.
//
// Pass 1 (pointwise) writes the temporal estimate and lists the pixels
// whose history is short, except in tiles that hold many of them; pass 2
// computes the spatial estimate of the listed pixels, eight lanes per pixel,
// spread over every CU, and of the dense tiles, from LDS where there are many.
// (Where the temporal step has written the first part, it has listed every
// short pixel.)
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
                                                     float dx, float dy) {
    const float den = fmaf(a.sigma_z, fabsf(grad_offset(gx, gy, dx, dy)), a.eps_z);
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
// A tile with at least kDenseTile short pixels is not listed but marked.  Many
// of them are computed by one workgroup each: its window, (64 + 2 R) x
// (4 + 2 R) pixels of depth, normal and moments, is staged once in LDS, and
// the short pixels are packed onto the threads.  Every
// value is then loaded about 2.7 times (R = 3) where the listed form gathers
// it 49 times.  The sums run in the listed form's order (eight partial sums of
// taps sub, sub + 8, ..., joined as its butterfly joins them), so a pixel's
// result does not depend on which form computed it.  An empty or outside pixel
// is staged with an infinite depth, which marks it: its weight is 0.
// A quarter of a tile: below it the list is as fast, and its pixels spread over
// the whole chip.  In a frame of up to kScanWords words of marks (2048 tiles),
// up to 96 dense tiles (R <= 4, see dense_blocks) take the listed form as well,
// straight from the marks: a workgroup per tile leaves most of the chip idle
// there, while in a larger frame the list hides it and counting the marks (2
// to 3 us at 8160 tiles) is the loss.
// The call with its short pixels in 16x16 patches, binary32, R = 3, everything
// listed -> as here: at 1920x1080 none short 8.5 -> 9.5 us, 2 % 24.8 -> 24.9,
// 20 % 128 -> 94, all 454 -> 151 (there the pointwise pass goes from 79 to 7 us:
// a listing tile takes an atomic, and those of a sublist run one after the
// other); at 256x256 none 4.5 -> 4.9, 10 % 8.0 -> 10.0 (with the LDS form for
// every dense tile 10.4), all 17.8 -> 13.6.
constexpr uint32_t kDenseTile = 65;
constexpr int kScanWords = 512;    // words of marks, four tiles each, up to which they are counted

// The pointwise pass leaves one byte per tile, dense or not, at the end of
// the last sublist, where no entry of it can be: a sublist has 1024 bytes per
// tile of its own, and a tile lists fewer than kDenseTile pixels.  Before the
// marks, on a line of their own (in the counters' line they slowed its atomics
// down: the pass took 60 us for 36), three words tell whether there is a mark:
//   kTurn   a number, written by the reading pass of the last call,
//   kCall   the next one, this call's, and
//   kDense  that of the last call that had a dense tile,
// the last two written by the pointwise pass.  Whatever an earlier use of the
// workspace left there, a call's own dense tile is seen, and at worst marks
// are counted that do not exist.
constexpr int kTurn = 0, kCall = 1, kDense = 2;

__device__ __forceinline__ int tile_count(const VarianceArgs &a) {
    return ((a.w + kVX - 1) / kVX) * ((a.h + kVY - 1) / kVY);
}
__device__ __forceinline__ uint32_t *dense_marks(const VarianceArgs &a) {
    return a.work->list + kXCD * a.cap - (tile_count(a) + 3) / 4;
}
__device__ __forceinline__ uint32_t *dense_words(const VarianceArgs &a) {
    const uint32_t marks = kXCD * a.cap - (uint32_t)((tile_count(a) + 3) / 4);
    return a.work->list + ((marks - kLines) & ~(kLines - 1u));
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
        const int t = q + 4 * j, dx = t % D - R, dy = t / D - R;
        // past the window: the empty entry after the tile's
        const int i = t < NT ? ci + dy * S::COLS + dx : S::N;
        const float2 m = s_m[i];
        const float4 g = s_g[i];
        const float v = spatial_weight(a, pg.x - g.x,
                                       spatial_depth_scale(a, gx, gy, (float)dx, (float)dy),
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
    if (R < 6 && fabsf(mean1) < INFINITY) {  // (R = 6 spills with both loops)
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            const float d = m1[j] - mean1;
            s1[j & 1] = fmaf(w[j] * d, d, s1[j & 1]);
        }
    } else {  // an empty tap's 0 times d may be NaN
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            const float d = m1[j] - mean1;
            s1[j & 1] = signbit(w[j]) ? s1[j & 1] : fmaf(w[j] * d, d, s1[j & 1]);
        }
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
    for (uint32_t k = threadIdx.x / 4; k < total; k += 64) {  // whole groups of four
        const int px = s_px[k], lx = px & 63, ly = px >> 6;
        const float2 d = s_d[px];
        const int q = threadIdx.x & 3;
        const float v =
            dense_estimate<R>(a, s_g, s_m, (ly + R) * S::COLS + lx + R, d.x, d.y, q);
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
    const int gxt = (a.w + kVX - 1) / kVX, tile = xcd_tile(tile_count(a));
    int x, y;
    const bool spatial = variance_point_px<T>(a, tile, tile % gxt, tile / gxt, x, y);
    const bool dense = list_short_pixel<kDenseTile - 1>(a.work, a.cap, tile, spatial, x, y,
                                                        wave_n, base_sh);
    if (tile < 0 || threadIdx.x != 0) return;
    ((uint8_t *)dense_marks(a))[tile] = dense;
    if (dense || tile == 0) {
        uint32_t *words = dense_words(a);
        const uint32_t call = words[kTurn] + 1u;
        if (tile == 0) words[kCall] = call;
        if (dense) words[kDense] = call;
    }
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

// The spatial estimate of pixel (x, y), in the image, by eight lanes: lane
// `sub` takes taps sub, sub + 8, ...  Every tap's loads are issued before any
// weight is formed, and the weights and m1 stay in registers for the second
// pass.  TEST: the pixel may be one that needs no estimate.
template <typename T, int R, bool TEST = false>
__device__ __forceinline__ void spatial_estimate(const VarianceArgs &a, int x, int y, int sub) {
    constexpr int D = 2 * R + 1, NT = D * D, PER = (NT + 7) / 8, CTR = R * D + R;
    const uint32_t po = (uint32_t)y * (uint32_t)a.pitch + (uint32_t)x;
    const float zc = ldo<T>(a.z, po), gx = ldo<T>(a.dzdx, po), gy = ldo<T>(a.dzdy, po);
    const float nxp = ldo<T>(a.nx, po), nyp = ldo<T>(a.ny, po), nzp = ldo<T>(a.nz, po);
    const int n = TEST ? a.n[po] : 0;
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
    if (TEST && !(n >= 1 && n < a.min_hist && !empty_px(zc))) return;  // all eight lanes
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
            const float kz = spatial_depth_scale(a, gx, gy, (float)dx, (float)dy);
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

// Where the sublists start when laid end to end (pre[kXCD]: all entries).
__device__ __forceinline__ void list_starts(const VarianceArgs &a, uint32_t (&pre)[kXCD + 1]) {
    pre[0] = 0;
#pragma unroll
    for (int k = 0; k < kXCD; ++k)
        pre[k + 1] = pre[k] + min(a.work->count[k * kLines + kCount] -
                                      a.work->count[k * kLines + kBase],
                                  a.cap);
}

// Pixel e of the list; false for a stale entry outside the image.
__device__ __forceinline__ bool list_pixel(const VarianceArgs &a, const uint32_t (&pre)[kXCD + 1],
                                           uint32_t e, int &x, int &y) {
    int k = 0;
#pragma unroll
    for (int j = 1; j < kXCD; ++j) k += e >= pre[j] ? 1 : 0;
    const uint32_t packed = a.work->list[k * a.cap + (e - pre[k])];
    x = (int)(packed & 32767u), y = (int)(packed >> 15);
    return x < a.w && y < a.h;
}

// The list is consumed: the next appending pass starts after it (no
// workgroup of this pass reads kNext).
__device__ __forceinline__ void list_done(const VarianceArgs &a, uint32_t b) {
    if (b == 0 && threadIdx.x < kXCD)
        a.work->count[threadIdx.x * kLines + kNext] = a.work->count[threadIdx.x * kLines + kCount];
}

constexpr int kGroups = 256 / 8;  // pixels of a workgroup at a time

template <typename T, int R, bool ANEW = false>
__device__ __forceinline__ void variance_spatial_stream(const VarianceArgs &a, uint32_t b,
                                                        uint32_t blocks) {
    uint32_t pre[kXCD + 1];
    list_starts(a, pre);
    list_done(a, b);
    int x, y;
    for (uint32_t e = b * kGroups + threadIdx.x / 8; e < pre[kXCD]; e += blocks * kGroups) {
        // ANEW: nothing about the lane's taps is kept from pixel to pixel
        const int sub = ANEW ? (int)vofs(threadIdx.x & 7) : threadIdx.x & 7;
        if (list_pixel(a, pre, e, x, y)) spatial_estimate<T, R>(a, x, y, sub);
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

// The second pass after variance_point_k: the first `dense` workgroups for the
// dense tiles, then the list's, side by side, so that few dense tiles hide
// behind the list and many fill the chip before it (workgroups of the two kinds
// in turn left half of the CUs without tiles: all pixels of 1920x1080 short 275
// us for 157).  Where no tile is dense they end on one load of two words.
// Registers: as many waves per SIMD as the listed form alone has, or one fewer
// (R = 4 and 5), without spilling.  Capped at four for every R, R = 4 to 7
// spilled 26 to 346 registers: 1920x1080, 2 % of the pixels short, R = 5 65 us
// and R = 7 185, now 34 and 61 (everything listed: 32 and 55); all short 507
// and 1802, now 340 and 872 (728 and 1422).
template <int R>
constexpr int short_waves() { return R <= 3 ? 4 : R == 4 ? 3 : R <= 6 ? 2 : 1; }
// One to three workgroups a CU, no more than are resident at once (R = 7, none
// short, 1920x1080: 11.6 us with three).  A multiple of kXCD.
template <int R>
constexpr int dense_blocks() { return 256 * std::min(short_waves<R>(), 3); }

template <typename T, int R>
__global__ __launch_bounds__(256, short_waves<R>()) void variance_short_k(
    VarianceArgs a, int dense) {
    using S = DenseShape<R>;
    __shared__ float4 s_g[S::N + 1];
    __shared__ float2 s_m[S::N + 1], s_d[256];
    __shared__ uint32_t s_before[256];
    __shared__ uint8_t s_px[256];
    __shared__ uint32_t wave_n[4];
    const int b = (int)blockIdx.x;
    uint32_t *const state = dense_words(a);
    if (b >= dense) {
        const uint32_t call = state[kCall];
        // (R = 6 would spill 2 registers in binary16)
        variance_spatial_stream<T, R, R == 6>(a, (uint32_t)(b - dense),
                                              gridDim.x - (uint32_t)dense);
        // (a store before the list's loads would make them vector loads)
        if (b == dense && threadIdx.x == 0) state[kTurn] = call;
        return;
    }
    if (state[kDense] != state[kCall]) return;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int tiles = tile_count(a), words = (tiles + 3) / 4;
    const uint32_t *marks = dense_marks(a);
    // the workgroup's own tiles in the LDS form: a strided run of its XCD's
    // contiguous range, 64 marks at a time and alike in every wave
    const int slots = dense / kXCD, per = (tiles + kXCD - 1) / kXCD;
    const int last = min(tiles, (b % kXCD + 1) * per);
    int base = b % kXCD * per + b / kXCD;
    auto own = [&](int from) {
        const int t = from + lane * slots;
        return t < last && ((const uint8_t *)marks)[t] != 0;
    };
    bool marked = own(base);
    if (words <= kScanWords) {
        // thread t counts the marks of words t, t + 256, ... (a word holds none
        // past the tiles)
        auto word = [&](int i) {
            const uint32_t v = i < words ? marks[i] & 0x01010101u : 0u;
            return 4 * i + 4 > tiles && i < words ? v & ((1u << (8 * (tiles & 3))) - 1u) : v;
        };
        uint32_t mine = 0;
#pragma unroll
        for (int k = 0; k < kScanWords / 256; ++k)
            mine += (uint32_t)__popc(word((int)threadIdx.x + 256 * k));
        uint32_t upto = mine;
#pragma unroll
        for (int m = 1; m < 64; m *= 2) {
            const uint32_t v = (uint32_t)__shfl_up((int)upto, m, 64);
            upto += lane >= m ? v : 0u;
        }
        if (lane == 63) wave_n[wave] = upto;
        __syncthreads();
        const uint32_t n0 = wave_n[0], n1 = wave_n[1], n2 = wave_n[2],
                       total = n0 + n1 + n2 + wave_n[3];
        if (total * 8u <= (uint32_t)dense) {        // few
            if ((uint32_t)b >= total * 8u) return;  // uniform
            const uint32_t rank = (uint32_t)b / 8u;  // of the tile this workgroup takes 32 pixels of
            s_before[threadIdx.x] =
                upto - mine + (wave > 0 ? n0 : 0u) + (wave > 1 ? n1 : 0u) + (wave > 2 ? n2 : 0u);
            __syncthreads();
            int t = 0;  // the thread that counted it
#pragma unroll
            for (int m = 128; m > 0; m /= 2) t += s_before[t + m] <= rank ? m : 0;
            uint32_t left = rank - s_before[t], v = word(t);
            int i = t;
            for (uint32_t n; left >= (n = (uint32_t)__popc(v)); v = word(i)) left -= n, i += 256;
            for (; left > 0u; --left) v &= v - 1u;
            const int gxt = (a.w + kVX - 1) / kVX, tile = 4 * i + (__ffs((int)v) - 1) / 8;
            const int px = b % 8 * kGroups + (int)threadIdx.x / 8;
            const int x = tile % gxt * kVX + px % kVX, y = tile / gxt * kVY + px / kVX;
            if (x < a.w && y < a.h) spatial_estimate<T, R, true>(a, x, y, (int)threadIdx.x & 7);
            return;
        }
    }
    for (; base < last; base += 64 * slots, marked = own(base))
        for (uint64_t set = __ballot(marked); set != 0ull; set &= set - 1ull) {
            __syncthreads();  // the last tile is read
            variance_dense_tile<T, R>(a, base + (__ffsll((unsigned long long)set) - 1) * slots,
                                      s_g, s_m, s_d, s_px, wave_n);
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
        hipLaunchKernelGGL((variance_short_k<T, R>), dim3(dense_blocks<R>() + kSpatialBlocks),
                           dim3(256), 0, s, a, dense_blocks<R>());
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
