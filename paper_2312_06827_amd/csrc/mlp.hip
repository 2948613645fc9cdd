// Learned blend factor and edge scale: a 14 -> 32 -> 32 -> 2 per-pixel
// network on the matrix cores (bfloat16 operands, binary32 accumulation),
// its backward pass, Adam, and the two truncated loss gradients that train
// it (through the temporal blend and through each a-trous level).
//
// The forward pass and the matrix layout are in mlp_impl.h.
#include "mlp_impl.h"

namespace sv {

struct MlpArgs {
    const float *params;
    const uint16_t *wq;
    const uint4 *feat;  // 2 x 16 bytes per pixel
    float *alpha, *kappa;
    const float *d_alpha, *d_kappa;
    float *part;  // backward: per-workgroup partial gradients
    int w, h, pitch;
    int npix, ngrp;  // pixels, 64-pixel groups
};

__device__ __forceinline__ bf16x8 load_x(const MlpArgs &a, int p, int hf) {
    return feature_operand((const uint2 *)(a.feat + 2 * (size_t)p), hf);
}

__device__ __forceinline__ uint32_t plane_off(const MlpArgs &a, int p) {
    const int y = p / a.w, x = p - y * a.w;
    return (uint32_t)y * (uint32_t)a.pitch + (uint32_t)x;
}

// A wave takes 64 pixels at a time, as two 32-pixel blocks: block hf's
// outputs are then kept by the lanes of half hf, so that the heads, the
// plane addresses and the stores are one pixel per lane.  One head
// evaluation per 64 pixels instead of two, one-instruction roundings, and
// the next group's features loaded before a group's heads (the first ones
// beside the weights), in the 128 registers of four waves per SIMD:
// 38 -> 24 us at 1920x1080 (83 MB: 16 us at the rate of a large copy; 28 us
// with each group's loads at its start, 27 us at three waves per SIMD), and
// 3.55 -> 3.65 at 64x64, where staging the weights in LDS is one step more
// (3.8 with the loads after it).
__global__ __launch_bounds__(256, 4) void mlp_forward_k(MlpArgs a) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int col = lane & 31, hf = lane >> 5;
    __shared__ u32x4 s_w[kNetStage];
    __shared__ __align__(16) float s_b[kNetFloats];
    NetStage ns;
    net_issue(a.params, a.wq, ns);
    int g = blockIdx.x * 4 + wave;
    const auto load = [&](bf16x8 (&x)[2]) {
#pragma unroll
        for (int blk = 0; blk < 2; ++blk)
            x[blk] = load_x(a, min(min(g, a.ngrp - 1) * 64 + blk * 32 + col, a.npix - 1), hf);
    };
    // the first features are in flight while the weights are staged
    bf16x8 x[2];
    load(x);
    net_store(ns, s_w, s_b);
    __syncthreads();
    NetW f;
    load_operands(s_w, lane, f);
    load_floats(s_b, hf, f);
    while (g < a.ngrp) {
        const int p = g * 64 + lane;
        float o0 = 0.f, o1 = 0.f;
#pragma unroll
        for (int blk = 0; blk < 2; ++blk) {
            FwdOut r;
            forward_block(f, x[blk], r);
            if (blk == hf) {
                o0 = r.o0;
                o1 = r.o1;
            }
        }
        g += gridDim.x * 4;
        if (g < a.ngrp) load(x);
        if (p < a.npix) {
            const uint32_t o = plane_off(a, p);
            float al, ka;
            mlp_heads(o0, o1, al, ka);
            if (a.alpha) a.alpha[o] = al;
            if (a.kappa) a.kappa[o] = ka;
        }
    }
}

// ---- backward ------------------------------------------------------------
//
// The weight gradients are contractions over pixels, so their operands hold
// pixels along K: lane l gives eight pixels of unit l % 32.  An operand with
// units along K, taken as A against a unit matrix as B, leaves exactly that
// in the accumulators (one product by 1 and zeros: exact for finite values),
// so the activations and the back-propagated gradients are turned on the
// matrix cores instead of through LDS.  Every value that is rounded to
// bfloat16 is formed as in a plain backward pass; 26 matrix instructions per
// 32 pixels, no LDS stores and no barrier in the loop.  At 1920x1080
// 99 us against 242 us for the form that turned four 32 x 32 tiles a block
// through 2-byte LDS stores and rounded in software.  The chain of dependent
// products at two waves per SIMD (256 registers) bounds it: with both of a
// wave's blocks in flight it spills, 176 us, and one wave per SIMD hides less.
//
// A value that is not finite, times the unit matrix's zeros, is NaN in every
// unit of its pixel, and so in every sum that the pixel enters.  A wave whose
// sums come out that way therefore runs its blocks again with the operands
// turned through LDS, which moves values without arithmetic: a NaN feature
// then reaches its own column of W1's gradient, and a head gradient that is
// not finite the units that it flows through.

// What the backward pass holds beside NetW.
struct BwdW {
    bf16x8 w2t[2];   // W2^T as A operand: [h1 unit = lane % 32][h2 unit]
    bf16x8 unit[2];  // K values 16 j + drow(i, hf) to their own columns
    bf16x8 unit_g;   // K values 0 and 1 of each half to columns 16 and 17
};

__device__ __forceinline__ void load_bwd(const uint16_t *wq, int lane, BwdW &b) {
    const int col = lane & 31, hf = lane >> 5;
    constexpr uint32_t kOne = 0x3F80u;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        u32x4 p, q;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int u = drow(8 * j + 2 * i, hf);
            p[i] = wq[kOffW2 + u * SV_MLP_HIDDEN + col] |
                   ((uint32_t)wq[kOffW2 + (u + 1) * SV_MLP_HIDDEN + col] << 16);
            q[i] = (col == u ? kOne : 0u) | (col == u + 1 ? kOne << 16 : 0u);
        }
        b.w2t[j] = as_operand(p);
        b.unit[j] = as_operand(q);
    }
    b.unit_g = as_operand(u32x4{col == 16 ? kOne : col == 17 ? kOne << 16 : 0u, 0u, 0u, 0u});
}

// A wave's tile in LDS, 32 units x 32 pixels (row pitch 36: fewer bank
// conflicts), and the order of its stores and loads: LDS serves a wave's
// accesses in order, so only the compiler has to keep them so.
constexpr int kTurnPitch = 36;
__device__ __forceinline__ void wave_order() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Row lane % 32 of the tile as the operand pair.
__device__ __forceinline__ void turn_read(const uint16_t *t, int lane, bf16x8 (&out)[2]) {
    const uint2 *row = (const uint2 *)(t + (lane & 31) * kTurnPitch);
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const uint2 a = row[4 * j + (lane >> 5)], b = row[4 * j + 2 + (lane >> 5)];
        out[j] = as_operand(u32x4{a.x, a.y, b.x, b.y});
    }
}

__device__ __forceinline__ void turn_store(uint16_t *t, int lane, int j, bf16x8 v) {
    const u32x4 d = __builtin_bit_cast(u32x4, v);
#pragma unroll
    for (int i = 0; i < 8; ++i)
        t[drow(8 * j + i, lane >> 5) * kTurnPitch + (lane & 31)] = (uint16_t)(d[i / 2] >> (i % 2 * 16));
}

// The operand pair (units along K) with its pixels along K instead.
template <bool LDS>
__device__ __forceinline__ void turn(const BwdW &w, uint16_t *t, int lane, const bf16x8 (&v)[2],
                                     bf16x8 (&out)[2]) {
    if constexpr (LDS) {
        turn_store(t, lane, 0, v[0]);
        turn_store(t, lane, 1, v[1]);
        wave_order();
        turn_read(t, lane, out);
        wave_order();
    } else {
        f32x16 d = {};
        d = mfma16(v[0], w.unit[0], d);
        d = mfma16(v[1], w.unit[1], d);
        out[0] = pack_operand(d, 0);
        out[1] = pack_operand(d, 1);
    }
}

// The features in columns 0..15 and the head gradients in 16 and 17, pixels
// along K (`g` counts in the lower half of the wave only).
template <bool LDS>
__device__ __forceinline__ void turn_xg(const BwdW &w, uint16_t *t, int lane, bf16x8 x, uint32_t g,
                                        bf16x8 (&out)[2]) {
    if constexpr (LDS) {
        turn_store(t, lane, 0, x);
        if (lane < 32) {
            t[16 * kTurnPitch + lane] = (uint16_t)g;
            t[17 * kTurnPitch + lane] = (uint16_t)(g >> 16);
        }
        wave_order();
        turn_read(t, lane, out);
        wave_order();
        if ((lane & 31) >= 18) out[0] = out[1] = as_operand(u32x4{});
    } else {
        f32x16 d = {};
        d = mfma16(x, w.unit[0], d);
        d = mfma16(as_operand(u32x4{lane < 32 ? g : 0u, 0u, 0u, 0u}), w.unit_g, d);
        out[0] = pack_operand(d, 0);
        out[1] = pack_operand(d, 1);
    }
}

// Sum over the 32 lanes of one half-wave (butterfly, fixed order).
__device__ __forceinline__ float half_sum(float v) {
#pragma unroll
    for (int m = 1; m < 32; m *= 2) v += __shfl_xor(v, m, 64);
    return v;
}

struct BwdAcc {
    f32x16 dw1, dw2, dw3;  // rows: units (of W1, W2; of W3: h2 units), columns lane % 32
    f32x16 db1, db2;       // this lane's units and pixels
    float db3a, db3b;      // this lane's pixels
};

// One 32-pixel block: g holds the two head gradients of pixel lane % 32 in
// bfloat16, in both halves of the wave.
template <bool LDS>
__device__ __forceinline__ void backward_block(const NetW &f, const BwdW &w, uint16_t *t, int lane,
                                               bf16x8 x, const FwdOut &r, uint32_t g,
                                               BwdAcc &acc) {
    const float g0 = __uint_as_float(g << 16), g1 = __uint_as_float(g & 0xFFFF0000u);
    f32x16 gh2;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        gh2[i] = r.a2[i] > 0.f ? fmaf(f.w3a[i], g0, f.w3b[i] * g1) : 0.f;
        acc.db2[i] += gh2[i];
    }
    const bf16x8 gb[2] = {pack_operand(gh2, 0), pack_operand(gh2, 1)};
    f32x16 gh1 = {};
    gh1 = mfma8(w.w2t[0], gb[0], gh1);
    gh1 = mfma8(w.w2t[1], gb[1], gh1);
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        gh1[i] = r.a1[i] > 0.f ? gh1[i] : 0.f;
        acc.db1[i] += gh1[i];
    }
    const bf16x8 g1b[2] = {pack_operand(gh1, 0), pack_operand(gh1, 1)};
    bf16x8 xg[2], g1t[2], g2t[2], h1t[2], h2t[2];
    turn_xg<LDS>(w, t, lane, x, g, xg);
    turn<LDS>(w, t, lane, g1b, g1t);
    turn<LDS>(w, t, lane, gb, g2t);
    turn<LDS>(w, t, lane, r.h1, h1t);
    turn<LDS>(w, t, lane, r.h2, h2t);
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        acc.dw1 = mfma16(g1t[j], xg[j], acc.dw1);
        acc.dw2 = mfma16(g2t[j], h1t[j], acc.dw2);
        acc.dw3 = mfma16(h2t[j], xg[j], acc.dw3);
    }
}

// A wave's blocks of 32 pixels.
template <bool LDS>
__device__ __forceinline__ void backward_wave(const MlpArgs &a, NetW &f, const BwdW &w,
                                              const float *s_b, uint16_t *t, int lane, int wave,
                                              BwdAcc &acc) {
    const int col = lane & 31, hf = lane >> 5;
    const int nblk = (a.npix + 31) / 32;
    acc = {};
    for (int blk = blockIdx.x * 4 + wave; blk < nblk; blk += gridDim.x * 4) {
        const int p = blk * 32 + col;
        const bool valid = p < a.npix;
        const bf16x8 x = load_x(a, valid ? p : 0, hf);
        float da = 0.f, dk = 0.f;
        if (valid) {
            const uint32_t o = plane_off(a, p);
            da = a.d_alpha ? a.d_alpha[o] : 0.f;
            dk = a.d_kappa ? a.d_kappa[o] : 0.f;
        }
        FwdOut r;
        // the binary32 parameters are read from LDS where they are used:
        // held over the loop their registers spill
        load_floats(s_b + vofs(0u), hf, f);
        forward_block(f, x, r);
        const float o0 = r.o0, o1 = r.o1;
        // the heads' slopes without cancellation: sigmoid' = e / (1 + e)^2
        // with e = exp(-|o|), and 1 - tanh^2 = 4 e / (1 + e)^2 with
        // e = exp(-2|o|) (1 - sg and 1 - th^2 would lose every digit once
        // the heads saturate)
        const float e0 = expf(-fabsf(o0)), d0 = 1.0f / (1.0f + e0);
        const float e1 = expf(-2.0f * fabsf(o1)), d1 = 1.0f / (1.0f + e1);
        const float kap = exp2f(2.0f * tanhf(o1));
        const float g0 = da * (1.0f - kAlphaMin) * (e0 * d0 * d0);
        const float g1 = dk * kap * 0.69314718055994531f * 2.0f * (4.0f * e1 * d1 * d1);
        if (hf == 0) {
            acc.db3a += g0;
            acc.db3b += g1;
        }
        backward_block<LDS>(f, w, t, lane, x, r, pack_bf16(g0, g1), acc);
    }
}

__global__ __launch_bounds__(256, 2) void mlp_backward_k(MlpArgs a) {
    __shared__ __align__(16) float s_part[4][SV_MLP_PARAMS];
    __shared__ u32x4 s_w[kNetStage];
    __shared__ __align__(16) float s_b[kNetFloats];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int col = lane & 31, hf = lane >> 5;
    NetStage ns;
    net_issue(a.params, a.wq, ns);
    net_store(ns, s_w, s_b);
    BwdW w;
    load_bwd(a.wq, lane, w);
    __syncthreads();
    NetW f;
    load_operands(s_w, lane, f);
    BwdAcc acc;
    float *sp = s_part[wave];
    backward_wave<false>(a, f, w, s_b, nullptr, lane, wave, acc);
    // a value that was not finite is in every element of its sums (above)
    const float any = acc.dw1[0] * 0.f + acc.dw2[0] * 0.f + acc.dw3[0] * 0.f;
    if (__any(!(any == 0.f)))
        backward_wave<true>(a, f, w, s_b, (uint16_t *)sp, lane, wave, acc);
    // this workgroup's partial gradient, flat order: the four waves' sums
    // joined in LDS
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int u = drow(i, hf);
        sp[kOffW2 + u * SV_MLP_HIDDEN + col] = acc.dw2[i];
        if (col < SV_MLP_IN) sp[kOffW1 + u * SV_MLP_IN + col] = acc.dw1[i];
        if (col == 16) sp[kOffW3 + u] = acc.dw3[i];
        if (col == 17) sp[kOffW3 + SV_MLP_HIDDEN + u] = acc.dw3[i];
        const float s1 = half_sum(acc.db1[i]), s2 = half_sum(acc.db2[i]);
        if (col == 0) {
            sp[kOffB1 + u] = s1;
            sp[kOffB2 + u] = s2;
        }
    }
    float s3a = half_sum(acc.db3a), s3b = half_sum(acc.db3b);
    s3a += __shfl_xor(s3a, 32, 64);
    s3b += __shfl_xor(s3b, 32, 64);
    if (lane == 0) {
        sp[kOffB3] = s3a;
        sp[kOffB3 + 1] = s3b;
    }
    __syncthreads();
    float *out = a.part + (size_t)blockIdx.x * SV_MLP_PARAMS;
    for (int j = threadIdx.x; j < SV_MLP_PARAMS; j += 256)
        out[j] = (s_part[0][j] + s_part[1][j]) + (s_part[2][j] + s_part[3][j]);
}

// Sum of the nw partial gradients, one parameter per column.  A workgroup
// owns 16 columns (one 64-byte piece of every partial) and splits the rows
// over 64 groups of lanes, whose sums a tree in LDS joins in a fixed order.
// One thread per parameter walking all rows put the whole sum on seven
// workgroups, each thread one chain of loads: of 8192 partials at 1920x1080
// 1910 us and of 1800 at 320x180 420 us, against 24 and 7; of the 512 and 225
// partials there are now, 5 and 4.  Shorter chains also round less.
constexpr int kRedCols = 16, kRedRows = 64;

__global__ __launch_bounds__(kRedCols *kRedRows) void mlp_reduce_k(const float *part, int nw,
                                                                   float scale, float *grad) {
    __shared__ float sum[kRedRows][kRedCols];
    const int c = threadIdx.x % kRedCols, g = threadIdx.x / kRedCols;
    const int j = blockIdx.x * kRedCols + c;
    float s = 0.f;
    if (j < SV_MLP_PARAMS) {
#pragma unroll 8
        for (int w = g; w < nw; w += kRedRows) s += part[(size_t)w * SV_MLP_PARAMS + j];
    }
    sum[g][c] = s;
    __syncthreads();
#pragma unroll
    for (int half = kRedRows / 2; half > 0; half /= 2) {
        if (g < half) sum[g][c] += sum[g + half][c];
        __syncthreads();
    }
    if (g == 0 && j < SV_MLP_PARAMS) grad[j] = sum[0][c] * scale;
}

inline void launch_reduce(const float *part, int nw, float scale, float *grad, hipStream_t s) {
    hipLaunchKernelGGL(mlp_reduce_k, dim3((SV_MLP_PARAMS + kRedCols - 1) / kRedCols),
                       dim3(kRedCols * kRedRows), 0, s, part, nw, scale, grad);
}

__global__ __launch_bounds__(256) void adam_k(float *params, uint16_t *wq, float *m, float *v,
                                              const float *g, int n, float lr, float b1, float b2,
                                              float eps, float c1, float c2) {
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= n) return;
    const float gj = g[j];
    const float mj = fmaf(b1, m[j], (1.0f - b1) * gj);
    const float vj = fmaf(b2, v[j], (1.0f - b2) * gj * gj);
    m[j] = mj;
    v[j] = vj;
    const float pj = params[j] - lr * (mj / c1) / (sqrtf(vj / c2) + eps);
    params[j] = pj;
    if (wq) wq[j] = to_bf16(pj);
}

// ---- truncated loss gradients ---------------------------------------------

struct AlphaGradArgs {
    const void *ctr, *ctg, *ctb, *cr, *cg, *cb;
    const float *hr, *hg, *hb, *yr, *yg, *yb, *alpha;
    const uint8_t *n;
    const void *z;
    float *d_alpha;
    int w, h, pitch;
    float tm_k;
};

// The two loss gradients are training-only passes, off the measured path.
// Their results are sums over channels (and, for kappa, over taps) of terms
// of either sign, so binary32 would lose digits to cancellation wherever the
// terms nearly balance; they are evaluated in binary64 from the stored
// (binary32 or binary16) inputs, like the definition they implement.
__device__ __forceinline__ double luma_d(double r, double g, double b) {
    return 0.2126 * r + 0.7152 * g + 0.0722 * b;
}

template <typename T>
__global__ __launch_bounds__(256) void alpha_grad_k(AlphaGradArgs a) {
    const int x = blockIdx.x * 64 + (threadIdx.x & 63), y = blockIdx.y * 4 + (threadIdx.x >> 6);
    if (x >= a.w || y >= a.h) return;
    const uint32_t o = (uint32_t)y * (uint32_t)a.pitch + (uint32_t)x;
    const int n = a.n[o];
    double g = 0.0;
    if (!empty_px(ldo<T>(a.z, o)) && n >= 1 && a.alpha[o] >= 1.0f / (float)n) {
        double c[3] = {ldo<T>(a.cr, o), ldo<T>(a.cg, o), ldo<T>(a.cb, o)};
        if (a.tm_k > 0.f) {
            const double sc = 1.0 / (1.0 + (double)a.tm_k * luma_d(c[0], c[1], c[2]));
            c[0] *= sc;
            c[1] *= sc;
            c[2] *= sc;
        }
        const double ct[3] = {ldo<T>(a.ctr, o), ldo<T>(a.ctg, o), ldo<T>(a.ctb, o)};
        const double hh[3] = {ldf(a.hr, o), ldf(a.hg, o), ldf(a.hb, o)};
        const double yy[3] = {ldf(a.yr, o), ldf(a.yg, o), ldf(a.yb, o)};
#pragma unroll
        for (int k = 0; k < 3; ++k) g += (ct[k] - yy[k]) / (yy[k] * yy[k] + 0.01) * (c[k] - hh[k]);
        g *= 2.0 / 3.0;
    }
    a.d_alpha[o] = (float)g;
}

struct KappaGradArgs {
    const void *cr, *cg, *cb;
    const float *var;
    const void *z, *dzdx, *dzdy, *nx, *ny, *nz;
    const float *kappa;
    const float *yr, *yg, *yb;
    const float *rr, *rg, *rb;  // optional: the colour whose residual is used
    float *d_kappa;
    int w, h, pitch, step;
    float sigma_z, sigma_n, sigma_l, eps_z, eps_l;
};

constexpr int kKappaLanes = 4;                // lanes of a pixel
constexpr int kKappaPx = 256 / kKappaLanes;   // pixels of a workgroup, in a row

// Sum over a pixel's lanes (butterfly: a fixed order).
__device__ __forceinline__ double px_sum(double v) {
#pragma unroll
    for (int m = kKappaLanes / 2; m > 0; m /= 2) v += __shfl_xor(v, m, 64);
    return v;
}

// Four lanes per pixel, taps read directly, in binary64 (see alpha_grad_k):
// lane s takes window taps s, s + 4, ... with every load issued before the
// first use.  The training frames are small, so one thread per pixel left the
// chip at one wave per SIMD walking 25 taps one after the other: 32 us per
// level at 320x180 against 20 (eight lanes: 23, its sums across lanes cost
// more).  The tap's three weights are one exponential of the summed exponents.
// The 3x3 variance prefilter runs over the in-image, non-empty taps, as in
// the level itself.
template <typename T>
__global__ __launch_bounds__(256) void kappa_grad_k(KappaGradArgs a) {
    constexpr int L = kKappaLanes, NT = (25 + L - 1) / L, NV = (9 + L - 1) / L;
    const int sub = threadIdx.x % L;
    const int x = blockIdx.x * kKappaPx + threadIdx.x / L, y = blockIdx.y;
    if (x >= a.w) return;  // whole pixels
    const uint32_t o = (uint32_t)y * (uint32_t)a.pitch + (uint32_t)x;
    const float zp32 = ldo<T>(a.z, o);
    float zq[NT], nxq[NT], nyq[NT], nzq[NT], rq[NT], gq[NT], bq[NT], vq[NV], vz[NV];
    bool in[NT], vin[NV];
#pragma unroll
    for (int j = 0; j < NT; ++j) {
        const int t = sub + L * j;
        const int qx = x + (t % 5 - 2) * a.step, qy = y + (t / 5 - 2) * a.step;
        in[j] = t < 25 && qx >= 0 && qx < a.w && qy >= 0 && qy < a.h;
        const uint32_t q = in[j] ? (uint32_t)qy * (uint32_t)a.pitch + (uint32_t)qx : o;
        zq[j] = ldo<T>(a.z, q);
        nxq[j] = ldo<T>(a.nx, q);
        nyq[j] = ldo<T>(a.ny, q);
        nzq[j] = ldo<T>(a.nz, q);
        rq[j] = ldo<T>(a.cr, q);
        gq[j] = ldo<T>(a.cg, q);
        bq[j] = ldo<T>(a.cb, q);
    }
#pragma unroll
    for (int j = 0; j < NV; ++j) {
        const int t = sub + L * j;
        const int qx = x + t % 3 - 1, qy = y + t / 3 - 1;
        vin[j] = t < 9 && qx >= 0 && qx < a.w && qy >= 0 && qy < a.h;
        const uint32_t q = vin[j] ? (uint32_t)qy * (uint32_t)a.pitch + (uint32_t)qx : o;
        vz[j] = ldo<T>(a.z, q);
        vq[j] = ldf(a.var, q);
    }
    const double np_[3] = {ldo<T>(a.nx, o), ldo<T>(a.ny, o), ldo<T>(a.nz, o)};
    const double gx = ldo<T>(a.dzdx, o), gy = ldo<T>(a.dzdy, o);
    const double lp = luma_d(ldo<T>(a.cr, o), ldo<T>(a.cg, o), ldo<T>(a.cb, o));
    const double kap = ldf(a.kappa, o);
    if (empty_px(zp32)) return;
    const double zp = zp32;
    double gs = 0.0, gw = 0.0;
#pragma unroll
    for (int j = 0; j < NV; ++j) {
        const int t = sub + L * j;
        if (!vin[j] || empty_px(vz[j])) continue;
        const double k = (t % 3 == 1 ? 0.5 : 0.25) * (t / 3 == 1 ? 0.5 : 0.25);
        gs += k * (double)vq[j];
        gw += k;
    }
    const double sg = sqrt(px_sum(gs) / px_sum(gw));
    const double sl = a.sigma_l;
    const double dl = sl * kap * sg + (double)a.eps_l;
    const double inv_dl = 1.0 / dl, dscale = sl * sg / (dl * dl);
    double sw = 0.0, sd = 0.0, sc[3] = {0.0, 0.0, 0.0}, sdc[3] = {0.0, 0.0, 0.0};
#pragma unroll
    for (int j = 0; j < NT; ++j) {
        const int t = sub + L * j, aa = t % 5 - 2, b = t / 5 - 2;
        if (!in[j] || (t != 12 && empty_px(zq[j]))) continue;
        const double ha = aa == 0 ? 0.375 : aa * aa == 1 ? 0.25 : 0.0625;
        const double hb = b == 0 ? 0.375 : b * b == 1 ? 0.25 : 0.0625;
        const double hh = ha * hb;
        const double cq[3] = {rq[j], gq[j], bq[j]};
        double w = 1.0, d = 0.0;
        if (t != 12) {
            const double den = (double)a.sigma_z *
                                   fabs(gx * (double)(a.step * aa) + gy * (double)(a.step * b)) +
                               (double)a.eps_z;
            const double ex = np_[0] - (double)nxq[j];
            const double ey = np_[1] - (double)nyq[j];
            const double ez = np_[2] - (double)nzq[j];
            const double cs = 1.0 - 0.5 * (ex * ex + ey * ey + ez * ez);
            // sigma_n log(cos), 0 where the normal weight is off or 1 whatever
            // sigma_n is (an infinite one times log(1) would be NaN)
            const double ln = a.sigma_n > 0.f && !(cs >= 1.0)
                                  ? (double)a.sigma_n * log(cs > 0.0 ? cs : 0.0)
                                  : 0.0;
            const double adl = fabs(lp - luma_d(cq[0], cq[1], cq[2]));
            w = exp(ln - fabs(zp - (double)zq[j]) / den - adl * inv_dl);
            d = w * adl * dscale;
        }
        sw += hh * w;
        sd += hh * d;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            sc[k] += hh * w * cq[k];
            sdc[k] += hh * d * cq[k];
        }
    }
    sw = px_sum(sw);
    sd = px_sum(sd);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        sc[k] = px_sum(sc[k]);
        sdc[k] = px_sum(sdc[k]);
    }
    if (sub != 0) return;
    const double yy[3] = {ldf(a.yr, o), ldf(a.yg, o), ldf(a.yb, o)};
    const float *rp[3] = {a.rr, a.rg, a.rb};
    double g = 0.0;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const double out = sc[k] / sw;
        const double der = (sdc[k] - out * sd) / sw;
        const double res = (a.rr ? (double)ldf(rp[k], o) : out) - yy[k];
        g += res / (yy[k] * yy[k] + 0.01) * der;
    }
    a.d_kappa[o] += (float)(g * (2.0 / 3.0));
}

// Workgroups of a network kernel over ngrp 64-pixel groups: one group per
// wave while that fits `per_cu` workgroups on each CU, then as many groups
// per wave as it takes.  The backward pass keeps its weights and its
// sums in registers, two waves per SIMD; more workgroups than are
// resident would only repeat its loads of the weights and its final sums.
// It walks blocks of 32 pixels, so a wave has two of them at least.  With one
// (twice the workgroups) the smallest frames gain, 64x64 13.9 -> 12.4 us and
// 480x270 21.3 -> 19.2, but at 256x256 and the trainer's 320x180 the doubled
// sums cost more: 15.9 -> 16.9 and 15.7 -> 17.8.
constexpr int kFwdPerCU = 8, kBwdPerCU = 2;

inline unsigned mlp_grid(int ngrp, int per_cu) {
    return (unsigned)std::max(1, std::min((ngrp + 3) / 4, 256 * per_cu));
}

inline bool valid_mlp(const sv_mlp *w) { return w && w->params && w->wq; }

}  // namespace sv

extern "C" int sv_mlp_forward(const sv_mlp *w, const void *feat, float *alpha, float *kappa,
                              sv_dims d, sv_stream stream) {
    using namespace sv;
    const int dc = check_dims(d);
    if (dc < 0 || !valid_mlp(w)) return SV_EINVAL;
    if (dc == 1) return SV_OK;
    if (!feat || ((uintptr_t)feat & 15u)) return SV_EINVAL;
    const span fs{(uintptr_t)feat, (uintptr_t)feat + (size_t)d.w * (size_t)d.h * 32u};
    if ((alpha && overlaps(plane_span(alpha, d, 4), fs)) ||
        (kappa && overlaps(plane_span(kappa, d, 4), fs)) ||
        (alpha && kappa && overlaps(plane_span(alpha, d, 4), plane_span(kappa, d, 4))))
        return SV_EALIAS;
    MlpArgs a{};
    a.params = w->params;
    a.wq = w->wq;
    a.feat = (const uint4 *)feat;
    a.alpha = alpha;
    a.kappa = kappa;
    a.w = d.w;
    a.h = d.h;
    a.pitch = d.pitch;
    a.npix = d.w * d.h;
    a.ngrp = (a.npix + 63) / 64;
    hipLaunchKernelGGL(mlp_forward_k, dim3(mlp_grid(a.ngrp, kFwdPerCU)), dim3(256), 0,
                       as_stream(stream), a);
    return hip_status(hipGetLastError());
}

extern "C" size_t sv_mlp_backward_work_bytes(sv_dims d) {
    using namespace sv;
    if (check_dims(d) < 0) return 0;
    // one partial gradient per wave of 2048 workgroups at most, a wave taking
    // 32 pixels: what callers have always sized their buffers by, and more
    // than the one partial per workgroup that is written
    const int wgs = std::max(1, std::min(((d.w * d.h + 31) / 32 + 3) / 4, 2048));
    return (size_t)wgs * 4u * SV_MLP_PARAMS * sizeof(float);
}

extern "C" int sv_mlp_backward(const sv_mlp *w, const void *feat, const float *d_alpha,
                               const float *d_kappa, float scale, float *grad, void *work,
                               sv_dims d, sv_stream stream) {
    using namespace sv;
    const int dc = check_dims(d);
    if (dc < 0 || !valid_mlp(w) || !grad) return SV_EINVAL;
    if (dc == 1) {  // no pixels: a zero gradient (a fill kernel, not a memset node)
        launch_reduce(nullptr, 0, 0.f, grad, as_stream(stream));
        return hip_status(hipGetLastError());
    }
    if (!feat || ((uintptr_t)feat & 15u) || !work) return SV_EINVAL;
    MlpArgs a{};
    a.params = w->params;
    a.wq = w->wq;
    a.feat = (const uint4 *)feat;
    a.d_alpha = d_alpha;
    a.d_kappa = d_kappa;
    a.part = (float *)work;
    a.w = d.w;
    a.h = d.h;
    a.pitch = d.pitch;
    a.npix = d.w * d.h;
    a.ngrp = (a.npix + 63) / 64;
    const span ws{(uintptr_t)work, (uintptr_t)work + sv_mlp_backward_work_bytes(d)};
    const span gs{(uintptr_t)grad, (uintptr_t)grad + SV_MLP_PARAMS * sizeof(float)};
    const span fs{(uintptr_t)feat, (uintptr_t)feat + (size_t)d.w * (size_t)d.h * 32u};
    if (overlaps(ws, gs) || overlaps(ws, fs) || overlaps(gs, fs) ||
        (d_alpha &&
         (overlaps(ws, plane_span(d_alpha, d, 4)) || overlaps(gs, plane_span(d_alpha, d, 4)))) ||
        (d_kappa &&
         (overlaps(ws, plane_span(d_kappa, d, 4)) || overlaps(gs, plane_span(d_kappa, d, 4)))))
        return SV_EALIAS;
    const unsigned grid = mlp_grid(a.ngrp, kBwdPerCU);
    hipStream_t s = as_stream(stream);
    hipLaunchKernelGGL(mlp_backward_k, dim3(grid), dim3(256), 0, s, a);
    launch_reduce((const float *)work, (int)grid, scale, grad, s);
    return hip_status(hipGetLastError());
}

extern "C" int sv_adam(float *params, uint16_t *wq, float *m, float *v, const float *grad,
                       int32_t n, int32_t t, const sv_adam_params *p, sv_stream stream) {
    using namespace sv;
    if (!params || !m || !v || !grad || !p || n < 0 || t < 1) return SV_EINVAL;
    if (n == 0) return SV_OK;
    const float c1 = 1.0f - powf(p->beta1, (float)t), c2 = 1.0f - powf(p->beta2, (float)t);
    hipLaunchKernelGGL(adam_k, dim3((n + 255) / 256), dim3(256), 0, as_stream(stream), params, wq,
                       m, v, grad, n, p->lr, p->beta1, p->beta2, p->eps, c1, c2);
    return hip_status(hipGetLastError());
}

extern "C" int sv_mlp_alpha_grad(const sv_rgb *c_t, const sv_rgb *cur, const sv_rgb *hist,
                                 const sv_rgb *y, const float *alpha, const uint8_t *n,
                                 const void *z, float tm_k, float *d_alpha, sv_dims d, sv_dtype t,
                                 sv_stream stream) {
    using namespace sv;
    if (!valid_dtype(t)) return SV_EDTYPE;
    const int dc = check_dims(d);
    if (dc < 0 || !c_t || !cur || !hist || !y) return SV_EINVAL;
    if (dc == 1) return SV_OK;
    const void *req[] = {c_t->r, c_t->g, c_t->b, cur->r, cur->g, cur->b, hist->r, hist->g,
                         hist->b, y->r, y->g, y->b, alpha, n, z, d_alpha};
    for (const void *q : req)
        if (!q) return SV_EINVAL;
    const size_t es = elem_size(t);
    const span so = plane_span(d_alpha, d, 4);
    const span ins[] = {plane_span(c_t->r, d, es), plane_span(c_t->g, d, es),
                        plane_span(c_t->b, d, es), plane_span(cur->r, d, es),
                        plane_span(cur->g, d, es), plane_span(cur->b, d, es),
                        plane_span(hist->r, d, 4), plane_span(hist->g, d, 4),
                        plane_span(hist->b, d, 4), plane_span(y->r, d, 4),
                        plane_span(y->g, d, 4), plane_span(y->b, d, 4),
                        plane_span(alpha, d, 4), plane_span(n, d, 1), plane_span(z, d, es)};
    for (const span &si : ins)
        if (overlaps(so, si)) return SV_EALIAS;
    AlphaGradArgs a{c_t->r, c_t->g, c_t->b, cur->r, cur->g, cur->b,
                    (const float *)hist->r, (const float *)hist->g, (const float *)hist->b,
                    (const float *)y->r, (const float *)y->g, (const float *)y->b, alpha, n, z,
                    d_alpha, d.w, d.h, d.pitch, tm_k};
    dim3 grid((d.w + 63) / 64, (d.h + 3) / 4);
    if (t == SV_F32)
        hipLaunchKernelGGL(alpha_grad_k<float>, grid, dim3(256), 0, as_stream(stream), a);
    else
        hipLaunchKernelGGL(alpha_grad_k<half_t>, grid, dim3(256), 0, as_stream(stream), a);
    return hip_status(hipGetLastError());
}

extern "C" int sv_atrous_kappa_grad(const sv_rgb *c_in, const float *var_in, const sv_gbuf *g,
                                    const float *kappa, const sv_rgb *y, const sv_rgb *ref,
                                    float *d_kappa, int32_t step, sv_dims d, sv_dtype t,
                                    const sv_atrous_params *p, sv_stream stream) {
    using namespace sv;
    if (!valid_dtype(t)) return SV_EDTYPE;
    const int dc = check_dims(d);
    if (dc < 0 || !c_in || !g || !y || !p || step < 1 || step > kMaxDim) return SV_EINVAL;
    if (dc == 1) return SV_OK;
    const void *req[] = {c_in->r, c_in->g, c_in->b, var_in, g->z, g->dzdx, g->dzdy, g->nx,
                         g->ny, g->nz, kappa, y->r, y->g, y->b, d_kappa};
    for (const void *q : req)
        if (!q) return SV_EINVAL;
    if (!(p->sigma_n >= 0.f)) return SV_EINVAL;
    if (ref && (!ref->r || !ref->g || !ref->b)) return SV_EINVAL;
    const size_t es = elem_size(t);
    const span so = plane_span(d_kappa, d, 4);
    if (ref && (overlaps(so, plane_span(ref->r, d, 4)) || overlaps(so, plane_span(ref->g, d, 4)) ||
                overlaps(so, plane_span(ref->b, d, 4))))
        return SV_EALIAS;
    const span ins[] = {plane_span(c_in->r, d, es), plane_span(c_in->g, d, es),
                        plane_span(c_in->b, d, es), plane_span(var_in, d, 4),
                        plane_span(g->z, d, es), plane_span(g->dzdx, d, es),
                        plane_span(g->dzdy, d, es), plane_span(g->nx, d, es),
                        plane_span(g->ny, d, es), plane_span(g->nz, d, es),
                        plane_span(kappa, d, 4), plane_span(y->r, d, 4),
                        plane_span(y->g, d, 4), plane_span(y->b, d, 4)};
    for (const span &si : ins)
        if (overlaps(so, si)) return SV_EALIAS;
    KappaGradArgs a{c_in->r, c_in->g, c_in->b, var_in, g->z, g->dzdx, g->dzdy, g->nx, g->ny,
                    g->nz, kappa, (const float *)y->r, (const float *)y->g, (const float *)y->b,
                    ref ? (const float *)ref->r : nullptr, ref ? (const float *)ref->g : nullptr,
                    ref ? (const float *)ref->b : nullptr,
                    d_kappa, d.w, d.h, d.pitch, step, p->sigma_z, p->sigma_n, p->sigma_l,
                    p->eps_z, p->eps_l};
    dim3 grid((d.w + kKappaPx - 1) / kKappaPx, d.h);
    if (t == SV_F32)
        hipLaunchKernelGGL(kappa_grad_k<float>, grid, dim3(256), 0, as_stream(stream), a);
    else
        hipLaunchKernelGGL(kappa_grad_k<half_t>, grid, dim3(256), 0, as_stream(stream), a);
    return hip_status(hipGetLastError());
}
