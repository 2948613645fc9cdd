// The per-pixel network's forward pass on the matrix cores, shared by the
// network kernels and by the temporal kernel's learned mode.
//
// Matrix layout.  Each layer is computed transposed, Y^T = W X^T: A = the
// weights (32 output units x K inputs), B = K inputs x 32 pixels.  An operand
// is eight bfloat16 values of row l % 32 of A (column l % 32 of B) in lane l,
// for the K values 16 j + drow(0 .. 7, l / 32): the two operands of two
// v_mfma_f32_32x32x8_bf16 (K blocks of eight in order), or of one
// v_mfma_f32_32x32x16_bf16, whose halves may hold any K values as long as
// A's and B's agree.  The result D[8 (r/4) + 4 (l/32) + r % 4][l % 32] is in
// accumulator r = 0..15, so after a layer, accumulators 8 j .. 8 j + 7 of a
// lane, rounded in pairs, are that lane's operand j of the next layer:
// activations never leave registers in the forward pass.
//
// Which instruction: both round a 32-term sum alike (1.07e-8 rms of the
// summed magnitudes), but not to the same bits, and a pre-activation that
// moves by an ulp can round to another bfloat16 value.  The sums that are
// rounded to bfloat16 next stay with K blocks of eight; sums that are not,
// and exact ones, take the wider instruction, at half the issue time.
#pragma once
#include "sv_internal.h"

namespace sv {

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kOffW1 = 0, kOffB1 = 448, kOffW2 = 480, kOffB2 = 1504, kOffW3 = 1536,
              kOffB3 = 1600;
static_assert(kOffB3 + 2 == SV_MLP_PARAMS, "parameter layout");
constexpr float kAlphaMin = 0.05f;

__device__ __forceinline__ uint16_t to_bf16(float f) {
    uint32_t u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u);  // round to nearest even
    return (uint16_t)(u >> 16);
}

// Two values rounded to bfloat16 (nearest even), a in the low half: one
// v_cvt_pk_bf16_f32, where to_bf16 takes four instructions a value.
__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
    f32x2 v;
    v.x = a;
    v.y = b;
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}

__device__ __forceinline__ bf16x8 as_operand(u32x4 v) { return __builtin_bit_cast(bf16x8, v); }

// Accumulators 8 j .. 8 j + 7 as one operand.
__device__ __forceinline__ bf16x8 pack_operand(const f32x16 &v, int j) {
    u32x4 p;
#pragma unroll
    for (int i = 0; i < 4; ++i) p[i] = pack_bf16(v[8 * j + 2 * i], v[8 * j + 2 * i + 1]);
    return as_operand(p);
}

__device__ __forceinline__ f32x16 mfma16(bf16x8 a, bf16x8 b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// The same product as two K blocks of eight, in order.
__device__ __forceinline__ f32x16 mfma8(bf16x8 a, bf16x8 b, f32x16 c) {
    typedef short s16x8 __attribute__((ext_vector_type(8)));
    const s16x8 p = __builtin_bit_cast(s16x8, a), q = __builtin_bit_cast(s16x8, b);
    c = __builtin_amdgcn_mfma_f32_32x32x8bf16_1k(p.lo, q.lo, c, 0, 0, 0);
    return __builtin_amdgcn_mfma_f32_32x32x8bf16_1k(p.hi, q.hi, c, 0, 0, 0);
}

// Output unit (row of D) held in accumulator r by a lane of half `hf`.
__device__ __forceinline__ int drow(int r, int hf) { return 8 * (r >> 2) + 4 * hf + (r & 3); }

// ---- the forward pass's weight operands -------------------------------------
//
// Three operands of eight values per lane: W1 (unit `lane % 32`; features 14
// and 15 zero) and W2 (two).  The two-unit output layer runs on the vector
// units, sixteen terms per lane: its weights are held as binary32.
constexpr int kNetOps = 3, kOpW1 = 0, kOpW2 = 1;

// Where in the bfloat16 parameters element i of operand k comes from for
// this lane; -1: zero.
__device__ __forceinline__ int op_source(int k, int lane, int i) {
    const int col = lane & 31, hf = lane >> 5;
    if (k == kOpW1) {
        const int f = drow(i, hf);
        return f < SV_MLP_IN ? kOffW1 + col * SV_MLP_IN + f : -1;
    }
    return kOffW2 + col * SV_MLP_HIDDEN + drow(8 * (k - kOpW2) + i, hf);
}

__device__ __forceinline__ uint16_t op_element(const uint16_t *wq, int k, int lane, int i) {
    const int src = op_source(k, lane, i);
    const uint16_t v = wq[max(src, 0)];  // always in the array
    return src < 0 ? (uint16_t)0 : v;
}

// What one lane holds for the forward pass.
struct NetW {
    bf16x8 w1, w2[2];
    f32x16 b1, b2;    // biases at this lane's D rows
    f32x16 w3a, w3b;  // W3 rows 0 and 1 there (bfloat16 values)
    float b3a, b3b;
};

// The feature operand of one lane: features 4 hf .. 4 hf + 3 and 8 + 4 hf ..
// of a 32-byte feature row.
__device__ __forceinline__ bf16x8 feature_operand(const uint2 *row, int hf) {
    const uint2 a = row[hf], b = row[2 + hf];
    return as_operand(u32x4{a.x, a.y, b.x, b.y});
}

// Forward pass of one 32-pixel block.  x: this lane's operand of layer 1;
// returns the pre-activations (with biases), the activations as operands, and
// the two outputs of pixel lane % 32 (the same in both halves).
struct FwdOut {
    f32x16 a1, a2;
    bf16x8 h1[2], h2[2];
    float o0, o1;
};

// max(a, 0), NaN to 0, as one median: fmaxf costs a second instruction that
// quiets its argument.
__device__ __forceinline__ f32x16 relu(const f32x16 &a) {
    f32x16 r;
#pragma unroll
    for (int i = 0; i < 16; ++i) r[i] = __builtin_amdgcn_fmed3f(a[i], 0.f, INFINITY);
    return r;
}

__device__ __forceinline__ void forward_block(const NetW &f, bf16x8 x, FwdOut &r) {
    r.a1 = mfma8(f.w1, x, f.b1);
    const f32x16 p1 = relu(r.a1);
    r.h1[0] = pack_operand(p1, 0);
    r.h1[1] = pack_operand(p1, 1);
    r.a2 = mfma8(f.w2[0], r.h1[0], f.b2);
    r.a2 = mfma8(f.w2[1], r.h1[1], r.a2);
    const f32x16 p2 = relu(r.a2);
    r.h2[0] = pack_operand(p2, 0);
    r.h2[1] = pack_operand(p2, 1);
    float o0 = 0.f, o1 = 0.f;
#pragma unroll
    for (int i = 0; i < 16; i += 2) {
        const uint32_t h = __builtin_bit_cast(u32x4, r.h2[i >> 3])[(i & 7) >> 1];
        const float lo = __uint_as_float(h << 16), hi = __uint_as_float(h & 0xFFFF0000u);
        o0 = fmaf(f.w3a[i], lo, o0);
        o1 = fmaf(f.w3b[i], lo, o1);
        o0 = fmaf(f.w3a[i + 1], hi, o0);
        o1 = fmaf(f.w3b[i + 1], hi, o1);
    }
    o0 += __shfl_xor(o0, 32, 64);
    o1 += __shfl_xor(o1, 32, 64);
    r.o0 = o0 + f.b3a;
    r.o1 = o1 + f.b3b;
}

// The parameters one workgroup stages in LDS: the operands in lane order (an
// operand is then one 16-byte read per lane) and, as binary32, the biases of
// the hidden layers, the rows of W3 and the output biases.
constexpr int kNetB1 = 0, kNetB2 = SV_MLP_HIDDEN, kNetW3 = 2 * SV_MLP_HIDDEN,
              kNetB3 = 4 * SV_MLP_HIDDEN, kNetFloats = kNetB3 + 2;
constexpr int kNetStage = kNetOps * 64;  // 16-byte operand pieces
static_assert(kNetFloats <= 256, "one float per thread");

// Entry t of the packed floats.
__device__ __forceinline__ float net_float(const float *params, const uint16_t *wq, int t) {
    if (t >= kNetW3 && t < kNetB3)
        return __uint_as_float((uint32_t)wq[kOffW3 + t - kNetW3] << 16);
    return params[t < kNetB2   ? kOffB1 + t
                  : t < kNetW3 ? kOffB2 + t - kNetB2
                               : kOffB3 + t - kNetB3];
}

struct NetStage {  // one thread's share of the staging loads
    uint32_t w[kNetOps];
    float b;
};

// Issue this thread's staging loads (256 threads cover every value).
__device__ __forceinline__ void net_issue(const float *params, const uint16_t *wq, NetStage &ns) {
    const int t = threadIdx.x;
#pragma unroll
    for (int k = 0; k < kNetOps; ++k) {
        // dword t of operand k: lane t / 4, elements 2 (t % 4) and the next
        const int lane = t >> 2, i = 2 * (t & 3);
        ns.w[k] = op_element(wq, k, lane, i) | ((uint32_t)op_element(wq, k, lane, i + 1) << 16);
    }
    ns.b = net_float(params, wq, min(t, kNetFloats - 1));
}

// Store them; visible after the caller's next barrier.
__device__ __forceinline__ void net_store(const NetStage &ns, u32x4 *s_w, float *s_b) {
    const int t = threadIdx.x;
#pragma unroll
    for (int k = 0; k < kNetOps; ++k) ((uint32_t *)s_w)[k * 256 + t] = ns.w[k];
    if (t < kNetFloats) s_b[t] = ns.b;
}

__device__ __forceinline__ void load_operands(const u32x4 *s_w, int lane, NetW &f) {
    f.w1 = as_operand(s_w[kOpW1 * 64 + lane]);
#pragma unroll
    for (int j = 0; j < 2; ++j) f.w2[j] = as_operand(s_w[(kOpW2 + j) * 64 + lane]);
}

__device__ __forceinline__ void load_floats(const float *s_b, int hf, NetW &f) {
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        f.b1[r] = s_b[kNetB1 + drow(r, hf)];
        f.b2[r] = s_b[kNetB2 + drow(r, hf)];
        f.w3a[r] = s_b[kNetW3 + drow(r, hf)];
        f.w3b[r] = s_b[kNetW3 + SV_MLP_HIDDEN + drow(r, hf)];
    }
    f.b3a = s_b[kNetB3];
    f.b3b = s_b[kNetB3 + 1];
}

// alpha = 0.05 + 0.95 sigmoid(o0), kappa = 2^(2 tanh(o1)).
__device__ __forceinline__ void mlp_heads(float o0, float o1, float &alpha, float &kappa) {
    alpha = kAlphaMin + (1.0f - kAlphaMin) / (1.0f + expf(-o0));
    kappa = exp2f(2.0f * tanhf(o1));
}

}  // namespace sv
