// Device code that the prompt scoring kernels share: tile products on the matrix cores and the logits' parameters.
#pragma once
#include "kf_device.h"
#include "kf_internal.h"

namespace kf {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int kTile = 32;
constexpr int kXcds = 8;

// One "group" = the 16 bytes a lane loads from a row: it feeds one bf16 MFMA
// (K = 16: 8 elements from each half of the wave) or four fp32 MFMAs (K = 2).
// Both operands use the same assignment of k indices to (wave half, element),
// so the contraction runs over every k exactly once.
template <typename T>
struct Mma;
template <>
struct Mma<bf16_t> {
    static __device__ __forceinline__ f32x16 group(const uint4& a, const uint4& b, f32x16 c) {
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a),
                                                       __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
    }
};
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
template <>
struct Mma<f16_t> {
    static __device__ __forceinline__ f32x16 group(const uint4& a, const uint4& b, f32x16 c) {
        return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
    }
};
template <>
struct Mma<float> {
    static __device__ __forceinline__ f32x16 group(const uint4& a, const uint4& b, f32x16 c) {
        c = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.x), __uint_as_float(b.x), c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.y), __uint_as_float(b.y), c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.z), __uint_as_float(b.z), c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.w), __uint_as_float(b.w), c, 0, 0, 0);
        return c;
    }
};

// Row of the 32x32 accumulator tile that register r of this lane holds
// (the column is lane % 32).
__device__ __forceinline__ int acc_row(int r, int half) { return (r >> 2) * 8 + half * 4 + (r & 3); }

// Issue priority of the wave from here on (0 or 1); nothing moves across.  Among a SIMD's waves a transcendental holds the vector
// unit for 8 cycles and nothing issues beside it, while two waves' simple fp32 or integer instructions go together at 2.4 cycles
// each (one alone takes 4; multiplies, shifts by funnel and SDWA forms 4.3).  Waves that reach their transcendentals at random
// break up each other's pairs.  With the hash of four logits first, then their logarithms, exponentials and quotients at priority 1,
// the transcendentals of a wave run back to back and the others' simple work is left together: the per-logit work by itself 28.8 ->
// 25.7 ns a wave and SIMD (batches of 8 or 16 logits 26.4 and 27.2; the priority the other way round 28.5).
template <int P>
__device__ __forceinline__ void wave_priority() {
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_setprio(P);
    __builtin_amdgcn_sched_barrier(0);
}

// y2 = log2(e) * (x + zeta)/tau for one logit, x = scale*acc - slope*dist.
// Gumbel (the method's adjustment) is the fast path: one hash, two hardware
// logarithms; zeta*log2(e) = -(log2(t) + log2(ln 2)) with t = -log2(u).
struct LogitParams {
    float sc1;      // scale * log2(e) / tau
    float slope1;   // slope * log2(e) / tau
    float inv_tau;
    float gz;       // -log2(ln 2) / tau : the constant part of the Gumbel term
    float c1;       // log2(e) / tau
    int noise;
    float fixed;    // the adjustment that is the same for every logit, times log2(e) / tau
};
__device__ __forceinline__ float logit2_gumbel(const LogitParams& lp, float acc, float dist, uint32_t folded) {
    const float l2t = hw_log2(neg_log2_uniform(mix32_folded(folded)));
    return fmaf(acc, lp.sc1, fmaf(dist, -lp.slope1, fmaf(l2t, -lp.inv_tau, lp.gz)));
}
__device__ __forceinline__ float logit2_other(const LogitParams& lp, float acc, float dist, uint32_t rkey,
                                              uint32_t k_pos) {
    return fmaf(acc, lp.sc1, fmaf(dist, -lp.slope1, zeta_log2e(lp.noise, rkey, k_pos) * lp.inv_tau));
}
// The same for adjustments that do not differ from logit to logit (none, constant), asked for once a tile: with the question in each
// logit, every logit was a block of instructions of its own.  With position bias, 8 x 32 heads x 4096 x 128 1409 -> 911 us, 64 x 32 x
// 1200 x 64 1410 -> 792, 32 x 20000 with flat slopes 6551 -> 4468.  (The Gaussian adjustment, 80 instructions, stays in blocks: in one
// stretch for 16 logits 4976 -> 5169 us.)
__device__ __forceinline__ float logit2_fixed(const LogitParams& lp, float acc, float dist) {
    return fmaf(acc, lp.sc1, fmaf(dist, -lp.slope1, lp.fixed));
}
__device__ __forceinline__ float fixed_adjustment(int noise) { return noise == kNoiseConstant ? kAdjMean * kLog2e : 0.0f; }

// <q, k> over the elements of the 16-byte pieces x and y
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
template <typename T>
__device__ __forceinline__ float dot_piece(const uint4& x, const uint4& y, float d) {
    const uint32_t xs[4] = {x.x, x.y, x.z, x.w}, ys[4] = {y.x, y.y, y.z, y.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        if constexpr (sizeof(T) == 4)
            d = fmaf(__uint_as_float(xs[e]), __uint_as_float(ys[e]), d);
        else if constexpr (__is_same(T, bf16_t))
            d = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, xs[e]), __builtin_bit_cast(bf16x2, ys[e]), d, false);
        else
            d = __builtin_amdgcn_fdot2(__builtin_bit_cast(f16x2, xs[e]), __builtin_bit_cast(f16x2, ys[e]), d, false);
    }
    return d;
}

}  // namespace kf
