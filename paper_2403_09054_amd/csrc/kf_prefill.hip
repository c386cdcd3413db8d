// Prompt-phase scoring of Keyformer for gfx950 (Sec. 3.4, Algorithm 1 prompt
// branch): for every unit
//     x_ij = scale*<Q_i,K_j> - slope*(i-j),  j <= i
//     z_i  = softmax_j((x_ij + zeta_ij)/tau)                 (Eq. 4, Eq. 11)
//     f[j] = sum_{i>=j} z_ij
// The logits are a dense n x n contraction: they are produced 32x32 tiles at a
// time on the matrix cores (MFMA).  The normaliser of row i must be known before
// any z_ij can be summed down a column, so two passes are made, each
// re-computing the logits instead of storing n^2 values:
//   pass 1  (row statistics)  computes the transposed tile K_tile * Q_tile^T so
//           that a lane owns ONE query and sees 16 of the tile's 32 keys: the
//           running max / sum of the row stay in the lane's registers.  Result:
//           c_i = log2(sum_j 2^(y2_ij)), y2 = log2(e)*(x+zeta)/tau, and the
//           row's noise key.
//   pass 2  (column sums)     computes Q_tile * K_tile^T so that a lane owns ONE
//           key and sees 16 of the tile's 32 queries: z_ij = 2^(y2_ij - c_i) is
//           added into the lane's column sum.
// Per logit the work is one 32-bit hash, two logarithms and one exponential; at
// temperature 1 (the method's in the prompt) the adjustment is a quotient, one
// logarithm and half a reciprocal instead.  That, not the MFMA rate, bounds the
// kernel (vector pipe 97 % busy, 1.9 T logit evaluations per second and pass at
// d = 128, 32768 rows), so the per-logit instruction count is what is trimmed:
// 16.7 a pass, 16 at temperature 1 (20.5 and 17.6 before the hash's first step
// left the loop, the masking compares moved into the edge tiles' branch and the
// accumulators into ordinary registers).  At temperature 1, 32 heads x 32768 rows
// 20.3 -> 17.0 to 17.9 ms from box to box, 256 x 4096 with position bias
// 3.13 -> 2.56 to 2.71.  With a logit's work in two phases, the second at a raised
// issue priority (wave_priority), on one box 17.05 -> 16.47 ms and, with the tiles
// that the bias leaves, 1667 -> 1559 us, the same results.  (Four waves per SIMD;
// three cost 2 % of the per-logit work, five and six spill.  The first of these
// two runs at 2.07 GHz, the second at 2.23: the chip's power, not only its issue.)
//
// With the Gumbel adjustment (the method; the others keep the plain form) pass 1
// sums every term against a reference exponent instead of searching each tile's
// maximum first: it starts at the row's own diagonal term (so the sum cannot
// vanish) and follows the sum's exponent upwards tile by tile; a tile whose sum
// overflows is summed again against a higher one.  Pass 1 leaves the row
// normaliser already combined with the adjustment's constant part; kernels built
// for "no position bias" drop that term.
//
// Prompts of up to 2048 rows mostly go another way, which evaluates a logit once (kf_strips.hip).
//
// Few units: the walks are cut into parts (plan_prefill).  Pass 1 then leaves a
// row's (reference, sum) per part, pass 2 puts them together while it loads, and a
// small launch adds the parts' column sums.
#include "kf_prefill.h"

namespace kf {

constexpr int kPrefillThreads = 256;  // 4 waves, 32 queries (pass 1) or keys (pass 2) each
// Waves per SIMD to compile for: four, three where a lane's own row takes 64 registers.  (With two or more the
// compiler keeps the MFMA accumulators in ordinary registers; allowed more than 256 registers per lane it puts
// them into accumulation registers and copies every one of a tile's 16 logits back with an instruction of its own.)
template <typename T, int D>
constexpr int kPrefillMinWaves = D * sizeof(T) >= 512 ? 3 : 4;

// Workgroup -> (unit, block of 128 rows, part of the block's tile walk).  Consecutive workgroup ids are dealt
// round-robin to the chip's 8 XCDs, each with an L2 of its own; the blocks of
// one unit re-read the same K / Q rows, so all blocks of a unit are given ids
// that are equal modulo 8 and therefore share one L2.  A block's later parts
// do not exist where its walk is short, and an XCD deals its workgroups to its shader engines in turn: with an even number
// of parts of a block in a row some engines would get the empty ones (40 heads x 6340 rows x 128, four parts, 1850 us;
// without parts 1129).  So an even number goes part by part (1003 us; 0.99 to 1.6 times as fast over 200 launches),
// an odd one block by block (0.98 to 1.09 times as fast as part by part; 16 x 2048 x 256, eleven parts, 95 against 103).
// With a position bias a group of 8 units starts at the next XCD each time: a head's work falls with its slope, and with
// equal ids modulo 8 one XCD would get the flattest slope of every 8 heads.
template <bool BIAS>
__device__ __forceinline__ void unit_and_block(int nblk, int parts, int64_t& u, int& blk, int& part) {
    const unsigned xcd = blockIdx.x % kXcds, local = blockIdx.x / kXcds;
    const unsigned group = local / (nblk * parts);
    u = (int64_t)group * kXcds + (BIAS ? (xcd + group) % kXcds : xcd);
    const int in_unit = (int)(local % (nblk * parts));
    blk = parts % 2 ? in_unit / parts : in_unit % nblk;
    part = parts % 2 ? in_unit % parts : in_unit / nblk;
}

// M + log2(S).  The hardware logarithm's error grows with its result and leans to one side: of a sum of 2^8 it
// left every row's normaliser low and with it every score high by 4e-7.  So the sum's exponent is taken off
// first (exact) and only its mantissa goes through the logarithm.
__device__ __forceinline__ float log2_of_sum(float M, float S) {
    const uint32_t b = __float_as_uint(S), ex = b >> 23;
    if (ex == 0u || ex >= 255u) return M + hw_log2(S);  // zero, denormal, infinite, NaN, negative
    return (M + (float)((int)ex - 127)) + hw_log2(__uint_as_float((b & 0x7FFFFFu) | 0x3F800000u));
}

// Log2 of a row's normaliser from the partial sums its parts left: sum over p of S_p * 2^(M_p).  A NaN among the row's
// logits makes the sum NaN, whichever part met it: it shows in the sum or, where the row's own diagonal term is the
// NaN, in the reference of every part while the sums are empty.
__device__ __forceinline__ float merged_normaliser(const float2* rec, size_t stride, int parts) {
    float M = -INFINITY, S = 0.0f;
    for (int p = 0; p < parts; ++p) {
        const float2 r = rec[p * stride];
        if (r.y <= 0.0f && r.x == r.x) continue;  // nothing in this part
        const float Mn = fmaxf(M, r.x);
        S = (M > -INFINITY ? S * hw_exp2(M - Mn) : 0.0f) + r.y * hw_exp2(r.x - Mn);
        M = Mn;
    }
    return log2_of_sum(M, S);
}

// ------------------------------------------------------------------ streamed tiles through LDS
// The four waves of a workgroup work on four 32-row groups of the SAME 128-row
// block and walk the same sequence of 32-row tiles of the other operand.  That
// tile is fetched once per workgroup (each thread a few 16-byte pieces, fully
// coalesced), parked in LDS and read from there as MFMA operands -- a quarter of
// the L2 traffic and D/4 fewer registers per lane than every wave loading its
// own copy, which is what lets more than two waves per SIMD overlap the MFMAs
// of one with the transcendental epilogue of another.  Two buffers; one
// barrier per tile.  Rows are padded by 16 bytes so that the 32 rows a wave
// reads in one instruction spread over the banks.
template <typename T, int D>
struct TileStage {
    static constexpr int kRowBytes = D * (int)sizeof(T);
    static constexpr int kPitch = kRowBytes + 16;                 // bytes between rows in LDS
    static constexpr int kPieces = kTile * kRowBytes / 16;        // 16-byte pieces of a tile
    static constexpr int NP = kPieces / kPrefillThreads;          // pieces per thread (1, 2 or 4)
    static constexpr int PPR = kRowBytes / 16;                    // pieces per row
    static constexpr int kBufBytes = kTile * kPitch;
    static_assert(kPieces % kPrefillThreads == 0, "a tile is a whole number of pieces per thread");

    // A thread's pieces of a tile on their way from memory to LDS (vector values, passed by value: an array of
    // uint4 handed around by reference ended up in scratch memory, each tile's loads waited for at once).
    struct Regs {
        u32x4_t r[NP];
    };
    // rows [row0, row0+32) of `rows` -> registers; rows from n on repeat row n-1.  A whole tile (workgroup-uniform)
    // is addressed by a scalar base and an offset that a thread keeps for all tiles, without vector arithmetic.
    static __device__ __forceinline__ Regs fetch(const T* rows, int row0, int n) {
        const char* base = (const char*)rows + (size_t)row0 * kRowBytes;
        Regs reg;
        if (row0 + kTile <= n) {
#pragma unroll
            for (int i = 0; i < NP; ++i) reg.r[i] = *(const u32x4_t*)(base + (threadIdx.x + i * kPrefillThreads) * 16u);
        } else {
            const uint32_t last = (uint32_t)(n - 1 - row0);
#pragma unroll
            for (int i = 0; i < NP; ++i) {
                const uint32_t p = threadIdx.x + i * kPrefillThreads;
                reg.r[i] = *(const u32x4_t*)(base + (min(p / PPR, last) * kRowBytes + (p % PPR) * 16u));
            }
        }
        return reg;
    }
    static __device__ __forceinline__ void park(char* buf, const Regs reg) {
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            const int p = threadIdx.x + i * kPrefillThreads;
            *(u32x4_t*)(buf + (p / PPR) * kPitch + (p % PPR) * 16) = reg.r[i];
        }
    }
    // The 32x32 products of the parked tile (A operand) with the lane's own row `own` (B operand).  The LDS reads
    // go out in batches ahead of their MFMAs: left to itself the compiler reads, waits and multiplies one 16-byte
    // piece at a time, D/16 LDS round trips per tile that only other waves can cover.
    static constexpr int kGroups = D / (2 * ElemTraits<T>::kPerVec);
    static constexpr int kBatch = kGroups < 8 ? kGroups : 8;
    static __device__ __forceinline__ f32x16 products(const char* buf, int n0, int half, const uint4 (&own)[kGroups]) {
        const char* p = buf + n0 * kPitch + half * 16;
        f32x16 acc;
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
#pragma unroll
        for (int g0 = 0; g0 < kGroups; g0 += kBatch) {
            uint4 a[kBatch];
#pragma unroll
            for (int g = 0; g < kBatch; ++g) a[g] = *(const uint4*)(p + (g0 + g) * 32);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int g = 0; g < kBatch; ++g) acc = Mma<T>::group(a[g], own[g0 + g], acc);
        }
        return acc;
    }
};

// ------------------------------------------------------------------ tiles that a position bias rules out
// With a position bias of positive slope the far tiles of a walk cannot matter: by Cauchy-Schwarz
//     y2_ij <= |q_i| |k_j| scale log2(e)/tau + (largest adjustment) - slope log2(e)/tau (i - j)
// for every finite input.  A walk that is not cut into parts begins at the diagonal.  kSkipAhead tiles behind the block's own
// it looks at what its rows (pass 2: columns) have gathered so far, and leaves out the tiles at the far end whose terms, by
// that bound, all together stay below 2^-28 of it: less than a rounding of the result.  (Against what has been gathered, not
// against the diagonal term alone, which is 2^15 smaller in the rows that decide; and the terms' bounds added up tile by
// tile, the far ones being smaller by the bias, instead of n times the largest: 22 of 95 bits that the bias has to outweigh.
// One layer of 8 x 32 heads x 4096 rows with slopes 2^(-h/4), h = 1..32, 2676 us with all tiles: 1678 against the diagonal terms;
// 1556 so, later, and 1470 against the sums on the same box.  Sums that begin with their largest tiles are added up with a carry,
// `lost` below and carry_sum, so that the error against float64 is none the larger.)
// A part of a walk does not have the others' sums: pass 1 takes the diagonal term instead, and so does pass 2, there with n
// times the largest term for the sum over the tiles, whose normalisers it has not.
// The bounds are taken from the data (norms, sums and normalisers per tile); a NaN or an infinity in any of them makes every
// comparison below fail, and the tile is walked.  A unit whose largest possible bias cannot outweigh the constants takes none
// of this (skip_reach).
constexpr float kSkipBits = 29.0f;  // 28, and one for the rounding of the bound itself

// Largest adjustment zeta log2(e) that the generator can produce (Gumbel: -ln(-ln(1 - 2^-24)) log2(e) = 24; Gaussian: radius
// sqrt(2 ln 2^24)).
__device__ __forceinline__ float largest_adjustment(int noise) {
    return noise == kNoiseGumbel ? 24.01f : noise == kNoiseGaussian ? (kAdjMean + kAdjStd * 5.77f) * 1.4427f + 0.01f
         : noise == kNoiseConstant ? kAdjMean * 1.4427f + 0.01f : 0.0f;
}
// What the bias has to outweigh, for vectors of no length: a walk whose bias stays below it is not searched (the search is
// a trip to memory ahead of the walk, 1 to 3 us of a launch).
__device__ __forceinline__ float skip_reach(int noise, float inv_tau, int n) {
    return largest_adjustment(noise) * inv_tau + kSkipBits + hw_log2((float)n);
}
constexpr int kSkipAhead = 2;
constexpr float kSkipTileBits = kSkipBits + 5.0f;  // a tile's terms of a row (or column): 32 of the bound each
__device__ __forceinline__ float not_above(float x) { return x > -INFINITY ? x : -INFINITY; }  // lower bound: NaN is none
__device__ __forceinline__ float wave_min(float v) { return -wave_max(-v); }
// Of `count` tiles in the order of a walk's far end: how many of the first ones may be left out, all together.  term(x): what
// tile x can add to the most affected row, of what the row may lose.  The same in every wave that asks.
template <typename F>
__device__ __forceinline__ int tiles_ruled_out(int count, F term) {
    const int lane = threadIdx.x & 63;
    float before = 0.0f;
    for (int x0 = 0; x0 < count; x0 += kWave) {
        float e = x0 + lane < count ? term(x0 + lane) : INFINITY;
#pragma unroll
        for (int o = 1; o < kWave; o <<= 1) {
            const float t = __shfl_up(e, o, kWave);
            if (lane >= o) e += t;
        }
        const unsigned long long most = __ballot(!(before + e <= 1.0f));
        if (most) return x0 + __ffsll((long long)most) - 1;
        before += __shfl(e, kWave - 1, kWave);
    }
    return count;
}
// The plain form's walk from the diagonal: what has been summed since the last call joins the walk's sum `all`, against the
// reference M from now on (Mall: the one before), with a carry.  (A function: written as a lambda in the kernel, it changes where
// the compiler puts the blocks of the forms that have none of it.)
constexpr int kCarryTiles = 4;
__device__ __forceinline__ void carry_sum(float M, float& Ssum, float& all, float& Mall, float& lost) {
    const float down = hw_exp2(Mall - M);
    all *= down;
    lost *= down;
    Mall = M;
    const float add = Ssum - lost, sum = all + add;
    lost = (sum - all) - add;
    all = sum;
    Ssum = 0.0f;
}
// Norm from its square: never too small (256 squares that underflowed are 3e-36 together), infinite where the square is no
// number (every maximum that follows would pass a NaN over).
__device__ __forceinline__ float norm_bound(float sq) { return sq < INFINITY ? sqrtf(fmaxf(sq, 4e-36f)) * 1.0001f : INFINITY; }

// ------------------------------------------------------------------ pass 1
// Largest |k| of every 32-row tile of a cached head, for the bound above: a wave a tile, one read of K.
constexpr int kNormWaves = 4;
template <typename T, int D>
__global__ void __launch_bounds__(kNormWaves * kWave) prefill_key_norms_kernel(const PrefillArgs a, int64_t kv_units) {
    constexpr int LPR = D * (int)sizeof(T) / 16, RPL = kWave / LPR, NL = kTile / RPL;  // lanes a row, rows a load, loads a tile
    const int64_t u = blockIdx.x;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, jt = blockIdx.y * kNormWaves + wv;
    if (u >= kv_units) return;
    const int n = a.seq_n ? a.seq_n[(u / (a.H / a.G)) % a.B] : a.n;
    if (n < 1 || n > a.n || jt * kTile >= n) return;
    float slope = 0.0f;
    for (int g = 0; g < a.G; ++g) slope = fmaxf(slope, a.slopes[(u * a.G + g) % a.H]);
    // none of the heads looks (the product in the order of the passes': the two sides of the limit must be the same there)
    if (!(slope * (a.inv_tau * kLog2e) * (float)n > skip_reach(a.noise, a.inv_tau, n))) return;
    const char* Ku = (const char*)a.K + (size_t)u * a.cap * D * sizeof(T);
    uint4 r[NL];
#pragma unroll
    for (int i = 0; i < NL; ++i)
        r[i] = *(const uint4*)(Ku + (size_t)min(jt * kTile + i * RPL + lane / LPR, n - 1) * D * sizeof(T) + (lane % LPR) * 16);
    float most = 0.0f;
#pragma unroll
    for (int i = 0; i < NL; ++i) {
        float sq = dot_piece<T>(r[i], r[i], 0.0f);
#pragma unroll
        for (int o = 1; o < LPR; o <<= 1) sq += __shfl_xor(sq, o, kWave);
        most = fmaxf(most, norm_bound(sq));
    }
    most = wave_max(most);
    if (lane == 0) a.ws_kn[(size_t)u * (a.n_pad / kTile) + jt] = most;
}

// s + sum of e[i]/t[i], t = -l2u: the Gumbel factor (-ln u)^(-1/tau) at temperature 1 (its ln 2 rides in the
// exponents).  Two quotients share a reciprocal, e0/t0 + e1/t1 = (e0*t1 + e1*t0) / (t0*t1); t lies in [8e-8, 24].
__device__ __forceinline__ float add_over_t(const float (&e)[4], const float (&l2u)[4], float s) {
#pragma unroll
    for (int i = 0; i < 4; i += 2) {
        const float num = fmaf(e[i], l2u[i + 1], e[i + 1] * l2u[i]);
        s = fmaf(-num, __builtin_amdgcn_rcpf(l2u[i] * l2u[i + 1]), s);
    }
    return s;
}

// Sum over this lane's 16 logits of a tile of 2^(y2 - reference), Gumbel adjustment; `base` is the
// adjustment's constant part less the reference (and the position bias of the lane's first key), rfold the
// folded row key, kfold the folded key positions of the tile (this lane's: words 8*q4 + 4*half + e).  MASK:
// keep only the keys up to `room` places behind the lane's first one (the tile crosses the diagonal).
template <bool BIAS, bool MASK, bool TAU1>
__device__ __forceinline__ float tile_sum(const LogitParams& lp, const f32x16& acc, float base, uint32_t rfold,
                                          const uint32_t* kfold, int half, int room) {
    float ssum = 0.0f;
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4) {
        const uint4 k4 = *(const uint4*)&kfold[q4 * 8 + half * 4];
        const uint32_t ks[4] = {k4.x, k4.y, k4.z, k4.w};
        float e[4], l2u[4];
        uint32_t bits[4];
#pragma unroll
        for (int e4 = 0; e4 < 4; ++e4) bits[e4] = mix32_folded(rfold ^ ks[e4]);
        wave_priority<1>();
#pragma unroll
        for (int e4 = 0; e4 < 4; ++e4) l2u[e4] = hw_log2(uniform_of(bits[e4]));
#pragma unroll
        for (int e4 = 0; e4 < 4; ++e4) {
            const int ro = q4 * 8 + e4;
            // position bias -slope*(dist0 - ro): its dist0 part rides in `base`, the ro part is a literal multiple
            float t = BIAS ? fmaf(lp.slope1, (float)ro, base) : base;
            if (!TAU1) t = fmaf(hw_log2(-l2u[e4]), -lp.inv_tau, t);
            e[e4] = hw_exp2(fmaf(acc[q4 * 4 + e4], lp.sc1, t));
            if (MASK) e[e4] = ro <= room ? e[e4] : 0.0f;
        }
        ssum = TAU1 ? add_over_t(e, l2u, ssum) : (((ssum + e[0]) + e[1]) + e[2]) + e[3];
        wave_priority<0>();
    }
    return ssum;
}

// GUMBEL: the method's adjustment, trimmed form; otherwise any adjustment, plain form.  BIAS: slopes given.  TAU1:
// Gumbel at temperature 1, the method's temperature of the prompt: the adjustment's exponential is a quotient, one
// logarithm and one multiply-add per logit less against half a reciprocal and three cheaper operations.
template <typename T, int D, bool GUMBEL, bool BIAS, bool TAU1>
__global__ void __launch_bounds__(kPrefillThreads, (kPrefillMinWaves<T, D>)) prefill_rowstats_kernel(const PrefillArgs a, int nblk, int64_t units) {
    constexpr int EPV = ElemTraits<T>::kPerVec;
    constexpr int NG = D / (2 * EPV);
    using Stage = TileStage<T, D>;
    __shared__ __attribute__((aligned(16))) char kbuf[2][Stage::kBufBytes];
    __shared__ __attribute__((aligned(16))) uint32_t kfold[2][kTile];  // folded positions of the tile's keys
    __shared__ float2 wstat[kPrefillThreads / kWave];  // of a wave's rows: largest norm, smallest sum so far (or diagonal term)
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n0 = lane & 31, half = lane >> 5;
    int64_t u;
    int blk, part;
    unit_and_block<BIAS>(nblk, a.parts, u, blk, part);
    if (u >= units) return;  // workgroup-uniform
    const int rb = nblk - 1 - blk;  // longest rows first
    const int h = (int)(u % a.H), b = (int)((u / a.H) % a.B), l = a.layer0 + (int)(u / ((int64_t)a.H * a.B));
    const int n = a.seq_n ? a.seq_n[b] : a.n;  // this sequence's prompt length; rows n..a.n-1 are padding
    // workgroup-uniform exits: a length out of range (the second pass reports it), a block inside the padding
    if (n < 1 || n > a.n || rb * (4 * kTile) >= n) return;
    // this workgroup's tiles [jt_first, jt_last] of the block's walk
    int jt_first = part * a.part_tiles;
    const int jt_last = min(min(rb * (4 * kTile) + 4 * kTile - 1, n - 1) / kTile, jt_first + a.part_tiles - 1);
    if (jt_first > jt_last) return;  // workgroup-uniform: the block has fewer parts
    const int i0 = rb * (4 * kTile) + wv * kTile;
    const bool active = i0 < n;  // wave-uniform; inactive waves still fetch tiles and meet the barriers
    const int i = i0 + n0;
    const T* Qu = (const T*)a.Q + (size_t)u * a.n * D;
    const T* Ku = (const T*)a.K + (size_t)(u / a.G) * a.cap * D;  // G query heads read one cached head

    uint4 bq[NG];
    {
        const T* row = Qu + (size_t)min(i, n - 1) * D + half * EPV;
#pragma unroll
        for (int g = 0; g < NG; ++g) bq[g] = *(const uint4*)(row + g * 2 * EPV);
    }
    const bool rnd = (a.noise == kNoiseGumbel || a.noise == kNoiseGaussian);
    const uint32_t rkey = rnd ? row_key(unit_key(a.seeds[b], (uint32_t)l, (uint32_t)h), (uint32_t)i) : 0u;
    LogitParams lp;
    lp.c1 = a.inv_tau * kLog2e;
    lp.sc1 = a.scale * lp.c1;
    lp.slope1 = (BIAS ? a.slopes[h] : 0.0f) * lp.c1;
    lp.inv_tau = a.inv_tau;
    lp.gz = -kLog2Ln2 * a.inv_tau;
    lp.noise = a.noise;
    if constexpr (!GUMBEL) lp.fixed = fixed_adjustment(a.noise) * a.inv_tau;
    const bool fixed = !GUMBEL && (a.noise == kNoiseNone || a.noise == kNoiseConstant);  // the same adjustment for every logit
    // a logit's hash input is rkey ^ (k_pos * kKposMul); both sides enter the loop folded (mix32's first step),
    // the keys' side as a table that travels with the tile
    const uint32_t rfold = fold16(rkey);
    auto park_keys = [&](int buf, int jt) {
        if (threadIdx.x < kTile) kfold[buf][threadIdx.x] = fold16((uint32_t)(jt * kTile + threadIdx.x) * kKposMul);
    };

    // The plain form starts from the lowest finite reference: with -inf a tile whose unmasked logits are all NaN would not be
    // told from one that has none.
    float M = GUMBEL ? -INFINITY : -0x1.fffffep127f, Ssum = 0.0f;
    const float reach = BIAS ? skip_reach(a.noise, a.inv_tau, n) : 0.0f;
    const bool skips = BIAS && a.ws_kn && lp.slope1 * (float)n > reach;  // of the unit
    float own = -INFINITY, qnorm = 0.0f;                     // the row's diagonal term, the norm of its query
    // how many of the walk's first `count` tiles do not matter to the block's rows (wstat is there)
    auto ruled_out = [&](int count) {
        const float* kn = a.ws_kn + (size_t)(u / a.G) * (a.n_pad / kTile);
        const float most = largest_adjustment(a.noise) * a.inv_tau + kSkipTileBits;
        return __builtin_amdgcn_readfirstlane(tiles_ruled_out(count, [&](int jt) {
            const float norm = kn[jt] * fabsf(lp.sc1);
            float e = 0.0f;
            for (int v = 0; v < kPrefillThreads / kWave; ++v) {
                const int first = rb * (4 * kTile) + v * kTile;  // the wave's first row
                if (first >= n) break;
                const float bias = lp.slope1 * (float)(first - (jt * kTile + kTile - 1));
                e += hw_exp2(wstat[v].x * norm + most - bias - wstat[v].y);
            }
            return e;
        }));
    };
    if (GUMBEL || skips) {
        // Reference exponent of the row's sum: its own diagonal term y2_ii, formed here from the query's and the
        // key's elements this lane holds (both halves of the wave added up).  It is a term of the sum, so the
        // sum against it cannot vanish however far below it the others lie.
        const T* krow = Ku + (size_t)min(i, n - 1) * D + half * EPV;
        float dot = 0.0f;
#pragma unroll
        for (int g = 0; g < NG; ++g) dot = dot_piece<T>(bq[g], *(const uint4*)(krow + g * 2 * EPV), dot);
        dot += __shfl_xor(dot, 32, kWave);
        own = GUMBEL ? logit2_gumbel(lp, dot, 0.0f, rfold ^ fold16((uint32_t)i * kKposMul)) : logit2_other(lp, dot, 0.0f, rkey, (uint32_t)i);
        if (GUMBEL) M = own > -INFINITY || own != own ? own : 0.0f;  // (no reference: every other term would be infinite)
    }
    if (skips) {
        float sq = 0.0f;
#pragma unroll
        for (int g = 0; g < NG; ++g) sq = dot_piece<T>(bq[g], bq[g], sq);
        qnorm = wave_max(norm_bound(sq + __shfl_xor(sq, 32, kWave)));
        if (a.parts > 1) {
            const float least = wave_min(not_above(own));
            if (lane == 0) wstat[wv] = make_float2(qnorm, least);
            if (lane == 0 && active && part == 0) a.ws_tile[(size_t)u * (a.n_pad / kTile) + i0 / kTile] = make_float4(qnorm, least, 0.0f, 0.0f);
            if (lp.slope1 * (float)((rb * 4 - jt_first) * kTile) > reach) {  // workgroup-uniform: the part's first tile may be (1 x 8 x 17000 without adjustment 558 -> 549 us)
                __syncthreads();
                jt_first = max(jt_first, ruled_out(min(rb * 4, jt_last + 1)));  // behind jt_last: nothing is left of the part
            }
        }
    }
    const int jt_end = min(i0 + kTile - 1, n - 1) / kTile;  // this wave's last key tile
    // What rounding has added to the sum so far: from the diagonal down the largest tiles come first, and the others would each
    // lose half a unit of the whole sum's last place (2.2e-7 of a score instead of 2.0e-7, 256 x 4096).
    float lost = 0.0f;
    // The plain form takes a sum of kCarryTiles tiles at a time and adds that to the walk's (`all`, against reference Mall).
    // Scores without adjustment against float64, slope 1e-3: 20000 rows 4.0e-7 -> 0.4e-7, 32768 rows 6.6e-7 -> 0.4e-7 (upwards, without: 0.8e-7).
    float all = 0.0f, Mall = M;
    // the walk: upwards, or with a position bias from the diagonal down
    const int jt_begin = BIAS ? max(jt_last, jt_first) : min(jt_first, jt_last), looks_at = skips && a.parts == 1 ? rb * 4 - kSkipAhead : -1;
    typename Stage::Regs stage = Stage::fetch(Ku, min(jt_begin, jt_last) * kTile, n);
    Stage::park(kbuf[0], stage);
    if constexpr (GUMBEL) park_keys(0, jt_begin);
    __syncthreads();
    for (int jt = BIAS ? jt_last : jt_first, cur = 0; BIAS ? jt >= jt_first : jt <= jt_last; jt += BIAS ? -1 : 1, cur ^= 1) {
        // the next tile (the last one again at the end: rows stay in range), in flight during this tile's work;
        // asking two tiles ahead measured the same
        const int jt_next = BIAS ? max(jt - 1, jt_first) : min(jt + 1, jt_last);
        stage = Stage::fetch(Ku, jt_next * kTile, n);
        if (active && jt <= jt_end) {
            const char* kb = kbuf[cur];
            const f32x16 acc = Stage::products(kb, n0, half, bq);
            const int jb = jt * kTile;
            const int jl = jb + half * 4;                       // first key of this lane in the tile
            const float dist0 = (float)(i - jl);
            if constexpr (GUMBEL) {
                // every term against the reference as it stands, (gz - M) folded into the chain: no search for the
                // tile's maximum, no subtraction per logit.  A later, larger logit just gives a term above one.
                // Only the wave's last tile crosses the diagonal.  Its masking compares are kept inside their branch
                // (the empty asm makes them depend on it): hoisted, they cost every tile an instruction per logit.
                const bool diag = jt == jt_end;
                for (int attempt = 0;; ++attempt) {
                    const float base = BIAS ? fmaf(dist0, -lp.slope1, lp.gz - M) : lp.gz - M;
                    float ssum;
                    if (diag) {
                        int room = i - jl;
                        asm volatile("" : "+v"(room));
                        ssum = tile_sum<BIAS, true, TAU1>(lp, acc, base, rfold, kfold[cur], half, room);
                    } else {
                        ssum = tile_sum<BIAS, false, TAU1>(lp, acc, base, rfold, kfold[cur], half, 0);
                    }
                    const float add = BIAS ? ssum - lost : ssum;
                    const float Snew = Ssum + add;
                    // a sum beyond fp32 in some lane (a logit 2^120 above its row's reference): that lane raises its
                    // reference and the wave sums the tile again (the other lanes arrive at the same sums as
                    // before); bounded, so that NaN inputs end as NaN
                    const bool over = !(Snew < 0x1p120f);
                    if (__any(over) && attempt < 64) {
                        if (over) {
                            M += 100.0f;
                            Ssum *= 0x1p-100f;
                            lost *= 0x1p-100f;
                        }
                        continue;
                    }
                    if (BIAS) lost = Snew < INFINITY ? (Snew - Ssum) - add : 0.0f;
                    Ssum = Snew;
                    break;
                }
                // the reference follows the sum's exponent (exact: a power of two)
                if (Ssum > 0x1p40f) {
                    const int sh = (int)(__float_as_uint(Ssum) >> 23) - 127;
                    M += (float)sh;
                    Ssum = __uint_as_float(__float_as_uint(Ssum) - ((uint32_t)sh << 23));
                    if (BIAS) lost *= __uint_as_float((uint32_t)(127 - min(sh, 126)) << 23);
                }
            } else {
            float y2[16];
            if (fixed) {  // (asked once a tile, not for each logit)
#pragma unroll
                for (int r = 0; r < 16; ++r) y2[r] = logit2_fixed(lp, acc[r], dist0 - (float)((r >> 2) * 8 + (r & 3)));
            } else {
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int ro = (r >> 2) * 8 + (r & 3);
                    y2[r] = logit2_other(lp, acc[r], dist0 - (float)ro, rkey, (uint32_t)(jl + ro));
                }
            }
            if (jb + kTile - 1 > i0) {  // the tile crosses the diagonal for some lane: causal mask
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int ro = (r >> 2) * 8 + (r & 3);
                    y2[r] = (jl + ro <= i) ? y2[r] : -INFINITY;
                }
            }
            float tmax = y2[0];
#pragma unroll
            for (int r = 1; r < 16; ++r) tmax = fmaxf(tmax, y2[r]);
            const float Mn = fmaxf(M, tmax);
            float ssum = 0.0f;
#pragma unroll
            for (int r = 0; r < 16; ++r) ssum += hw_exp2(y2[r] - Mn);
            Ssum = Ssum * hw_exp2(M - Mn) + ssum;
            M = Mn;
            if constexpr (BIAS) {
                if (jt % kCarryTiles == 0) carry_sum(M, Ssum, all, Mall, lost);
            }
            }
        }
        if (jt != jt_next) {
            Stage::park(kbuf[cur ^ 1], stage);
            if constexpr (GUMBEL) park_keys(cur ^ 1, jt_next);
        }
        const bool looks = BIAS && jt == looks_at;  // workgroup-uniform
        if (looks) {
            float S = Ssum;
            if constexpr (BIAS && !GUMBEL) {
                carry_sum(M, Ssum, all, Mall, lost);
                S = all;
            }
            const float M2 = __shfl_xor(M, 32, kWave), S2 = __shfl_xor(S, 32, kWave), Mt = fmaxf(M, M2);
            const float c = log2_of_sum(Mt, (M > -INFINITY ? S * hw_exp2(M - Mt) : 0.0f) + (M2 > -INFINITY ? S2 * hw_exp2(M2 - Mt) : 0.0f));
            const float least = wave_min(i < n ? not_above(c) : INFINITY);
            if (lane == 0) wstat[wv] = make_float2(qnorm, least);
        }
        __syncthreads();
        if (looks) jt_first = ruled_out(jt);
    }
    if (!active) return;
    // the two halves of the wave hold disjoint key subsets of the same query
    float S = Ssum;
    if constexpr (BIAS && !GUMBEL) {
        carry_sum(M, Ssum, all, Mall, lost);
        S = all;
    }
    const float M2 = __shfl_xor(M, 32, kWave), S2 = __shfl_xor(S, 32, kWave);
    const float Mt = fmaxf(M, M2);
    const float St = (M > -INFINITY ? S * hw_exp2(M - Mt) : 0.0f) + (M2 > -INFINITY ? S2 * hw_exp2(M2 - Mt) : 0.0f);
    if (half == 0 && i < n) {
        if (a.parts > 1) {  // the second pass puts the parts together
            a.ws_part[((size_t)u * a.parts + part) * a.n_pad + i] = make_float2(Mt, St);
            if (part == 0) a.ws_r[(size_t)u * a.n_pad + i] = GUMBEL ? rfold : rkey;
            return;
        }
        // log2 of the row's normaliser; the trimmed second pass wants it subtracted from the adjustment's
        // constant part, so that is what is left for it
        const float c = log2_of_sum(Mt, St);
        a.ws_c[(size_t)u * a.n_pad + i] = GUMBEL ? lp.gz - c : c;
        a.ws_r[(size_t)u * a.n_pad + i] = GUMBEL ? rfold : rkey;
    }
    if (skips && a.parts == 1) {  // of the wave's rows: norm, smallest normaliser
        const float cmin = wave_min(i < n ? not_above(log2_of_sum(Mt, St)) : INFINITY);
        if (lane == 0) a.ws_tile[(size_t)u * (a.n_pad / kTile) + i0 / kTile] = make_float4(qnorm, cmin, 0.0f, 0.0f);
    }
}

// ------------------------------------------------------------------ pass 2
// Sum of this lane's 16 terms of a tile, a part of its key's column sum.  cs, rs: the tile's row statistics and row noise
// keys (folded with the Gumbel adjustment); i_first: the lane's first query row.  MASK: the tile crosses the
// diagonal or the end of the prompt.
template <bool GUMBEL, bool BIAS, bool TAU1, bool MASK, bool FIXED = false>
__device__ __forceinline__ float column_sum(const LogitParams& lp, const f32x16& acc, const float* cs, const uint32_t* rs,
                                            int i_first, int half, int j, uint32_t kfold, int n) {
    float sum = 0.0f;  // of the tile: a long prompt's column takes n/2 terms, added one by one they would lose 1e-5
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4) {  // 4 consecutive query rows each
        const float4 c4 = *(const float4*)&cs[q4 * 8 + half * 4];
        const uint4 r4 = *(const uint4*)&rs[q4 * 8 + half * 4];
        const float cv[4] = {c4.x, c4.y, c4.z, c4.w};
        const uint32_t rv[4] = {r4.x, r4.y, r4.z, r4.w};
        const float dist0 = (float)(i_first + q4 * 8 - j);
        float z[4], l2u[4];
        if constexpr (GUMBEL) {
            uint32_t bits[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) bits[e] = mix32_folded(rv[e] ^ kfold);
            wave_priority<1>();
#pragma unroll
            for (int e = 0; e < 4; ++e) l2u[e] = hw_log2(uniform_of(bits[e]));
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float x = acc[q4 * 4 + e];
            if constexpr (GUMBEL) {
                // cv holds (adjustment's constant part - row normaliser): z = 2^(x2 - log2(t)/tau + cv)
                float t = cv[e];
                if (!TAU1) t = fmaf(hw_log2(-l2u[e]), -lp.inv_tau, t);
                if (BIAS) t = fmaf(dist0 + (float)e, -lp.slope1, t);
                z[e] = hw_exp2(fmaf(x, lp.sc1, t));
            } else {
                const float y2 = FIXED ? logit2_fixed(lp, x, dist0 + (float)e) : logit2_other(lp, x, dist0 + (float)e, rv[e], (uint32_t)j);
                z[e] = hw_exp2(y2 - cv[e]);
            }
            const int i = i_first + q4 * 8 + e;
            if (MASK) z[e] = (i >= j && i < n) ? z[e] : 0.0f;
        }
        sum = TAU1 ? add_over_t(z, l2u, sum) : (((sum + z[0]) + z[1]) + z[2]) + z[3];
        if (GUMBEL) wave_priority<0>();
    }
    return sum;
}

// PARTS: the query tiles of a column block are cut into parts, one workgroup each.
template <typename T, int D, bool GUMBEL, bool BIAS, bool TAU1, bool PARTS>
__global__ void __launch_bounds__(kPrefillThreads, (kPrefillMinWaves<T, D>)) prefill_colsum_kernel(const PrefillArgs a, int nblk, int64_t units) {
    constexpr int EPV = ElemTraits<T>::kPerVec;
    constexpr int NG = D / (2 * EPV);
    using Stage = TileStage<T, D>;
    __shared__ __attribute__((aligned(16))) char qbuf[2][Stage::kBufBytes];
    __shared__ __attribute__((aligned(16))) float cbuf[2][kTile];     // the tile's row normalisers ...
    __shared__ __attribute__((aligned(16))) uint32_t rbuf[2][kTile];  // ... and row noise keys
    __shared__ __attribute__((aligned(16))) float call[PARTS ? kPrefillMaxPartTiles * kTile : 4];     // all tiles'
    __shared__ __attribute__((aligned(16))) uint32_t rall[PARTS ? kPrefillMaxPartTiles * kTile : 4];  // (PARTS)
    __shared__ float share_s[2];
    __shared__ int tile_s;
    __shared__ float2 wstat[kPrefillThreads / kWave];  // of a wave's columns: largest norm, smallest sum so far
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n0 = lane & 31, half = lane >> 5;
    int64_t u;
    int cb, part;  // longest columns (lowest keys) first
    unit_and_block<BIAS>(nblk, PARTS ? a.parts : 1, u, cb, part);
    if (u >= units) return;  // workgroup-uniform
    const int h = (int)(u % a.H), b = (int)((u / a.H) % a.B);
    const int n = a.seq_n ? a.seq_n[b] : a.n;  // this sequence's prompt length; rows n..a.n-1 are padding
    const bool first_of_group = (u % a.G) == 0;
    if (n < 1 || n > a.n) {  // workgroup-uniform: the unit is skipped and counted
        if (cb == 0 && part == 0 && threadIdx.x == 0 && first_of_group) atomicAdd(a.ws_err, 1);
        return;
    }
    if (cb == 0 && threadIdx.x == 0 && first_of_group) a.len[u / a.G] = n;
    if (cb * (4 * kTile) >= n) return;  // workgroup-uniform: the block lies in the padding
    // this workgroup's query tiles it_end, it_end-1, .. it_first
    int it_end = (n - 1) / kTile - (PARTS ? part * a.part_tiles : 0);
    const int it_first = PARTS ? max(cb * 4, it_end - a.part_tiles + 1) : cb * 4;
    if (it_end < it_first) return;  // workgroup-uniform: the block has fewer parts
    const int j0 = cb * (4 * kTile) + wv * kTile;
    const bool active = j0 < n;  // wave-uniform; inactive waves still fetch tiles and meet the barriers
    const int j = j0 + n0;
    const T* Qu = (const T*)a.Q + (size_t)u * a.n * D;
    const T* Ku = (const T*)a.K + (size_t)(u / a.G) * a.cap * D;  // G query heads read one cached head

    uint4 bk[NG];
    {
        const T* row = Ku + (size_t)min(j, n - 1) * D + half * EPV;
#pragma unroll
        for (int g = 0; g < NG; ++g) bk[g] = *(const uint4*)(row + g * 2 * EPV);
    }
    LogitParams lp;
    lp.c1 = a.inv_tau * kLog2e;
    lp.sc1 = a.scale * lp.c1;
    lp.slope1 = (BIAS ? a.slopes[h] : 0.0f) * lp.c1;
    lp.inv_tau = a.inv_tau;
    lp.gz = -kLog2Ln2 * a.inv_tau;
    lp.noise = a.noise;
    if constexpr (!GUMBEL) lp.fixed = fixed_adjustment(a.noise) * a.inv_tau;
    const bool fixed = !GUMBEL && (a.noise == kNoiseNone || a.noise == kNoiseConstant);  // the same adjustment for every logit
    const uint32_t kfold = fold16((uint32_t)j * kKposMul);  // this lane's key in every hash (row keys come folded)
    const float* wc = a.ws_c + (size_t)u * a.n_pad;
    const uint32_t* wr = a.ws_r + (size_t)u * a.n_pad;

    float colsum = 0.0f, lost = 0.0f;  // lost: what rounding has added to it (UP, as in pass 1)
    const int it_begin = j0 / kTile;                    // this wave's first query tile (the diagonal one)
    // a tile's 32 row statistics ride with the tile: one wave fetches them (n_pad covers whole tiles)
    struct Staged {
        typename Stage::Regs rows;
        float c;
        uint32_t r;
    };
    if constexpr (PARTS) {
        // row statistics of all this workgroup's tiles, put together from pass 1's parts
        const int row0 = it_first * kTile, rows = (it_end - it_first + 1) * kTile;
        for (int r = threadIdx.x; r < rows; r += kPrefillThreads) {
            const int i = row0 + r;  // rows from n on: left over, masked below
            const float c = merged_normaliser(a.ws_part + (size_t)u * a.parts * a.n_pad + i, a.n_pad,
                                              i < n ? (i / kTile) / a.part_tiles + 1 : 0);
            call[r] = GUMBEL ? lp.gz - c : c;
            rall[r] = i < n ? wr[i] : 0u;
        }
    }
    const float reach = BIAS ? skip_reach(a.noise, a.inv_tau, n) : 0.0f;
    const bool skips = BIAS && a.ws_kn && lp.slope1 * (float)n > reach;  // of the unit: its bounds are there
    const float4* tiles = a.ws_tile + (size_t)u * (a.n_pad / kTile);
    const float* kn = a.ws_kn + (size_t)(u / a.G) * (a.n_pad / kTile);
    if (PARTS && skips && lp.slope1 * (float)((it_end - cb * 4) * kTile) > reach) {
        // workgroup-uniform: the last tile may be ruled out
        const int own_last = min(cb * 4 + 3, (n - 1) / kTile);  // the block's own tiles are walked in any case
        const int limit = max(own_last + 1, it_first);
        // the block's columns: smallest share of a diagonal term in its row, largest key
        const int i = cb * (4 * kTile) + (int)threadIdx.x;
        float share = INFINITY;
        if (threadIdx.x < 4 * kTile && i < n)
            share = not_above(tiles[i / kTile].y - merged_normaliser(a.ws_part + (size_t)u * a.parts * a.n_pad + i, a.n_pad, (i / kTile) / a.part_tiles + 1));
        share = wave_min(share);
        if (lane == 0 && wv < 2) share_s[wv] = share;
        if (threadIdx.x == 0) tile_s = limit - 1;
        __syncthreads();  // (and the normalisers of this workgroup's rows are complete)
        share = fminf(share_s[0], share_s[1]);
        float kmax = 0.0f;
        for (int t = cb * 4; t <= own_last; ++t) kmax = fmaxf(kmax, kn[t]);
        for (int it = it_end - (int)threadIdx.x; it >= limit; it -= kPrefillThreads) {
            float c = INFINITY;  // smallest normaliser of the tile's rows
            for (int r = 0; r < kTile; ++r)
                if (it * kTile + r < n) {
                    const float v = call[(it - it_first) * kTile + r];
                    c = fminf(c, not_above(GUMBEL ? lp.gz - v : v));
                }
            const float bias = lp.slope1 * (float)(it * kTile - (cb * (4 * kTile) + 4 * kTile - 1));
            if (!(tiles[it].x * kmax * fabsf(lp.sc1) + reach - bias - c < share)) {
                atomicMax(&tile_s, it);
                break;
            }
        }
        __syncthreads();
        it_end = min(it_end, __builtin_amdgcn_readfirstlane(tile_s));  // before it_first: nothing is left of the part
    }
    auto fetch = [&](int it) {
        Staged s;
        s.rows = Stage::fetch(Qu, it * kTile, n);
        s.c = 0.0f;
        s.r = 0u;
        if (!PARTS && threadIdx.x < kTile) {
            s.c = wc[it * kTile + threadIdx.x];
            s.r = wr[it * kTile + threadIdx.x];
        }
        return s;
    };
    auto park = [&](int buf, const Staged& s) {
        Stage::park(qbuf[buf], s.rows);
        if (!PARTS && threadIdx.x < kTile) {
            cbuf[buf][threadIdx.x] = s.c;
            rbuf[buf][threadIdx.x] = s.r;
        }
    };
    // The query tiles are walked from the LAST one down: every column block of a unit then starts at the same
    // tile and the blocks, which run at the same time on one XCD, ask its L2 for the same rows at about the
    // same time (walking up, each block starts at its own diagonal and the L2 sees 16 unrelated streams:
    // 2.7 GB instead of 1.0 GB fetched on the GPT-J-shaped workload).  With a position bias the far end may not matter, and
    // the walk goes up from the diagonal.
    constexpr bool UP = BIAS && !PARTS;
    const int looks_at = UP && skips && it_end > it_first + 3 + kSkipAhead ? it_first + 3 + kSkipAhead : -1;
    Staged stage = fetch(UP ? it_first : max(it_end, it_first));
    park(0, stage);
    __syncthreads();
    for (int it = UP ? it_first : it_end, cur = 0; UP ? it <= it_end : it >= it_first; it += UP ? 1 : -1, cur ^= 1) {
        // the next tile (the last one again at the end: rows stay in range), in flight during this tile's work
        const int it_next = UP ? min(it + 1, it_end) : max(it - 1, it_first);
        stage = fetch(it_next);
        if (active && it >= it_begin) {
            const char* qb = qbuf[cur];
            const f32x16 acc = Stage::products(qb, n0, half, bk);
            const int ib = it * kTile;
            const float* cs = PARTS ? call + (it - it_first) * kTile : cbuf[cur];
            const uint32_t* rs = PARTS ? rall + (it - it_first) * kTile : rbuf[cur];
            const bool edge = (ib < j0 + kTile) || (ib + kTile > n);  // crosses the diagonal or the end of the prompt
            float add;
            if (edge) {
                int first = ib + half * 4;  // (the empty asm keeps the masking compares inside this branch, as in pass 1)
                asm volatile("" : "+v"(first));
                if (fixed) add = column_sum<GUMBEL, BIAS, TAU1, true, true>(lp, acc, cs, rs, first, half, j, kfold, n);
                else add = column_sum<GUMBEL, BIAS, TAU1, true>(lp, acc, cs, rs, first, half, j, kfold, n);
            } else if (fixed) {
                add = column_sum<GUMBEL, BIAS, TAU1, false, true>(lp, acc, cs, rs, ib + half * 4, half, j, kfold, n);
            } else {
                add = column_sum<GUMBEL, BIAS, TAU1, false>(lp, acc, cs, rs, ib + half * 4, half, j, kfold, n);
            }
            if (UP) add -= lost;
            const float sum = colsum + add;
            if (UP) lost = fabsf(sum) < INFINITY ? (sum - colsum) - add : 0.0f;
            colsum = sum;
        }
        if (it != it_next) park(cur ^ 1, stage);
        const bool looks = UP && it == looks_at;  // workgroup-uniform
        if (looks) {
            const float sum = colsum + __shfl_xor(colsum, 32, kWave);
            const float least = wave_min(j < n ? not_above(hw_log2(sum)) : INFINITY);
            if (lane == 0) wstat[wv] = make_float2(active ? kn[j0 / kTile] : 0.0f, least);
        }
        __syncthreads();
        if (looks) {
            const float most = largest_adjustment(a.noise) * a.inv_tau + kSkipTileBits;
            it_end -= __builtin_amdgcn_readfirstlane(tiles_ruled_out(it_end - it, [&](int x) {
                const int jt = it_end - x;
                const float4 rows = tiles[jt];
                float e = 0.0f;
                for (int v = 0; v < kPrefillThreads / kWave; ++v) {
                    const int first = cb * (4 * kTile) + v * kTile;  // the wave's first column
                    if (first >= n) break;
                    const float bias = lp.slope1 * (float)(jt * kTile - (first + kTile - 1));
                    e += hw_exp2(rows.x * wstat[v].x * fabsf(lp.sc1) + most - bias - rows.y - wstat[v].y);
                }
                return e;
            }));
        }
    }
    if (!active) return;
    colsum += __shfl_xor(colsum, 32, kWave);
    if (half == 0 && j < n) {
        // one query head per cached head: the column sum is the score; else the heads' sums are
        // added up by the launch that follows
        if (PARTS) a.ws_f[((size_t)u * a.parts + part) * a.n_pad + j] = colsum;
        else if (a.G == 1) a.score[(size_t)u * a.cap + j] = colsum;
        else a.ws_f[(size_t)u * a.n_pad + j] = colsum;
        if (first_of_group && part == 0) a.pos[(size_t)(u / a.G) * a.cap + j] = j;
    }
}

// Grouped-query attention: the score of a cached head is the sum of its query heads' column sums; a column
// block walked in parts: the sum of its parts' (added in head order, then part order, so the result does not
// depend on scheduling).
__global__ void __launch_bounds__(256) prefill_group_sum_kernel(const PrefillArgs a, int64_t kv_units) {
    const int64_t u = blockIdx.x;
    const int j = blockIdx.y * 256 + threadIdx.x;
    if (u >= kv_units) return;
    const int hkv = a.H / a.G, b = (int)((u / hkv) % a.B);
    const int n = a.seq_n ? a.seq_n[b] : a.n;
    if (n > a.n || j >= n) return;
    // parts of this column's block: its query tiles run from the prompt's last one down to the block's first
    const int tiles = (n - 1) / kTile + 1 - j / (4 * kTile) * 4;
    const int parts = a.parts > 1 ? (tiles + a.part_tiles - 1) / a.part_tiles : 1;
    float s = 0.0f;
    for (int g = 0; g < a.G; ++g)
#pragma unroll 4
        for (int p = 0; p < parts; ++p) s += a.ws_f[(((size_t)u * a.G + g) * a.parts + p) * a.n_pad + j];
    a.score[(size_t)u * a.cap + j] = s;
}

// How the tile walks of a launch's 128-row blocks are cut.  A block's walk is serial, up to n/32 tiles, and the
// blocks of a unit are of all lengths: with few units the launch lasts as long as the longest block while most of
// the chip has run out of work (16 heads x 2048 tokens: 136 blocks' worth of work in 256 workgroups, 88 us a pass
// for 10 us of arithmetic).  Below kPrefillPartsRowLimit rows in all, and kPrefillPartsMaxRows of a unit, the walks are
// cut into at most kPrefillMaxParts parts of equal length, one workgroup each, so that about kPrefillPartsWanted
// workgroups have work (wanting 768 to 3072 measured within 20 %, fewer or more slower).  Against uncut walks, both
// passes, d = 128: 16 heads x 2048 rows 1.7 times as fast, x 4224 1.67, 32 x 3524 1.28, 1 x 8192 1.28, 24 x 6340 1.15,
// 1 x 16384 1.01; of 858 launches measured 20 below the second limit lost, 1 to 11 % (192 x 580 rows 0.90, one head of
// d = 256 from 10000 rows on 0.89 to 0.98).  Above the first limit the longest walk is a small share of the launch; above
// the second a walk has so many parts that putting a row's records together costs what the cut gains (1 x 24000 0.94,
// 1 x 32768 0.90).
constexpr int64_t kPrefillPartsWanted = 1536;
constexpr int64_t kPrefillMinPartTiles = 4;
PrefillParts plan_prefill(int64_t U, int32_t n) {
    const int64_t nblk = (n + 4 * kTile - 1) / (4 * kTile);
    if (n > kPrefillPartsMaxRows || U * 4 * kTile * nblk >= kPrefillPartsRowLimit) return kPrefillWhole;
    const int64_t steps = U * nblk * (nblk + 1) / 2 * 4;  // tiles walked by all blocks
    int64_t tiles = (steps + kPrefillPartsWanted - 1) / kPrefillPartsWanted;
    const int64_t least = (nblk * 4 + kPrefillMaxParts - 1) / kPrefillMaxParts;  // of the longest walk
    if (tiles < least) tiles = least;
    if (tiles < kPrefillMinPartTiles) tiles = kPrefillMinPartTiles;
    if (tiles > kPrefillMaxPartTiles) tiles = kPrefillMaxPartTiles;
    const int64_t parts = (nblk * 4 + tiles - 1) / tiles;
    if (parts <= 1) return kPrefillWhole;
    return {(int32_t)parts, (int32_t)tiles};
}

template <typename T, int D, bool GUMBEL, bool BIAS, bool TAU1>
static hipError_t launch_passes(const PrefillArgs& a, int64_t U, hipStream_t st) {
    const int nblk = (a.n + 4 * kTile - 1) / (4 * kTile);
    const int64_t groups = (U + kXcds - 1) / kXcds;  // units are dealt to XCDs in groups of 8
    const dim3 grid((unsigned)(groups * kXcds * nblk * a.parts)), block(kPrefillThreads);
    hipError_t e;
    if (BIAS && a.ws_kn) {
        const dim3 tiles((unsigned)(U / a.G), (unsigned)((a.n + kNormWaves * kTile - 1) / (kNormWaves * kTile)));
        hipLaunchKernelGGL((prefill_key_norms_kernel<T, D>), tiles, dim3(kNormWaves * kWave), 0, st, a, U / a.G);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL((prefill_rowstats_kernel<T, D, GUMBEL, BIAS, TAU1>), grid, block, 0, st, a, nblk, U);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (a.parts > 1) hipLaunchKernelGGL((prefill_colsum_kernel<T, D, GUMBEL, BIAS, TAU1, true>), grid, block, 0, st, a, nblk, U);
    else hipLaunchKernelGGL((prefill_colsum_kernel<T, D, GUMBEL, BIAS, TAU1, false>), grid, block, 0, st, a, nblk, U);
    return hipGetLastError();
}

template <typename T, int D>
static hipError_t launch_prefill_t(const PrefillArgs& a, int64_t U, hipStream_t st) {
    // six builds of each pass: the Gumbel adjustment in the trimmed form, at temperature 1 or any other, or any
    // adjustment in the plain form; with or without the position-bias term
    const bool bias = a.slopes != nullptr;
    hipError_t e;
    if (a.noise != kNoiseGumbel) e = bias ? launch_passes<T, D, false, true, false>(a, U, st) : launch_passes<T, D, false, false, false>(a, U, st);
    else if (a.inv_tau == 1.0f) e = bias ? launch_passes<T, D, true, true, true>(a, U, st) : launch_passes<T, D, true, false, true>(a, U, st);
    else e = bias ? launch_passes<T, D, true, true, false>(a, U, st) : launch_passes<T, D, true, false, false>(a, U, st);
    if (e != hipSuccess || (a.G == 1 && a.parts == 1)) return e;
    hipLaunchKernelGGL(prefill_group_sum_kernel, dim3((unsigned)(U / a.G), (unsigned)((a.n + 255) / 256)), dim3(256), 0,
                       st, a, U / a.G);
    return hipGetLastError();
}

hipError_t launch_prefill(const PrefillArgs& a, int64_t U, int32_t d, int32_t dtype, hipStream_t stream) {
    if (dtype == KF_BF16) {
        if (d == 64) return launch_prefill_t<bf16_t, 64>(a, U, stream);
        if (d == 128) return launch_prefill_t<bf16_t, 128>(a, U, stream);
        if (d == 256) return launch_prefill_t<bf16_t, 256>(a, U, stream);
    } else if (dtype == KF_F16) {
        if (d == 64) return launch_prefill_t<f16_t, 64>(a, U, stream);
        if (d == 128) return launch_prefill_t<f16_t, 128>(a, U, stream);
        if (d == 256) return launch_prefill_t<f16_t, 256>(a, U, stream);
    } else {
        if (d == 64) return launch_prefill_t<float, 64>(a, U, stream);
        if (d == 128) return launch_prefill_t<float, 128>(a, U, stream);
    }
    return hipErrorInvalidValue;
}

}  // namespace kf
