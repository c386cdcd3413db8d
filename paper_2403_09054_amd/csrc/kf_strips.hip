// Prompt scoring of prompts of at most kStripMaxRows rows, Gumbel adjustment: every logit is evaluated ONCE.
//
// The two passes of kf_prefill.hip form each logit, hash and adjustment twice, since a row's normaliser must be known
// before its terms can go into the columns' sums.  Here a workgroup takes a strip of 32 query rows and keeps the terms
// of the whole strip, up to 32 x 2048, in its registers until the rows' sums are known:
//   * wave v of W owns the key tiles v, v+W, ..; a tile's logits come from the matrix cores as in the second pass (a
//     lane owns one key and 16 of the strip's rows) and stay in the lane, 16 registers a tile, at most 8 tiles;
//   * all exponentials, row sums over lanes and waves, one barrier.  The exponentials are taken as they are: a softmax
//     needs a row's maximum only where a term leaves the range of fp32 or all of them vanish, and then the strip is
//     evaluated again and every row taken against its maximum, and so are the next ones, at once, while their maxima ask
//     for it (all logits beyond the range: 256 x 2048 x 128 686 us, 1024 x 512 x 128 269, 300 x 100 x 64 22; two passes 683, 261,
//     16; every strip twice 1183, 392, 29 where two passes took 795, 334, 24);
//   * each term times its row's 1/sum goes into the lane's column sums, which stay in registers over all strips that
//     the workgroup walks, and are written once.
// Two waves per SIMD at 256 registers a lane: 8 waves (2048 keys), or two workgroups of 4 waves (1024 keys) on a CU.
// Keys go through LDS in parts of 128 bytes a row: two workgroups of 4 waves fit also with 512-byte rows (against 8 waves 64
// heads x 1024 x 256 72 -> 53 us, 256 x 1024 x 128 fp32 525 -> 441), and only the form for fp32, d = 128 and 4 waves spills, 4
// registers (against parts of 256 bytes 16 x 2048 x 256 62 -> 57 us, 256 x 2048 x 128 577 -> 569, 512 x 1024 x 128 299 -> 290; all
// on one box).
// With so few waves a wave has to cover its own round trips: while the vector units work on a tile, its next one's
// products are formed in batches of two MFMAs, and the keys of the one after are on their way from memory; the strip's
// query rows lie in LDS, asked for two strips ahead.
//
// A batch asks the LDS for its rows' noise keys before its operands, so that its hashes do not wait for those, and the logarithms
// run at a raised issue priority (wave_priority): with the terms' range told from the sums, 8 x 32 heads x 2048 x 128 567 -> 513 us, 32
// x 2048 x 128 72.4 -> 66.2, with position bias 74.4 -> 66.9, 16 x 2048 x 256 49.5 -> 47.7, 32 x 1024 x 128 24.4 -> 22.7, fp32 64 x
// 2000 x 128 405 -> 398 (one box).  Measured and left: keys by direct loads to LDS (asked for 4 to 8 logits ahead, no key registers):
// 530, 68.4, 48.5 and, 64 x 1024 x 256, 52 -> 56; noise keys asked for a batch ahead: the same, 5 to 13 registers spilled.  With
// 512-byte rows the keys alone, 16 KB a tile, take 33 of 105 thousand cycles of a CU's way from its L2 at 64 bytes each.
//
// (Also left: with 512-byte rows and 4 waves the two settle at a few shapes 2 to 3 % behind the order before, 160 heads x 478 x 256
// 52.0 -> 53.5 us, where most gain as much, 160 x 900 125.2 -> 121.4; without the raised priority the first take 52.2, the second
// 122.1, with the noise keys behind the operands 54.0 and 129.9.)
//
// What bounds it: the vector pipe, 21 instructions a logit in all where the two passes take 32 (8 x 32 heads x 2048 x 128, pipe
// busy 64 % of the time; 16 x 2048 x 256 24 where they take 38, 40 %); the rest is the strips' ends, where a workgroup's waves wait
// for each other, and with 512-byte rows the LDS (a wave waits for it an eighth of its time, with 256-byte rows a sixteenth).  8 x
// 32 heads x 2048 x 128 take 506 us, the two passes 690 on the same box.  On the way, when this took 552: 672 us with the key rows
// read from memory as operands, 664 by way of LDS (512-byte rows 1.3 times as fast), 595 with products ahead, 552 without row
// references formed ahead of a strip and with row sums folded inside the lanes' rows.  Against float64 0.7e-7 to 1.1e-7 relative
// (the passes 1.1e-7 to 2.5e-7): numerator and sum hold the same rounded term.
#include "kf_prefill.h"

namespace kf {

constexpr int kStripTiles = 8;         // key tiles of a wave
constexpr int strip_waves(int n) { return n > kStripSmallRows ? 8 : 4; }
// A row whose sum is larger, or infinite, is taken against its maximum; below, the sum has a reciprocal that is no denormal.  (The
// sums tell of a term too large; a running maximum of the terms would take an instruction a logit for it.)
constexpr float kStripMost = 0x1p118f;
constexpr float kStripTop = 107.0f;    // 2048 terms of this exponent stay below that
// A row whose sum is smaller is taken against its maximum: a term is kept down to 2^-126, the hardware's smallest, so down to
// 2^-86 of its row's sum.  (At 2^-100, a term 2^-26 of its row could vanish, and a column of such terms with it.)
constexpr float kStripLeast = 0x1p-40f;
constexpr float kStripBottom = -40.0f; // rows whose largest exponent lies from here to the top are taken as they are for certain

// Folds 16 values per lane over the 32 lanes of each half: lanes 0-15 of a half get the results of values 0-7, lanes 16-31
// those of values 8-15.  One exchange of rows of 16 lanes folds two values at a time, rotations inside the rows do the rest
// (through the LDS crossbar it was five trips in series).
template <int CTRL>
__device__ __forceinline__ float rotated(float v) {
    return __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(v), CTRL, 0xF, 0xF, false));
}
template <typename OP>
__device__ __forceinline__ void fold_rows(const float (&v)[16], float (&a)[8], OP op) {
#pragma unroll
    for (int r = 0; r < 8; ++r) {
        const auto x = __builtin_amdgcn_permlane16_swap(__float_as_uint(v[r]), __float_as_uint(v[r + 8]), false, false);
        a[r] = op(__uint_as_float(x[0]), __uint_as_float(x[1]));
    }
#pragma unroll
    for (int r = 0; r < 8; ++r) a[r] = op(a[r], rotated<0x128>(a[r]));  // row_ror:8
#pragma unroll
    for (int r = 0; r < 8; ++r) a[r] = op(a[r], rotated<0x124>(a[r]));
#pragma unroll
    for (int r = 0; r < 8; ++r) a[r] = op(a[r], rotated<0x122>(a[r]));
#pragma unroll
    for (int r = 0; r < 8; ++r) a[r] = op(a[r], rotated<0x121>(a[r]));
}

// Orders a wave's accesses to LDS that its own lanes exchange values through (the LDS serves a wave's accesses in order).
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <typename T, int D, bool BIAS, int W>
__global__ void __launch_bounds__(W * kWave, 2) prefill_strips_kernel(const PrefillArgs a, int64_t units, int grouped) {
    constexpr int NT = W * kWave, RB = D * (int)sizeof(T), NG = RB / 32, PITCH = RB + 16;
    constexpr int PPR = RB / 16, TPR = NT / kTile, PT = (PPR + TPR - 1) / TPR;  // 16-byte pieces a row, threads a row, pieces a thread
    constexpr int HB = 128, NGA = HB / 32, HPR = HB / 16, KPITCH = HB + 16;  // key rows, part by part
    constexpr int QB = 2, NB = NG / QB, NS = 8 / NB;  // products a batch, batches a tile, pairs of logits a batch
    __shared__ __attribute__((aligned(16))) char qbuf[3][kTile * PITCH];
    __shared__ __attribute__((aligned(16))) char kbuf[W][kTile * KPITCH];
    __shared__ __attribute__((aligned(16))) uint32_t fold_s[3][kTile];  // folded noise keys of the rows
    __shared__ __attribute__((aligned(16))) float part_s[2][W][kTile];  // what each wave has of the rows' sums
    __shared__ __attribute__((aligned(16))) float own_s[W][kTile];      // a wave's own copy of the rows' factors
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n0 = lane & 31, half = lane >> 5;
    const int walkers = a.parts;
    int64_t u;
    int p;
    if (grouped) {  // a unit's workgroups share an XCD and its L2
        const unsigned xcd = blockIdx.x % kXcds, local = blockIdx.x / kXcds, group = local / walkers;
        u = (int64_t)group * kXcds + (xcd + group) % kXcds;
        p = (int)(local % walkers);
    } else {        // few units: over all XCDs
        u = blockIdx.x % (unsigned)units;
        p = (int)(blockIdx.x / (unsigned)units);
    }
    if (u >= units) return;  // workgroup-uniform, as all exits
    const unsigned lb = (unsigned)u / (unsigned)a.H;  // (a launch has fewer than 2^31 units)
    const int h = (int)((unsigned)u - lb * (unsigned)a.H), b = (int)(lb % (unsigned)a.B), l = a.layer0 + (int)(lb / (unsigned)a.B);
    const int n = a.seq_n ? a.seq_n[b] : a.n;
    const bool first_of_group = (unsigned)u % (unsigned)a.G == 0;
    if (n < 1 || n > a.n) {  // the unit is skipped and counted
        if (p == 0 && threadIdx.x == 0 && first_of_group) atomicAdd(a.ws_err, 1);
        return;
    }
    if (p == 0 && threadIdx.x == 0 && first_of_group) a.len[u / a.G] = n;
    const int strips = (n + kTile - 1) / kTile;
    if (p >= strips) return;
    const char* Qu = (const char*)a.Q + (size_t)u * a.n * RB;
    const char* Ku = (const char*)a.K + (size_t)((unsigned)u / (unsigned)a.G) * a.cap * RB;  // G query heads read one cached head

    LogitParams lp;
    lp.c1 = a.inv_tau * kLog2e;
    lp.sc1 = a.scale * lp.c1;
    lp.slope1 = (BIAS ? a.slopes[h] : 0.0f) * lp.c1;
    lp.inv_tau = a.inv_tau;
    lp.gz = -kLog2Ln2 * a.inv_tau;
    lp.noise = a.noise;
    const uint64_t ukey = unit_key(a.seeds[b], (uint32_t)l, (uint32_t)h);

    // number of a wave's tiles in a strip (formed where it is used: eight comparisons held over a strip take registers)
    auto tiles_of = [&](int s) {
        int e = s;
        asm volatile("" : "+s"(e));
        return wv <= e ? (e - wv) / W + 1 : 0;
    };
    // the k-th strip of this workgroup: there and back over the walkers, so that all have about the same work
    auto strip_of = [&](int k) { return k & 1 ? (k + 1) * walkers - 1 - p : k * walkers + p; };

    // A strip's query rows into LDS, with the rows' noise keys: TPR threads a row.  (What follows from the thread's number is
    // formed where it is used: held over the strips it would be spilled.)
    auto thread_here = [] {
        unsigned t = threadIdx.x;
        asm volatile("" : "+v"(t));
        return t;
    };
    struct Rows {
        u32x4_t q[PT];
    };
    auto fetch_strip = [&](int s) {
        Rows r;
        const unsigned t = thread_here();
        const uint32_t at = (uint32_t)min(s * kTile + (int)(t / TPR), n - 1) * RB;
#pragma unroll
        for (int x = 0; x < PT; ++x) r.q[x] = *(const u32x4_t*)(Qu + (at + min(t % TPR + x * TPR, (unsigned)PPR - 1u) * 16u));
        return r;
    };
    auto park_strip = [&](int s, int buf, const Rows r) {
        const unsigned t = thread_here(), row = t / TPR, col = t % TPR;
#pragma unroll
        for (int x = 0; x < PT; ++x)
            if (col + x * TPR < PPR) *(u32x4_t*)(qbuf[buf] + row * PITCH + (col + x * TPR) * 16) = r.q[x];
        if (t < kTile) fold_s[buf][t] = fold16(row_key(ukey, (uint32_t)(s * kTile) + t));
    };
    // The wave's next key tile, in whole lines, 16-byte pieces of 128-byte parts of its rows: asked
    // for while the piece of work before is under way, then by way of the wave's own LDS into the operand's layout.  (Asked
    // for in that layout, 32 rows an instruction, a tile of 256-byte rows kept the CU's address unit busy for 500 cycles.
    // The empty asm keeps addresses of all tiles from being formed ahead and held in registers.)
    u32x4_t key[NGA];
    const uint32_t klane = (uint32_t)lane / HPR, kcol = (uint32_t)lane % HPR * 16u;  // of a lane's pieces: row, byte
    auto load_keys = [&](int tile, int h) {
        const int jt = min(tile, strips - 1);
        const char* base = Ku + (size_t)jt * kTile * RB + h * HB;
        uint32_t over = (uint32_t)(n - 1 - jt * kTile), row = klane;  // rows from n on repeat row n-1
        asm volatile("" : "+s"(over), "+v"(row));
#pragma unroll
        for (int g = 0; g < NGA; ++g) key[g] = *(const u32x4_t*)(base + (min(row + g * (kWave / HPR), over) * RB + kcol));
    };
    char* const kb = kbuf[wv];
    const char* const kp = kb + n0 * KPITCH + half * 16;
    // operands of QB products, batch x of a tile: key tile jt (at the head of a part: parked here, and the next one, of tile
    // `after` behind the last part, asked for), query rows at q
    struct Batch {
        uint4 q[QB], k[QB];
    };
    auto operands = [&](int x, int jt, int after, const char* q) {
        if (x * QB % NGA == 0) {
            wave_sync();
#pragma unroll
            for (int g = 0; g < NGA; ++g) {
                *(u32x4_t*)(kb + (klane + g * (kWave / HPR)) * KPITCH + kcol) = key[g];
            }
            wave_sync();
            constexpr int chunks = NG / NGA;
            const int c = x * QB / NGA + 1;
            if (c < chunks) load_keys(jt, c);
            else load_keys(after, 0);
        }
        Batch o;
#pragma unroll
        for (int g = 0; g < QB; ++g) {
            o.q[g] = *(const uint4*)(q + (x * QB + g) * 32);
            o.k[g] = *(const uint4*)(kp + (x * QB % NGA + g) * 32);
        }
        return o;
    };
    auto multiply = [&](const Batch o, f32x16 acc) {
#pragma unroll
        for (int g = 0; g < QB; ++g) acc = Mma<T>::group(o.q[g], o.k[g], acc);
        return acc;
    };
    // 16 values of a lane's rows from an array of 32
    auto rows_of = [&](const float* src, float (&v)[16]) {
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
            const float4 f = *(const float4*)&src[q4 * 8 + half * 4];
            v[q4 * 4] = f.x;
            v[q4 * 4 + 1] = f.y;
            v[q4 * 4 + 2] = f.z;
            v[q4 * 4 + 3] = f.w;
        }
    };
    // a value per row (lane n0 holds row n0's) to every lane's 16 rows, by way of the wave's own LDS
    auto spread = [&](float x, float (&v)[16]) {
        if (half == 0) own_s[wv][n0] = x;
        wave_sync();
        rows_of(own_s[wv], v);
        wave_sync();
    };

    int par = 0;  // of part_s: a value written before a barrier is read before the next one
    // what the wave has of the rows' sums (or maxima) to the other waves
    auto leave_rows = [&](const float (&v)[16], auto op) {
        float f[8];
        fold_rows(v, f, op);
        if ((lane & 15) == 0) {
            float* at = &part_s[par][wv][(lane & 16) + half * 4];
            *(float4*)at = make_float4(f[0], f[1], f[2], f[3]);
            *(float4*)(at + 8) = make_float4(f[4], f[5], f[6], f[7]);
        }
    };

    float col[kStripTiles];
#pragma unroll
    for (int t = 0; t < kStripTiles; ++t) col[t] = 0.0f;
    float y[kStripTiles][16];

    f32x16 acc;          // products of the wave's first tile of the strip, if ready
    bool ready = false;
    int start = 0;       // how the next strip is begun: 0 plainly, 2 against its rows' maxima, as the strip before had to be
    park_strip(p, 0, fetch_strip(p));
    park_strip(strip_of(1), 1, fetch_strip(strip_of(1)));
    __syncthreads();
    for (int k = 0;; ++k) {
        const int s = strip_of(k), next = strip_of(k + 1), cur = k % 3, nxt = (k + 1) % 3;
        if (s >= strips) break;
        const int coming = strip_of(k + 2);  // (behind the last strip: the last row again)
        const Rows rows = fetch_strip(coming);
#pragma clang loop unroll(disable)
        for (int mode = start;; mode = 1) {  // 1: again, against the rows' maxima
            // ---- logits (log2).  While the vector units work on a tile, the matrix cores form the next one's products (behind
            // the last tile: of the next strip's first).
            if (!ready && wv <= s) {
                load_keys(wv, 0);
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
#pragma unroll
                for (int x = 0; x < NB; ++x)
                    acc = multiply(operands(x, wv, wv + W <= s ? wv + W : wv, qbuf[cur] + n0 * PITCH + half * 16), acc);
            }
#pragma unroll
            for (int t = 0; t < kStripTiles; ++t) {
                int jt = wv + W * t, end = s;
                asm volatile("" : "+s"(jt), "+s"(end));  // (keeps the eight tiles' limits from being formed ahead and held)
                if (jt <= end) {
                    const bool more = jt + W <= end;
                    const int coming = more ? jt + W : wv, last = more ? end : next;
                    const int after = coming + W <= last ? coming + W : wv;
                    int qrow = n0 * PITCH + half * 16;
                    asm volatile("" : "+v"(qrow));
                    const char* qp = qbuf[more ? cur : nxt] + qrow;
                    f32x16 ahead;
#pragma unroll
                    for (int r = 0; r < 16; ++r) ahead[r] = 0.0f;
                    int j = jt * kTile + n0;
                    asm volatile("" : "+v"(j));  // (keeps the eight tiles' positions from being formed ahead and held)
                    uint32_t kfold = fold16((uint32_t)j * kKposMul);
                    asm volatile("" : "+v"(kfold));  // (else its two halves go into every logit apart)
                    auto folds = [&](int r) { return *(const uint2*)&fold_s[cur][(r >> 2) * 8 + half * 4 + (r & 3)]; };
                    // position bias -slope*(i - j): the lane's part here, that of its 16 rows as literal multiples
                    const float back = BIAS ? fmaf(lp.slope1, (float)(j - end * kTile - half * 4), lp.gz) : lp.gz;
#pragma unroll
                    for (int x = 0; x < NB; ++x) {
                        uint2 fold[NS];  // (ahead of the operands: the LDS answers in order)
#pragma unroll
                        for (int i = 0; i < NS; ++i) fold[i] = folds(x * NS * 2 + 2 * i);
                        __builtin_amdgcn_sched_barrier(0);
                        const Batch o = operands(x, coming, after, qp);
                        __builtin_amdgcn_sched_barrier(0);
                        uint32_t bits[2 * NS];
#pragma unroll
                        for (int i = 0; i < NS; ++i) {  // two rows
                            bits[2 * i] = mix32_folded(fold[i].x ^ kfold);
                            bits[2 * i + 1] = mix32_folded(fold[i].y ^ kfold);
                        }
                        wave_priority<1>();
#pragma unroll
                        for (int i = 0; i < 2 * NS; ++i) {
                            const int r = x * NS * 2 + i;
                            const float l2u = hw_log2(uniform_of(bits[i]));
                            const float c = BIAS ? fmaf(lp.slope1, -(float)((r >> 2) * 8 + (r & 3)), back) : back;
                            y[t][r] = fmaf(acc[r], lp.sc1, fmaf(hw_log2(-l2u), -lp.inv_tau, c));
                        }
                        wave_priority<0>();
                        ahead = multiply(o, ahead);
                    }
                    if (jt == end) {  // crosses the diagonal (the empty asm keeps the compares inside this branch)
                        int first = half * 4 - n0;
                        asm volatile("" : "+v"(first));
#pragma unroll
                        for (int r = 0; r < 16; ++r) {
                            const int past = first + (r >> 2) * 8 + (r & 3);  // rows behind the diagonal
                            // (an infinite logit on the diagonal makes its row NaN, as where that logit is the row's reference)
                            const float x = past == 0 && y[t][r] == INFINITY ? NAN : y[t][r];
                            y[t][r] = past >= 0 ? x : -INFINITY;
                        }
                    }
                    acc = ahead;
                }
            }
            ready = wv <= s;
            if (mode > 0) {
                // the rare way: a term too large, or a row without a term that counts: every row against its maximum (which
                // tells whether the next strip is likely to need it too; the same in every wave)
                float v[16];
                const int tiles = tiles_of(s);
#pragma unroll
                for (int r = 0; r < 16; ++r) v[r] = -INFINITY;
#pragma unroll
                for (int t = 0; t < kStripTiles; ++t)
                    if (t < tiles)
#pragma unroll
                        for (int r = 0; r < 16; ++r) v[r] = fmaxf(v[r], y[t][r]);
                leave_rows(v, [](float x, float z) { return fmaxf(x, z); });
                __syncthreads();
                float most = -INFINITY;
#pragma unroll
                for (int w = 0; w < W; ++w) most = fmaxf(most, part_s[par][w][n0]);
                par ^= 1;
                // Against an infinite logit all others vanish, and it stays infinite.  The last strip's rows behind the prompt's end
                // repeat its last row: only here can a term of theirs be infinite (which times their factor of 0 would be no
                // number in the column), so here their logits become 0.  (By masks of bits: compares held over the tiles made the
                // compiler spill scalar registers, which cost the whole kernel 1 to 4 %.)
                const int left = n - s * kTile;
                const bool row = (int)(thread_here() & 31) < left;
                start = __any(row && !(most >= kStripBottom && most < kStripTop)) ? 2 : 0;
                spread(row ? fminf(most, 0x1.fffffep127f) : 0.0f, v);
                const uint32_t inside = left < kTile ? (1u << left) - 1u : ~0u;  // by rows of the strip
#pragma unroll
                for (int t = 0; t < kStripTiles; ++t)
                    if (t < tiles) {
                        const uint32_t mine = inside >> (thread_here() >> 5 & 1) * 4;
#pragma unroll
                        for (int r = 0; r < 16; ++r) {
                            const int keep = __builtin_amdgcn_sbfe((int)mine, (r >> 2) * 8 + (r & 3), 1);  // all bits or none
                            y[t][r] = __uint_as_float(__float_as_uint(y[t][r]) & (uint32_t)keep) - v[r];
                        }
                    }
            }
            // ---- terms and row sums; the rows of the strip after the next
            {
                float v[16];
                const int tiles = tiles_of(s);
#pragma unroll
                for (int r = 0; r < 16; ++r) v[r] = 0.0f;
#pragma unroll
                for (int t = 0; t < kStripTiles; ++t)
                    if (t < tiles)
#pragma unroll
                        for (int r = 0; r < 16; ++r) {
                            y[t][r] = hw_exp2(y[t][r]);
                            v[r] += y[t][r];
                        }
                leave_rows(v, [](float x, float z) { return x + z; });
                if (mode != 1) park_strip(coming, (k + 2) % 3, rows);
            }
            __syncthreads();
            float sum = 0.0f;
#pragma unroll
            for (int w = 0; w < W; ++w) sum += part_s[par][w][n0];
            par ^= 1;
            const bool row = s * kTile + (int)(thread_here() & 31) < n;
            // (the same in every wave: all read the same sums.  Also a sum of a row behind the prompt's end: an infinite term of its
            // times the row's factor of 0 would be no number.)
            if (mode == 0 && __any(sum >= kStripMost || (row && sum < kStripLeast))) {
                ready = false;
                continue;
            }
            // ---- column sums
            float f[16];
            const int tiles = tiles_of(s);
            const bool edge = wv + W * (tiles - 1) == s;  // the wave's last tile crosses the diagonal
            spread(row ? (sum < INFINITY || sum != sum ? 1.0f / sum : 1.0f) : 0.0f, f);
#pragma unroll
            for (int t = 0; t < kStripTiles; ++t)
                if (t < tiles) {
                    if (edge && t == tiles - 1) {  // masked terms are no part of a column, also where the row's sum is no number
                        int first = half * 4 - n0;
                        asm volatile("" : "+v"(first));
#pragma unroll
                        for (int r = 0; r < 16; ++r) y[t][r] = first + (r >> 2) * 8 + (r & 3) >= 0 ? y[t][r] * f[r] : 0.0f;
#pragma unroll
                        for (int r = 0; r < 16; ++r) f[r] = 1.0f;  // (the strip's last tile)
                    }
                    float c = 0.0f;
#pragma unroll
                    for (int r = 0; r < 16; ++r) c = fmaf(y[t][r], f[r], c);
                    col[t] += c;
                }
            break;
        }
    }
#pragma unroll
    for (int t = 0; t < kStripTiles; ++t) {
        const int j = (wv + W * t) * kTile + n0;
        const float c = col[t] + __shfl_xor(col[t], 32, kWave);
        if (half == 0 && j < n) {
            if (a.ws_f) a.ws_f[((size_t)u * walkers + p) * a.n_pad + j] = c;
            else a.score[(size_t)u * a.cap + j] = c;
            if (first_of_group && p == 0) a.pos[(size_t)((unsigned)u / (unsigned)a.G) * a.cap + j] = j;
        }
    }
}

// The score of a cached head: the sum over its query heads and their walkers, in that order.
__global__ void __launch_bounds__(256) strips_sum_kernel(const PrefillArgs a, int64_t kv_units) {
    const int64_t u = blockIdx.x;
    const int j = blockIdx.y * 256 + threadIdx.x;
    if (u >= kv_units) return;
    const int hkv = a.H / a.G, b = (int)((u / hkv) % a.B);
    const int n = a.seq_n ? a.seq_n[b] : a.n;
    if (n < 1 || n > a.n || j >= n) return;
    const int walkers = min(a.parts, (n + kTile - 1) / kTile);  // the others had no strip
    float s = 0.0f;
    for (int g = 0; g < a.G; ++g)
#pragma unroll 8
        for (int p = 0; p < walkers; ++p) s += a.ws_f[(((size_t)u * a.G + g) * a.parts + p) * a.n_pad + j];
    a.score[(size_t)u * a.cap + j] = s;
}

// Which prompts are scored this way.  Against the two passes (whole calls, 1.0 = the same time; d = 64 to 256; "units" are heads
// times sequences times layers).  Up to 256 units 1.03 to 2.2 everywhere (16 heads x 2048 x 256 96 -> 49 us, 32 x 2048 x 128
// 115 -> 66, 32 x 1024 52 -> 24, 256 x 2048 x 128 690 -> 506; fp32, whose products take the time, 256 x 1024 x 128 1016 -> 453).
// With more units the passes fill the chip by themselves, and a short strip's sums and barrier weigh more than its logits.  Below
// 256 rows 320 units 0.95 to 1.8, 512 0.9 to 2.3, 1024 0.8 to 1.2; 256 to 399 rows 512 units 1.27 to 1.6, 1024 0.9 to 1.2;
// from 400 rows on (512-byte rows: 512) 1.02 to 1.8 up to 2048 units.  From 1025 rows on, where every strip goes to 8 waves, 160
// units 1.13 to 1.35, 256 1.07 to 1.28, 512 0.94 to 1.12, and from 1280 rows on 1.03 to 1.34 up to 1024 units.  With a position
// bias the passes leave out tiles from 1025 rows on: up to 256 units 1.03 to 2.1, 384 0.98 to 1.12, 512 0.93 to 1.05, 1024 0.86 to
// 1.03 with slopes 2^(-8h/H); with slopes that rule nothing out 1.16 to 1.5, fp32 1.3 to 1.6.  (The limits were drawn when strips
// cost an eighth more: those at 256 and 1280 rows, and that of fp32 with a bias, now leave out shapes that would gain.)
static int64_t most_strip_units(int32_t n, int32_t dtype, int32_t row_bytes, bool bias) {
    const bool narrow = dtype != KF_F32;
    int64_t most = n < 256 ? 320 : n < (narrow && row_bytes > 256 ? 512 : 400) ? 512 : INT64_MAX;
    if (bias && n >= kPrefillSkipMinRows && most > 256) most = 256;
    if (narrow && n > kStripSmallRows && n < 1280) most = 160;
    return most;
}

// Workgroups that share a unit's strips.  A round of workgroups fills the chip (one of 8 waves on a CU, or two of 4); the
// cost of a choice is its rounds times the longest workgroup's walk, in tiles of a wave: half the longest strip's for each
// of its strips, about one for a strip's sums and barrier, three to begin and end.  Where units have to queue, those
// that are worked on at the same time should fit the L2 of their XCD with their keys.
constexpr int kStripMaxWalkers = 64;
constexpr int64_t kStripL2Bytes = 2500000;
int32_t plan_strips(int64_t U, int32_t n, int32_t d, int32_t dtype, bool bias) {
    if (n > kStripMaxRows) return 0;
    const int32_t row_bytes = d * (dtype == KF_F32 ? 4 : 2);
    if (U > most_strip_units(n, dtype, row_bytes, bias)) return 0;
    const int64_t padded = (n + kPrefillRowPad - 1) / kPrefillRowPad * kPrefillRowPad, strips = padded / kTile;
    const int waves = strip_waves(n);
    const int64_t slots = waves == 8 ? 256 : 512;
    const int64_t most = strips < kStripMaxWalkers ? strips : kStripMaxWalkers;
    int64_t least = 1;
    if (U > slots / 8) {
        least = (slots / kXcds * padded * row_bytes + kStripL2Bytes - 1) / kStripL2Bytes;
        if (least > most) least = most;
    }
    int64_t best = 0, best_cost = 0;
    for (int64_t P = least; P <= most; ++P) {
        const int64_t rounds = (U * P + slots - 1) / slots, walk = (strips + P - 1) / P;
        const int64_t cost = rounds * (walk * (strips + 4 * waves) + 8 * waves);
        if (!best || cost < best_cost) best = P, best_cost = cost;
    }
    return (int32_t)best;
}

template <typename T, int D>
static hipError_t launch_strips_t(const PrefillArgs& a, int64_t U, hipStream_t st) {
    const int grouped = U % kXcds == 0 || U >= 8 * kXcds;
    const int64_t all = (grouped ? (U + kXcds - 1) / kXcds * kXcds : U) * a.parts;
    const dim3 grid((unsigned)all);
    const bool bias = a.slopes != nullptr;
    if (strip_waves(a.n) == 8) {
        if (bias) hipLaunchKernelGGL((prefill_strips_kernel<T, D, true, 8>), grid, dim3(8 * kWave), 0, st, a, U, grouped);
        else hipLaunchKernelGGL((prefill_strips_kernel<T, D, false, 8>), grid, dim3(8 * kWave), 0, st, a, U, grouped);
    } else {
        if (bias) hipLaunchKernelGGL((prefill_strips_kernel<T, D, true, 4>), grid, dim3(4 * kWave), 0, st, a, U, grouped);
        else hipLaunchKernelGGL((prefill_strips_kernel<T, D, false, 4>), grid, dim3(4 * kWave), 0, st, a, U, grouped);
    }
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess || !a.ws_f) return e;
    hipLaunchKernelGGL(strips_sum_kernel, dim3((unsigned)(U / a.G), (unsigned)((a.n + 255) / 256)), dim3(256), 0, st, a, U / a.G);
    return hipGetLastError();
}

hipError_t launch_strips(const PrefillArgs& a, int64_t U, int32_t d, int32_t dtype, hipStream_t stream) {
    if (dtype == KF_BF16) {
        if (d == 64) return launch_strips_t<bf16_t, 64>(a, U, stream);
        if (d == 128) return launch_strips_t<bf16_t, 128>(a, U, stream);
        if (d == 256) return launch_strips_t<bf16_t, 256>(a, U, stream);
    } else if (dtype == KF_F16) {
        if (d == 64) return launch_strips_t<f16_t, 64>(a, U, stream);
        if (d == 128) return launch_strips_t<f16_t, 128>(a, U, stream);
        if (d == 256) return launch_strips_t<f16_t, 256>(a, U, stream);
    } else {
        if (d == 64) return launch_strips_t<float, 64>(a, U, stream);
        if (d == 128) return launch_strips_t<float, 128>(a, U, stream);
    }
    return hipErrorInvalidValue;
}

}  // namespace kf
