// Key-token selection and in-place, order-preserving KV compaction for gfx950.
//
// Per unit (Algorithm 1: S_w, S_key, S_k):  keep the last w slots and the k-w
// slots of [0, len-w) with the largest accumulated score, equal scores resolved
// toward the lower slot; move the survivors' K, V, score and pos rows to slots
// [0,k) in their original order; len = k.
//
// One workgroup per unit.
//   select   radix select on order-preserving uint32 keys of the scores: four
//            8-bit passes with an LDS histogram find the (k-w)-th largest key T
//            and how many candidates equal to T still fit.
//   rank     one ordered sweep over the candidates: a candidate survives if its
//            key is above T, or equals T and fewer than `need` equal keys
//            precede it (lower slot wins).  Ballot/popcount prefix counts give
//            each survivor its destination; the source slots are written to a
//            dense index list.
//            (A unit that is exactly one token over budget -- every decode
//            step -- skips both: the token to evict is the candidate with the
//            smallest score, the highest slot among equals, found by one
//            min-reduction; see evict_one.)
//   compact  rows are gathered front to back in tiles: a tile's sources are
//            read into registers, the workgroup synchronises, then the tile's
//            destinations are written.  Every source lies at or after its
//            destination, so a tile never overwrites a row a later tile still
//            has to read.  Rows that stay where they are are not touched.
#include <type_traits>

#include "kf_device.h"
#include "kf_internal.h"
#include "kf_merge.h"

namespace kf {

constexpr int kSelectThreads = 1024;     // ordered layout: many rows move, many waves stream them
constexpr int kSelectThreadsSlot = 512;  // slot layout: one row moves, smaller workgroups finish sooner
constexpr int kSelectGroups = 4;  // row groups a thread holds in registers per tile
constexpr int kShiftDepth = 8;    // independent 16-byte loads a lane keeps in flight while shifting

// One token over budget (len = k+1, the shape of every decode step): evict the
// candidate with the smallest score, the highest slot among equal minima (so
// that lower slots are kept), then close the gap: rows e+1..k move down by one.
//
// The rows that move are the candidates behind the evicted slot (usually a
// handful) and the whole recent window (always, whatever slot is evicted).  The
// window part therefore starts before the evicted slot is known: waves 2.. own
// fixed contiguous ranges of it and have their first rows in flight while the
// min-reduction runs.  A lane owns one 16-byte piece of a row, the two halves of
// a wave take K and V.  A wave walks its range upwards, several rows in flight:
// row i+1 is loaded before row i is stored, loads return in order, and the wave
// is the only writer of its range, so it never overwrites a row it still has to
// read.  The one row it reads from its neighbour's range (the first row above
// its own) is loaded before the barrier; the neighbour stores only after it.
// The candidate part is read completely before that same barrier -- into
// registers when it is short, by a streaming pass of its own when it is long --
// because its last source row is the window part's first destination.
// Waves 0 and 1 shift score and pos the same way, 64 elements per instruction.
// Row loads and stores are non-temporal: the shifted rows are not needed again
// before the next step's full sweep, and leaving them out of the caches shortens
// that sweep (the following decode launch ran 93 -> 83 us on the GPT-J-shaped
// workload, this kernel 47 -> 51 us).
struct RowLane {  // what a lane needs to address its piece of a row
    uint4* base;
    int PPR, RPI, rsub, piece;
    __device__ __forceinline__ uint4* at(int row) const { return base + (size_t)row * PPR + piece; }
};

// Streams dst rows [r0, r1) <- src rows [r0+1, r1+1) of one wave's range.  `first`
// holds the already loaded sources of the range's first G instructions, `last`
// those of its last instruction (the only rows read from beyond the range).
template <int G>
__device__ __forceinline__ void shift_range(const RowLane& L, int r0, int NI, const uint4 (&first)[G], bool has_last,
                                            int last_i, const uint4& last) {
#pragma unroll
    for (int g = 0; g < G; ++g)
        if (g < NI - 1) stream_store(L.at(r0 + g * L.RPI + L.rsub), first[g]);
    for (int ii = G; ii < NI - 1; ii += G) {
        uint4 regs[G];
#pragma unroll
        for (int g = 0; g < G; ++g) {
            regs[g] = make_uint4(0u, 0u, 0u, 0u);
            if (ii + g < NI - 1) regs[g] = stream_load(L.at(r0 + (ii + g) * L.RPI + L.rsub + 1));
        }
#pragma unroll
        for (int g = 0; g < G; ++g)
            if (ii + g < NI - 1) stream_store(L.at(r0 + (ii + g) * L.RPI + L.rsub), regs[g]);
    }
    if (has_last) stream_store(L.at(last_i), last);
}

// Loads what shift_range needs up front: the first G instructions' sources and the last one's.
template <int G>
__device__ __forceinline__ void preload_range(const RowLane& L, int r0, int r1, int& NI, uint4 (&first)[G],
                                              bool& has_last, int& last_i, uint4& last) {
    NI = r0 < r1 ? (r1 - r0 + L.RPI - 1) / L.RPI : 0;  // wave instructions of this range
    last_i = r0 + (NI - 1) * L.RPI + L.rsub;
    has_last = NI > 0 && last_i < r1;
    last = make_uint4(0u, 0u, 0u, 0u);
    if (has_last) last = stream_load(L.at(last_i + 1));
#pragma unroll
    for (int g = 0; g < G; ++g) {
        first[g] = make_uint4(0u, 0u, 0u, 0u);
        if (g < NI - 1) first[g] = stream_load(L.at(r0 + g * L.RPI + L.rsub + 1));
    }
}

template <int NT>
__device__ __forceinline__ void evict_one(const SelectArgs& a, int64_t u, int n, bool write_idx) {
    constexpr int NW = NT / kWave;
    constexpr int NRW = NW - 2;  // waves that move rows
    constexpr int G = kShiftDepth;
    __shared__ unsigned long long wmin[NW];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int k = a.k, w = a.w;
    const int ncand = n - w;
    float* fu = a.score + (size_t)u * a.cap;
    int32_t* pu = a.pos + (size_t)u * a.cap;

    RowLane L;
    L.PPR = a.row_bytes >> 4;  // 16-byte pieces per row: 8, 16 or 32
    L.RPI = 32 / L.PPR;        // rows per wave instruction (each half of the wave one tensor)
    L.rsub = (lane & 31) / L.PPR;
    L.piece = lane % L.PPR;
    L.base = (uint4*)((char*)((lane >> 5) ? a.V : a.K) + (size_t)u * a.cap * a.row_bytes);
    auto range_of = [&](int lo, int hi, int& r0, int& r1) {  // this wave's share of dst rows [lo, hi)
        int per = (hi - lo + NRW - 1) / NRW;
        per = (per + L.RPI - 1) / L.RPI * L.RPI;
        r0 = min(hi, lo + (wv - 2) * per);
        r1 = min(hi, r0 + per);
    };

    // candidate scores first, so that they return ahead of the row loads issued next
    // smallest (key, -slot): the low word holds ~slot so that the highest slot wins a tie
    unsigned long long best = ~0ull;
    for (int j = tid; j < ncand; j += NT) {
        const unsigned long long pack = ((unsigned long long)float_key(fu[j]) << 32) | (uint32_t)(~(uint32_t)j);
        best = pack < best ? pack : best;
    }

    // ---- window part, dst rows [ncand-1, k): in flight before the evicted slot is known
    const int w_lo = max(ncand - 1, 0);
    int wr0 = 0, wr1 = 0, wNI = 0, wlast_i = 0;
    bool whas_last = false;
    uint4 wfirst[G], wlast = make_uint4(0u, 0u, 0u, 0u);
    if (wv >= 2) {
        range_of(w_lo, k, wr0, wr1);
        preload_range<G>(L, wr0, wr1, wNI, wfirst, whas_last, wlast_i, wlast);
    }

    best = wave_min(best);
    if (lane == 0) wmin[wv] = best;
    __syncthreads();
    best = wmin[0];
#pragma unroll
    for (int i = 1; i < NW; ++i) best = wmin[i] < best ? wmin[i] : best;
    const int e = (int)(~(uint32_t)(best & 0xFFFFFFFFull));  // evicted slot, in [0, ncand)

    if (write_idx) {
        int32_t* idx = a.idx + (size_t)u * k;
        for (int i = tid; i < k; i += NT) idx[i] = i + (i >= e ? 1 : 0);
    }

    // ---- candidate part, dst rows [e, ncand-1)
    const int c = w_lo - e;                 // rows of it (>= 0)
    const bool c_in_regs = c <= NRW * L.RPI;  // one instruction per wave covers it
    uint4 creg = make_uint4(0u, 0u, 0u, 0u);
    int crow = -1;
    if (c > 0 && !c_in_regs) {
        // long: a streaming pass of its own, finished (reads and writes) before the window part stores
        if (wv >= 2) {
            int r0, r1, NI, last_i;
            bool has_last;
            uint4 first[G], last;
            range_of(e, w_lo, r0, r1);
            preload_range<G>(L, r0, r1, NI, first, has_last, last_i, last);
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __syncthreads();
            shift_range<G>(L, r0, NI, first, has_last, last_i, last);
        } else {
            __syncthreads();
        }
    } else if (c > 0 && wv >= 2) {
        const int r = e + (wv - 2) * L.RPI + L.rsub;
        if (r < w_lo) {
            crow = r;
            creg = stream_load(L.at(r + 1));
        }
    }
    // every source row that another wave will overwrite has been read
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();

    if (wv >= 2) {
        if (crow >= 0) stream_store(L.at(crow), creg);
        shift_range<G>(L, wr0, wNI, wfirst, whas_last, wlast_i, wlast);
    } else {
        // ---- score (wave 0) and pos (wave 1): one wave owns the whole range [e, k)
        uint32_t* arr = wv == 0 ? (uint32_t*)fu : (uint32_t*)pu;
        for (int i0 = e; i0 < k; i0 += kWave * G) {
            uint32_t regs[G];
#pragma unroll
            for (int g = 0; g < G; ++g) {
                const int i = i0 + g * kWave + lane;
                regs[g] = 0u;
                if (i < k) regs[g] = arr[i + 1];
            }
#pragma unroll
            for (int g = 0; g < G; ++g) {
                const int i = i0 + g * kWave + lane;
                if (i < k) arr[i] = regs[g];
            }
        }
    }
    if (tid == 0) a.len[u] = k;
}

// Candidate scan of long units ahead of the selection launch: workgroup (unit, slice) finds the smallest
// candidate of its slice of a decode-shape unit (len = k+1) -- by slot in the ordered layout (candidates are
// the slots below len-w, equal scores: the higher slot leaves), by position in the slot layout (candidates
// are the entries at least w positions behind the newest, equal scores: the higher position leaves).
constexpr int kPreselThreads = 256;
__global__ void __launch_bounds__(kPreselThreads) presel_kernel(const SelectArgs a, int64_t units) {
    __shared__ unsigned long long wmin_p[kPreselThreads / kWave];
    __shared__ int wslot_p[kPreselThreads / kWave];
    const int64_t u = blockIdx.x % units;  // slice-major ids: every XCD gets slices of every kind
    const int sl = (int)(blockIdx.x / units);
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int n = a.len[u];
    if (n != a.k + 1) return;  // the selection launch does not look at the slices of such a unit
    const float* fu = a.score + (size_t)u * a.cap;
    const int32_t* pu = a.pos + (size_t)u * a.cap;
    const int per = ((n + a.presel - 1) / a.presel + kPreselThreads - 1) / kPreselThreads * kPreselThreads;
    const int j0 = sl * per, j1 = min(n, j0 + per);
    const bool by_pos = a.layout == KF_LAYOUT_SLOT;
    const int newest = by_pos ? pu[n - 1] : 0;
    unsigned long long best = ~0ull;
    int best_slot = -1;
    for (int j = j0 + tid; j < j1; j += kPreselThreads) {
        const int pj = by_pos ? pu[j] : 0;
        const bool cand = by_pos ? (pj <= newest - a.w) : (j < n - a.w);
        if (cand) {
            const unsigned long long pack =
                ((unsigned long long)float_key(fu[j]) << 32) | (uint32_t)(~(uint32_t)(by_pos ? pj : j));
            if (pack < best) {
                best = pack;
                best_slot = j;
            }
        }
    }
    const unsigned long long mine = best;
    best = wave_min(best);
    // slots and positions are unique: one lane of the wave owns the wave's minimum
    const unsigned long long owner = __ballot(mine == best && best != ~0ull);
    const int wslot = __shfl(best_slot, owner ? __ffsll((long long)owner) - 1 : 0, kWave);
    if (lane == 0) {
        wmin_p[wv] = best;
        wslot_p[wv] = owner ? wslot : -1;
    }
    __syncthreads();
    if (tid == 0) {
        unsigned long long g = wmin_p[0];
        int gs = wslot_p[0];
        for (int i = 1; i < kPreselThreads / kWave; ++i)
            if (wmin_p[i] < g) {
                g = wmin_p[i];
                gs = wslot_p[i];
            }
        a.ws_pmin[(size_t)u * a.presel + sl] = g;
        a.ws_pslot[(size_t)u * a.presel + sl] = gs;
    }
}

// The evicted slot from the slices' minima (every lane gets it), -1 if no slice had a candidate.
__device__ __forceinline__ int presel_pick(const SelectArgs& a, int64_t u) {
    unsigned long long g = ~0ull;
    int gs = -1;
    for (int i = 0; i < a.presel; ++i) {
        const unsigned long long v = a.ws_pmin[(size_t)u * a.presel + i];
        if (v < g) {
            g = v;
            gs = a.ws_pslot[(size_t)u * a.presel + i];
        }
    }
    return gs;
}

// Slot-replacement variant of the same eviction (layout KF_LAYOUT_SLOT): the
// cache is an unordered set of (pos, K, V, score) entries.  The recent window
// is the w largest original positions -- positions are consecutive at the
// recent end, so "pos > newest - w" -- the candidate with the smallest score
// leaves (the highest position among equal minima, the same rule as above
// expressed through pos), and the newest entry (slot k) takes its slot: one row
// moves instead of every row behind the gap.
template <int NT>
__device__ __forceinline__ void evict_one_slot(const SelectArgs& a, int64_t u, int n, bool write_idx) {
    constexpr int NW = NT / kWave;
    __shared__ unsigned long long wmin_s[NW];
    __shared__ int s_slot;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int k = a.k, w = a.w;
    float* fu = a.score + (size_t)u * a.cap;
    int32_t* pu = a.pos + (size_t)u * a.cap;
    const int newest = pu[n - 1];

    if (!a.presel) {  // else the launch ahead scanned the candidates
        unsigned long long best = ~0ull, mine[2] = {~0ull, ~0ull};
        for (int j = tid, c = 0; j < n; j += NT, ++c) {
            const int pj = pu[j];
            unsigned long long pack = ~0ull;
            if (pj <= newest - w)  // a candidate: outside the recent window
                pack = ((unsigned long long)float_key(fu[j]) << 32) | (uint32_t)(~(uint32_t)pj);
            best = pack < best ? pack : best;
            if (c < 2) mine[c] = pack;
        }
        best = wave_min(best);
        if (lane == 0) wmin_s[wv] = best;
        if (tid == 0) s_slot = -1;
        __syncthreads();
        best = wmin_s[0];
#pragma unroll
        for (int i = 1; i < NW; ++i) best = wmin_s[i] < best ? wmin_s[i] : best;
        // positions are unique, so exactly one entry carries the winning pack
        if (best != ~0ull) {
            for (int j = tid, c = 0; j < n; j += NT, ++c) {
                unsigned long long pack;
                if (c < 2) {
                    pack = mine[c];
                } else {
                    const int pj = pu[j];
                    pack = (pj <= newest - w)
                               ? (((unsigned long long)float_key(fu[j]) << 32) | (uint32_t)(~(uint32_t)pj))
                               : ~0ull;
                }
                if (pack == best) s_slot = j;
            }
        }
        __syncthreads();
    }
    const int e = a.presel ? presel_pick(a, u) : s_slot;
    if (e < 0) {  // no entry lies outside the window (positions not consecutive at the recent end): report
        if (tid == 0) atomicAdd(a.ws_err, 1);
        return;
    }
    if (write_idx) {
        int32_t* idx = a.idx + (size_t)u * k;
        for (int i = tid; i < k; i += NT) idx[i] = (i == e) ? k : i;
    }
    if (e != k) {  // the newest entry moves into the freed slot
        const int PPR = a.row_bytes >> 4;
        if (tid < 2 * PPR) {
            uint4* base = (uint4*)((char*)(tid < PPR ? a.K : a.V) + (size_t)u * a.cap * a.row_bytes);
            const int piece = tid % PPR;
            base[(size_t)e * PPR + piece] = base[(size_t)k * PPR + piece];
        } else if (tid == 2 * PPR) {
            fu[e] = fu[k];
        } else if (tid == 2 * PPR + 1) {
            pu[e] = newest;
        }
    }
    if (tid == 0) a.len[u] = k;
}

// Decode-shape eviction in the ordered layout, first of two launches ("wide" mode, for workloads whose
// units are too few or too long for one workgroup each to move the rows): find the evicted slot e exactly
// as evict_one does, and save the entries at slots R, 2R, ... behind it.  The second launch gives every
// R-slot chunk of [e, k) to a workgroup of its own; a chunk's last source is the next chunk's first
// destination, and that one entry is read from the copy saved here, so the chunks need no order.
template <int NT>
__device__ __forceinline__ void evict_find(const SelectArgs& a, int64_t u, int n, bool write_idx) {
    constexpr int NW = NT / kWave;
    __shared__ unsigned long long wmin_f[NW];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int k = a.k, w = a.w;
    const int ncand = n - w;
    const float* fu = a.score + (size_t)u * a.cap;
    const int32_t* pu = a.pos + (size_t)u * a.cap;
    int e;
    if (a.presel) {
        e = presel_pick(a, u);  // the launch ahead scanned the candidates
    } else {
        unsigned long long best = ~0ull;
        for (int j = tid; j < ncand; j += NT) {
            const unsigned long long pack = ((unsigned long long)float_key(fu[j]) << 32) | (uint32_t)(~(uint32_t)j);
            best = pack < best ? pack : best;
        }
        best = wave_min(best);
        if (lane == 0) wmin_f[wv] = best;
        __syncthreads();
        best = wmin_f[0];
#pragma unroll
        for (int i = 1; i < NW; ++i) best = wmin_f[i] < best ? wmin_f[i] : best;
        e = (int)(~(uint32_t)(best & 0xFFFFFFFFull));  // evicted slot, in [0, ncand)
    }
    if (write_idx) {
        int32_t* idx = a.idx + (size_t)u * k;
        for (int i = tid; i < k; i += NT) idx[i] = i + (i >= e ? 1 : 0);
    }
    // boundary entries at slots b = (c+1)*R with e < b <= k
    const int R = a.chunk_rows, PPR = a.row_bytes >> 4;
    const int c0 = e / R, c1 = k / R;  // boundaries c0 .. c1-1
    const uint4* Kr = (const uint4*)((const char*)a.K + (size_t)u * a.cap * a.row_bytes);
    const uint4* Vr = (const uint4*)((const char*)a.V + (size_t)u * a.cap * a.row_bytes);
    uint4* brow = (uint4*)((char*)a.ws_brow + (size_t)u * a.nb * 2 * a.row_bytes);
    const int per = 2 * PPR;  // pieces per boundary: the K row, then the V row
    for (int p = tid; p < (c1 - c0) * per; p += NT) {
        const int c = c0 + p / per, q = p % per;
        const int b = (c + 1) * R;
        brow[(size_t)c * per + q] = (q < PPR) ? Kr[(size_t)b * PPR + q] : Vr[(size_t)b * PPR + q - PPR];
    }
    for (int c = c0 + tid; c < c1; c += NT) {
        a.ws_bscore[(size_t)u * a.nb + c] = fu[(c + 1) * R];
        a.ws_bpos[(size_t)u * a.nb + c] = pu[(c + 1) * R];
    }
    if (tid == 0) {
        a.ws_evict[u] = e;
        a.len[u] = k;
    }
}

// Second launch of the wide mode: workgroup (unit u, chunk c) moves entries [max(e, cR)+1, min(k, (c+1)R)]
// down by one slot.  Everything it reads is in registers before its one barrier; its last source, if it is
// the next chunk's first destination, comes from the copy the first launch saved.
constexpr int kWideThreads = 256;
constexpr int kWidePieces = 2048 / kWideThreads;  // 16-byte pieces per thread and tensor
// LDS that a workgroup asks for and does not use: two of them on a compute unit (128 KB of rows in flight) instead of the five that
// its registers allow.  A workgroup first only reads and then only writes; with fewer of them the memory changes direction less
// often.  Ordered steps, caches in turn, at five / three / two / one on a compute unit: 32 x 9830 x 128 61.0 / 59.7 / 58.9 / 62.0 us,
// 256 x 1501 x 128 with 4 query heads 63.5 / 61.4 / 61.1 / 63.3, 256 x 2048 x 128 73.0 / 71.8 / 72.4 / 75.6, 100 x 3000 x 128
// 54.2 / 53.7 / 52.6 / 54.1, 32 x 32000 x 128 162 / 162 / 160 / 169.  (Eviction into another cache, whose workgroups read
// and write a few rows at a time, loses by it: 399 us, 417 with six on a compute unit, 444 with five.)
// Launches of many units and chunks lose by it too (ordered steps, two / five on a compute unit, a window of half / nine tenths of the
// budget): 128 x 16000 x 128 497 / 493 and 578 / 568 us, 128 x 32000 999 / 978 and 1169 / 1134, 256 x 16000 1011 / 986 and 1182 /
// 1146.  The same or a gain: 256 x 8192 479 / 482 and 559 / 558, 64 x 16000 225 / 230 and 293 / 294, 32 x 60000 462 / 465 and 530 / 532.
constexpr int kShiftLds = 60 * 1024;
constexpr int64_t kShiftLdsMaxWorkgroups = 12288;  // above, only launches of up to this many units ask for it:
constexpr int64_t kShiftLdsMaxUnits = 32;
__global__ void __launch_bounds__(kWideThreads) shift_chunk_kernel(const SelectArgs a, int nchunks, int64_t units) {
    // chunk-major: the chunks that have work are the same few of every unit (those behind the evicted slot),
    // and consecutive workgroup ids go round-robin to the 8 XCDs -- unit-major ids would park all the work on
    // the XCDs those chunk numbers map to (measured: half the chip idle, 84 instead of 40 us)
    const int64_t u = blockIdx.x % units;
    const int c = (int)(blockIdx.x / units);
    const int e = a.ws_evict[u];
    if (e < 0) return;
    const int R = a.chunk_rows, k = a.k, PPR = a.row_bytes >> 4;
    const int lo = max(e, c * R), hi = min(k, (c + 1) * R);
    if (lo >= hi) return;
    const int rows = hi - lo, bnd = (c + 1) * R;  // sources lo+1 .. hi; source `bnd` is saved
    const int tid = threadIdx.x;
    uint4* Kr = (uint4*)((char*)a.K + (size_t)u * a.cap * a.row_bytes);
    uint4* Vr = (uint4*)((char*)a.V + (size_t)u * a.cap * a.row_bytes);
    const uint4* brow = (const uint4*)((const char*)a.ws_brow + ((size_t)u * a.nb + c) * 2 * a.row_bytes);
    float* fu = a.score + (size_t)u * a.cap;
    int32_t* pu = a.pos + (size_t)u * a.cap;
    // branch-free: a lane past the chunk's end re-reads the last source, the saved entry is a pointer choice
    uint4 kreg[kWidePieces], vreg[kWidePieces];
#pragma unroll
    for (int i = 0; i < kWidePieces; ++i) {
        const int p = tid + i * kWideThreads;
        const int q = p % PPR;
        const int src = lo + min(p / PPR, rows - 1) + 1;
        const uint4* ks = (src == bnd) ? brow + q : Kr + (size_t)src * PPR + q;
        const uint4* vs = (src == bnd) ? brow + PPR + q : Vr + (size_t)src * PPR + q;
        kreg[i] = stream_load(ks);
        vreg[i] = stream_load(vs);
    }
    float fs = 0.0f;
    int32_t ps = 0;
    if (tid < rows) {
        const int src = lo + tid + 1;
        fs = (src == bnd) ? a.ws_bscore[(size_t)u * a.nb + c] : fu[src];
        ps = (src == bnd) ? a.ws_bpos[(size_t)u * a.nb + c] : pu[src];
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // (the barrier by itself does not wait for loads)
    __syncthreads();  // every source of the chunk is in registers
#pragma unroll
    for (int i = 0; i < kWidePieces; ++i) {
        const int p = tid + i * kWideThreads;
        const int r = p / PPR, q = p % PPR;
        if (r < rows) {
            stream_store(Kr + (size_t)(lo + r) * PPR + q, kreg[i]);
            stream_store(Vr + (size_t)(lo + r) * PPR + q, vreg[i]);
        }
    }
    if (tid < rows) {
        fu[lo + tid] = fs;
        pu[lo + tid] = ps;
    }
}

// Selection and compaction of one unit by one workgroup.
template <int NT>
__device__ __forceinline__ void select_unit(const SelectArgs& a, int64_t u) {
    constexpr int NW = NT / kWave;
    __shared__ uint32_t hist[256];
    __shared__ uint32_t s_bin, s_rem;
    __shared__ uint32_t wtot[NW][2];
    __shared__ int s_first;

    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int n = a.len[u];
    const int k = a.k, w = a.w;
    int32_t* idx = a.idx + (size_t)u * k;

    if (a.wide && tid == 0) a.ws_evict[u] = -1;  // unless the decode-shape branch below says otherwise
    if (n <= k) {  // under budget: nothing leaves
        if (a.idx_is_output || !a.move)
            for (int i = tid; i < k; i += NT) idx[i] = (i < n) ? i : -1;
        return;
    }
    if (a.layout == KF_LAYOUT_SLOT) {
        if (n == k + 1) {
            evict_one_slot<NT>(a, u, n, a.idx_is_output != 0);
        } else if (tid == 0) {
            atomicAdd(a.ws_err, 1);  // more than one token over budget: not handled in this layout
        }
        return;
    }
    if (n == k + 1 && a.move) {  // decode shape
        if (a.wide) {
            __syncthreads();  // the -1 above is stored before this workgroup's own slot number
            evict_find<NT>(a, u, n, a.idx_is_output != 0);
        } else {
            evict_one<NT>(a, u, n, a.idx_is_output != 0);
        }
        return;
    }
    const int ncand = n - w, nkey = k - w;
    float* fu = a.score + (size_t)u * a.cap;
    int32_t* pu = a.pos + (size_t)u * a.cap;

    // ---- select: threshold key T = the nkey-th largest candidate key
    uint32_t T = 0xFFFFFFFFu, need = 0;
    if (nkey > 0) {
        uint32_t prefix = 0, mask = 0, remaining = (uint32_t)nkey;
        for (int shift = 24; shift >= 0; shift -= 8) {
            if (tid < 256) hist[tid] = 0;
            __syncthreads();
            for (int j = tid; j < ncand; j += NT) {
                const uint32_t key = float_key(fu[j]);
                if ((key & mask) == prefix) atomicAdd(&hist[(key >> shift) & 255u], 1u);
            }
            __syncthreads();
            if (tid < kWave) {
                // lane owns bins [4*lane, 4*lane+4); count of keys in higher bins first
                uint32_t c[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) c[i] = hist[tid * 4 + i];
                const uint32_t tot = c[0] + c[1] + c[2] + c[3];
                uint32_t incl = tot;  // becomes the sum over lanes >= this one
#pragma unroll
                for (int o = 1; o < kWave; o <<= 1) {
                    const uint32_t t = __shfl_down(incl, o, kWave);
                    if (tid + o < kWave) incl += t;
                }
                uint32_t above = incl - tot;
#pragma unroll
                for (int i = 3; i >= 0; --i) {
                    if (above < remaining && remaining <= above + c[i]) {
                        s_bin = (uint32_t)(tid * 4 + i);
                        s_rem = remaining - above;
                    }
                    above += c[i];
                }
            }
            __syncthreads();
            prefix |= s_bin << shift;
            mask |= 0xFFu << shift;
            remaining = s_rem;
        }
        T = prefix;
        need = remaining;  // how many candidates equal to T survive (lowest slots first)
    }

    // ---- rank: ordered sweep, destination of every survivor
    if (tid == 0) s_first = k;
    __syncthreads();
    uint32_t run_gt = 0, run_eq = 0;
    for (int base = 0; base < ncand; base += NT) {
        const int j = base + tid;
        bool gt = false, eq = false;
        if (j < ncand && nkey > 0) {
            const uint32_t key = float_key(fu[j]);
            gt = key > T;
            eq = key == T;
        }
        const unsigned long long bg = __ballot(gt), be = __ballot(eq);
        const unsigned long long below = (1ull << lane) - 1ull;
        if (lane == 0) {
            wtot[wv][0] = (uint32_t)__popcll(bg);
            wtot[wv][1] = (uint32_t)__popcll(be);
        }
        __syncthreads();
        uint32_t gt_before = run_gt + (uint32_t)__popcll(bg & below);
        uint32_t eq_before = run_eq + (uint32_t)__popcll(be & below);
        uint32_t tg = 0, te = 0;
#pragma unroll
        for (int i = 0; i < NW; ++i) {
            if (i < wv) {
                gt_before += wtot[i][0];
                eq_before += wtot[i][1];
            }
            tg += wtot[i][0];
            te += wtot[i][1];
        }
        const bool keep = gt || (eq && eq_before < need);
        if (keep) {
            const uint32_t dst = gt_before + min(eq_before, need);
            if (dst < (uint32_t)nkey) idx[dst] = j;  // always true; keeps a logic error in bounds
        } else if (j < ncand) {
            atomicMin(&s_first, j);  // first slot that changes occupant
        }
        run_gt += tg;
        run_eq += te;
        __syncthreads();
    }
    for (int i = tid; i < w; i += NT) idx[nkey + i] = ncand + i;  // the recent window
    __syncthreads();  // idx and s_first are complete for the whole workgroup
    if (!a.move) return;  // index list only: the rows are gathered into another cache by gather_kernel

    // ---- compact: front-to-back gather through registers
    const int PPR = a.row_bytes >> 4;  // 16-byte pieces per row
    const int rpp = NT / PPR;          // rows per pass of the workgroup
    const int R = rpp * kSelectGroups; // rows per tile
    const int piece = tid % PPR, rsub = tid / PPR;
    uint4* Kb = (uint4*)((char*)a.K + (size_t)u * a.cap * a.row_bytes);
    uint4* Vb = (uint4*)((char*)a.V + (size_t)u * a.cap * a.row_bytes);
    for (int t0 = s_first; t0 < k; t0 += R) {
        uint4 rk[kSelectGroups], rv[kSelectGroups];
        int src[kSelectGroups];
#pragma unroll
        for (int g = 0; g < kSelectGroups; ++g) {
            const int i = t0 + g * rpp + rsub;
            src[g] = (i < k) ? idx[i] : -1;
            if (src[g] >= n) src[g] = -1;  // cannot happen; never read past the unit
            rk[g] = make_uint4(0u, 0u, 0u, 0u);
            rv[g] = make_uint4(0u, 0u, 0u, 0u);
            if (src[g] >= 0 && src[g] != i) {
                rk[g] = Kb[(size_t)src[g] * PPR + piece];
                rv[g] = Vb[(size_t)src[g] * PPR + piece];
            }
        }
        float fv = 0.0f;
        int pv = 0, ssrc = -1;
        const int si = t0 + tid;
        if (tid < R && si < k) {
            ssrc = idx[si];
            if (ssrc >= n) ssrc = -1;
            if (ssrc >= 0) {
                fv = fu[ssrc];
                pv = pu[ssrc];
            }
        }
        // the loads above must have returned before any thread overwrites a row
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
#pragma unroll
        for (int g = 0; g < kSelectGroups; ++g) {
            const int i = t0 + g * rpp + rsub;
            if (src[g] >= 0 && src[g] != i) {
                Kb[(size_t)i * PPR + piece] = rk[g];
                Vb[(size_t)i * PPR + piece] = rv[g];
            }
        }
        if (ssrc >= 0 && ssrc != si) {
            fu[si] = fv;
            pu[si] = pv;
        }
    }
    if (tid == 0) a.len[u] = k;
}

// Last launch of a step whose number lives in device memory: one lane moves the
// counter on.  No workgroup of this launch reads the counter, and the next
// step's launches start after this one has drained.
__device__ __forceinline__ void advance_step(const SelectArgs& a) {
    if (a.step_inc && blockIdx.x == 0 && threadIdx.x == 0) *a.step_inc += 1;
}

template <int NT>
__global__ void __launch_bounds__(NT) select_kernel(const SelectArgs a) {
    select_unit<NT>(a, (int64_t)blockIdx.x);
    advance_step(a);
}

// Tail of a fused generation step: merge the decode kernel's split records of
// the unit (attention output, score accumulation, new length), then select and
// compact -- one launch instead of two.
template <int D, int NT, int G>
__global__ void __launch_bounds__(NT) step_tail_kernel(const DecodeArgs d, const SelectArgs a) {
    __shared__ float w_p[G * kDecodeMaxSplits], w_e[G * kDecodeMaxSplits];
    const int64_t u = blockIdx.x;
    const int len0 = d.len[u];
    if (len0 >= 0 && len0 < d.cap && len0 <= d.S * d.chunk) {  // else: skipped by the split kernel too
        merge_unit<D, NT, G>(d, u, len0, w_p, w_e, 0, len0 + 1, true);
        __syncthreads();  // the merged scores and the new length are visible to the whole workgroup
    } else if (d.pre_slices > 0 && len0 == d.pre_k + 1) {
        scan_slice_min<NT>(d, u, len0, 0, len0, 0);  // the selection below takes the evicted slot from the table
        __syncthreads();
    }
    select_unit<NT>(a, u);
    advance_step(a);
}

// Second and last launch of a generation step of few units in the ordered layout: merge of the split records,
// selection and compaction, several workgroups per unit.  Such a launch is bound by its chain of memory round trips,
// not by bytes, so one launch whose workgroups repeat each other's small work replaces two (merge + selection, then
// the row shift): workgroup (unit, chunk) merges the statistics and forms ALL the unit's new scores in LDS, finds the
// evicted slot by itself and moves the R entries of its own chunk.  The split launch left copies of what one
// workgroup overwrites while another still reads it: the old scores, and the rows and positions at slots R, 2R, ...
// (a chunk's last source is the next chunk's first destination).  Rows that move whatever slot leaves are loaded
// before it is known.  One more workgroup per unit writes the attention outputs (and does what the others leave).
//
// What bounds it besides the chain of trips is its own length: a compute unit has one such workgroup, a wave to a SIMD, so every
// instruction of a wave counts, and so does every line of the argument buffer that is fetched when first used.  Hence FinishArgs
// (what the usual path reads, in one stretch), addresses formed by shifts from one offset, and loads without a bound each: 16
// units x 1024 x 256 7.1 -> 6.0 us, the ordered step with its split launch 15.4 -> 13.0, 64 x 2048 x 128 28.5 -> 25.7, 4 heads
// 32 x 1024 x 128 20.9 -> 18.8, 8 heads 64 x 300 x 256 29.4 -> 27.0 (graphs, caches in turn).
constexpr int kFinishThreads = 256;
struct FinishArgs {
    const int32_t* m;    // tokens the splits scored per unit
    const float* part;   // their records
    const float* inc;    // ... and increments
    const float* f_old;  // the scores before the step
    char* K;
    char* V;
    float* score;
    int32_t* pos;
    const char* brow;    // rows and positions at the chunk boundaries
    const int32_t* bpos;
    float* out;
    int32_t* len;
    int32_t* idx;        // the caller's kept_idx, or NULL
    int32_t* step_inc;
    int32_t cap, k, w, S, chunk, R, nb, row_shift;  // row_shift: log2 of a row's bytes
};
struct FinishLaunch {
    FinishArgs f;
    DecodeArgs d;  // what the general way reads
    SelectArgs a;
};
template <int D, int G>
__global__ void __launch_bounds__(kFinishThreads) step_finish_kernel(const FinishLaunch x) {
    const FinishArgs& f = x.f;
    constexpr int NT = kFinishThreads, NW = NT / kWave, PW = D + 4, TOK = 4;
    __shared__ float w_p[G * kFewMaxSplits], w_e[G * kFewMaxSplits], inv_p[G];
    __shared__ float f_new[kFinishMaxTokens + 1];
    __shared__ unsigned long long wmin_f[NW];
    asm volatile("" ::"s"(f.m), "s"(f.part), "s"(f.inc), "s"(f.f_old), "s"(f.K), "s"(f.V), "s"(f.score), "s"(f.pos), "s"(f.brow), "s"(f.bpos),
                 "s"(f.out), "s"(f.len), "s"(f.idx), "s"(f.cap), "s"(f.k), "s"(f.w), "s"(f.S), "s"(f.chunk), "s"(f.R), "s"(f.nb), "s"(f.row_shift));
    const int64_t u = blockIdx.x;         // chunk-major: every XCD gets chunks of every kind
    const int c = (int)blockIdx.y - 1;    // -1: the attention outputs
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int k = f.k, w = f.w, S = f.S, last = f.cap - 1;
    int m = uniform_load(f.m + u);  // tokens the splits scored; 0: they skipped the unit
    const int R = f.R;
    const int lo = c * R, hi = min(k, lo + R), rows = hi - lo;  // destinations [lo, hi), sources lo+1 .. hi
    const int saved = lo + R < k ? lo + R : -1;                 // this source comes from the copy
    const size_t unit_bytes = (size_t)f.cap << f.row_shift;
    char *Kr = f.K + u * unit_bytes, *Vr = f.V + u * unit_bytes;
    float* fu = f.score + (size_t)u * f.cap;
    int32_t* pu = f.pos + (size_t)u * f.cap;

    // ---- everything that can be asked for now, before m is known (another trip to memory): split statistics, increments, old
    // scores, positions, certain rows.  Of a unit that turns out to go the general way it is dropped, and slot k, which a cache
    // of capacity k does not have, is read as its last one.
    constexpr int HPW = (G + NW - 1) / NW;  // heads per wave: one wave merges a head's statistics, a lane a split
    const float* parts = f.part + (size_t)u * S * G * PW;
    float4 rec[HPW];
#pragma unroll
    for (int i = 0; i < HPW; ++i) {
        const int g = wv + i * NW;
        rec[i] = make_float4(-INFINITY, 0.0f, -INFINITY, 0.0f);
        if (g < G && lane < S) rec[i] = *reinterpret_cast<const float4*>(parts + (lane * G + g) * PW + D);
    }
    const float* we = f.inc + (size_t)u * G * f.cap;
    const float* f_old = f.f_old + (size_t)u * f.cap;
    float te[TOK][G], tf[TOK], tnew[G];
    auto load_tokens = [&](int j0) {
#pragma unroll
        for (int i = 0; i < TOK; ++i) {
            const int j = min(j0 + i * NT, last);
#pragma unroll
            for (int g = 0; g < G; ++g) te[i][g] = we[g * f.cap + j];
            tf[i] = f_old[j];
        }
    };
    // the outputs' first split records, or what the scores and the move need
    constexpr int OREC = 16, OPT = (G * D + NT - 1) / NT;  // records in flight, outputs per thread
    auto load_records = [&](int o, int s0, float(&rec)[OREC]) {
        const int idx = min(tid + o * NT, G * D - 1);
        const float* pr = parts + (idx / D) * PW + idx % D;
#pragma unroll
        for (int i = 0; i < OREC; i += 8)
            if (s0 + i < S) {
#pragma unroll
                for (int j = 0; j < 8; ++j) rec[i + j] = pr[min(s0 + i + j, S - 1) * G * PW];
            }
    };
    const int q16 = (tid << 4) & ((1 << f.row_shift) - 1), r0 = (tid << 4) >> f.row_shift, rstep = (NT << 4) >> f.row_shift;
    const char* brow = f.brow + (((size_t)u * f.nb + max(c, 0)) << (f.row_shift + 1));
    uint4 kreg[kWidePieces], vreg[kWidePieces];
    auto load_rows = [&]() {  // branch-free: a lane past the chunk's end re-reads the last source
#pragma unroll
        for (int i = 0; i < kWidePieces; ++i) {
            const int src = min(lo + 1 + r0 + i * rstep, min(hi, last));
            const uint32_t off = ((uint32_t)src << f.row_shift) + q16;
            if (i < kWidePieces - 1) {
                kreg[i] = stream_load((const uint4*)(Kr + off));
                vreg[i] = stream_load((const uint4*)(Vr + off));
            } else {  // (a chunk whose last source is saved is a whole one: its last row is the last piece's)
                const bool copy = src == saved;
                kreg[i] = stream_load((const uint4*)(copy ? brow + q16 : Kr + off));
                vreg[i] = stream_load((const uint4*)(copy ? brow + (1 << f.row_shift) + q16 : Vr + off));
            }
        }
    };
    // statistics of the splits -> weights
    auto weights = [&]() {
#pragma unroll
        for (int i = 0; i < HPW; ++i) {
            const int g = wv + i * NW;
            const float Mx = wave_max(rec[i].x), My = wave_max(rec[i].z);
            const float wp = rec[i].y > 0.0f ? hw_exp2(rec[i].x - Mx) : 0.0f;  // empty splits weigh nothing
            const float we_ = rec[i].w > 0.0f ? hw_exp2(rec[i].z - My) : 0.0f;
            const float sumP = wave_sum(fmaf(wp, rec[i].y, 0.0f)), invE = 1.0f / wave_sum(fmaf(we_, rec[i].w, 0.0f));  // as merge_unit, to the bit
            if (g < G && lane < S) {
                w_p[g * S + lane] = wp;
                w_e[g * S + lane] = we_ * invE;
            }
            if (g < G && lane == 0) inv_p[g] = 1.0f / sumP;
        }
        __syncthreads();
    };
    if (c < 0) {  // the attention outputs
        float first[OREC], next[OREC];
        load_records(0, 0, first);
        asm volatile("" : "+s"(m)::"memory");  // (the loads stay ahead of the branch)
        if (m != k + 1) {                      // within budget, or far over it: this workgroup does the unit the general way
            // (its arguments by way of a pointer that the compiler does not see through: it fetched them ahead of the branch)
            const __attribute__((address_space(4))) char* arg = (const __attribute__((address_space(4))) char*)__builtin_amdgcn_kernarg_segment_ptr();
            asm volatile("" : "+s"(arg));
            const DecodeArgs d = *(const DecodeArgs*)(arg + offsetof(FinishLaunch, d));
            const SelectArgs a = *(const SelectArgs*)(arg + offsetof(FinishLaunch, a));
            if (m > 0) merge_unit<D, NT, G>(d, u, m - 1, w_p, w_e, 0, m, true);
            if (!a.rest) {
                __syncthreads();
                select_unit<NT>(a, u);
            }
        } else {
            load_records(0, OREC, next);
            weights();
            for (int o = 0; o < OPT; ++o) {
                const int idx = tid + o * NT, g = min(idx / D, G - 1);
                float sum = 0.0f;
                for (int s0 = 0; s0 < S; s0 += 2 * OREC) {  // summed in split order
                    if (o > 0 || s0 > 0) {
                        load_records(o, s0, first);
                        load_records(o, s0 + OREC, next);
                    }
#pragma unroll
                    for (int i = 0; i < OREC; ++i)
                        if (s0 + i < S) sum = fmaf(w_p[g * S + s0 + i], first[i], sum);
#pragma unroll
                    for (int i = 0; i < OREC; ++i)
                        if (s0 + OREC + i < S) sum = fmaf(w_p[g * S + s0 + OREC + i], next[i], sum);
                }
                if (idx < G * D) f.out[u * G * D + idx] = sum * inv_p[g];
            }
            if (tid == 0) f.len[u] = k;
        }
        if (u == 0 && tid == 0 && f.step_inc) *f.step_inc += 1;  // (no workgroup of this launch reads it)
        return;
    }
    load_tokens(tid);
#pragma unroll
    for (int g = 0; g < G; ++g) tnew[g] = we[g * f.cap + min(k, last)];
    int32_t p_next = 0;
    if (tid < rows) p_next = *(lo + tid + 1 == saved ? f.bpos + (size_t)u * f.nb + c : pu + min(lo + tid + 1, last));
    const bool sure = hi > k - w;  // the chunk reaches into the part behind the candidates, which moves in any case
    if (sure) load_rows();
    asm volatile("" : "+s"(m)::"memory");
    if (m != k + 1) return;
    weights();

    // ---- new scores of the whole unit, smallest candidate (the highest slot among equals)
    unsigned long long best = ~0ull;
    auto increment = [&](const float(&e)[G], int split) {
        float df = 0.0f;
#pragma unroll
        for (int g = 0; g < G; ++g) df = fmaf(e[g], w_e[g * S + split], df);
        return df;
    };
    auto candidate = [&](float v, int j) {
        f_new[j] = v;
        if (j < k + 1 - w) {
            const unsigned long long pack = ((unsigned long long)float_key(v) << 32) | (uint32_t)(~(uint32_t)j);
            best = pack < best ? pack : best;
        }
    };
    // j / chunk: (j + 1/2) / chunk is no closer than 1/1024 to a whole number, and at most 64
    const float per_chunk = __builtin_amdgcn_rcpf((float)f.chunk);
    for (int j0 = tid; j0 < k; j0 += TOK * NT) {
        if (j0 != tid) load_tokens(j0);
#pragma unroll
        for (int i = 0; i < TOK; ++i) {
            const int j = j0 + i * NT;
            if (j < k) candidate(tf[i] + increment(te[i], (int)(((float)j + 0.5f) * per_chunk)), j);
        }
    }
    if (tid == 0) candidate(increment(tnew, S - 1), k);  // the new token belongs to the last split and starts from zero
    best = wave_min(best);
    if (lane == 0) wmin_f[wv] = best;
    __syncthreads();
    best = wmin_f[0];
#pragma unroll
    for (int i = 1; i < NW; ++i) best = wmin_f[i] < best ? wmin_f[i] : best;
    const int e = (int)(~(uint32_t)(best & 0xFFFFFFFFull));  // evicted slot, in [0, k+1-w)

    // ---- move the chunk
    if (!sure && hi > e) load_rows();
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // every source of this chunk is in registers ...
    __syncthreads();                                  // ... of every wave, before any of them is overwritten
    if (hi > e) {
#pragma unroll
        for (int i = 0; i < kWidePieces; ++i) {
            const int dst = lo + r0 + i * rstep;
            const uint32_t off = ((uint32_t)dst << f.row_shift) + q16;
            if (dst < hi && dst >= e) {
                stream_store((uint4*)(Kr + off), kreg[i]);
                stream_store((uint4*)(Vr + off), vreg[i]);
            }
        }
    }
    if (tid < rows) {
        const int i = lo + tid;
        fu[i] = f_new[i + (i >= e ? 1 : 0)];
        if (i >= e) pu[i] = p_next;
        if (f.idx) f.idx[(size_t)u * k + i] = i + (i >= e ? 1 : 0);
    }
}

// The kernel reads parts of its argument by way of the argument buffer: it is the only one, so it lies at the buffer's begin.
static_assert(std::is_same<decltype(&step_finish_kernel<64, 1>), void (*)(FinishLaunch)>::value, "one argument");
static_assert(std::is_standard_layout<FinishLaunch>::value && std::is_trivially_copyable<FinishLaunch>::value, "read as bytes");

template <int D>
static hipError_t launch_step_finish_d(const DecodeArgs& d, const SelectArgs& a, int64_t U, hipStream_t st) {
    const int nchunks = (a.k + a.chunk_rows - 1) / a.chunk_rows;
    FinishLaunch x{{}, d, a};
    FinishArgs& f = x.f;
    f.m = d.ws_m;
    f.part = d.ws_part;
    f.inc = d.ws_e;
    f.f_old = d.few_f;
    f.K = (char*)a.K;
    f.V = (char*)a.V;
    f.score = a.score;
    f.pos = a.pos;
    f.brow = (const char*)a.ws_brow;
    f.bpos = a.ws_bpos;
    f.out = d.out;
    f.len = a.len;
    f.idx = a.idx_is_output ? a.idx : nullptr;
    f.step_inc = a.step_inc;
    f.cap = a.cap;
    f.k = a.k;
    f.w = a.w;
    f.S = d.S;
    f.chunk = d.chunk;
    f.R = a.chunk_rows;
    f.nb = a.nb;
    f.row_shift = __builtin_ctz(a.row_bytes);
    const dim3 grid((unsigned)U, (unsigned)(nchunks + 1)), block(kFinishThreads);
    switch (d.G) {
        case 1: hipLaunchKernelGGL((step_finish_kernel<D, 1>), grid, block, 0, st, x); break;
        case 2: hipLaunchKernelGGL((step_finish_kernel<D, 2>), grid, block, 0, st, x); break;
        case 4: hipLaunchKernelGGL((step_finish_kernel<D, 4>), grid, block, 0, st, x); break;
        case 8: hipLaunchKernelGGL((step_finish_kernel<D, 8>), grid, block, 0, st, x); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_step_finish(const DecodeArgs& d, const SelectArgs& a, int64_t U, int32_t hd, hipStream_t stream) {
    // what the kernel's tables hold
    if (a.k > kFinishMaxTokens || d.S > kWave || d.S > kFewMaxSplits || a.chunk_rows > kFinishThreads) return hipErrorInvalidValue;
    if (hd == 64) return launch_step_finish_d<64>(d, a, U, stream);
    if (hd == 128) return launch_step_finish_d<128>(d, a, U, stream);
    if (hd == 256) return launch_step_finish_d<256>(d, a, U, stream);
    return hipErrorInvalidValue;
}

// Where a unit can be further over its budget (the launch above is told by a.rest): those units, by workgroups large
// enough to move their rows.  The launch above's own 256 threads took 146 us for 16 units of 2047 tokens x 256 cut to
// 1024 (78 so; 32 x 4095 x 128 to 2048: 161, 94); made of 1024 threads it cost every ordinary step 10 to 20 %.
// An empty launch otherwise.
__global__ void __launch_bounds__(kSelectThreads) step_rest_kernel(const int32_t* m, const SelectArgs a) {
    if (m[blockIdx.x] == a.k + 1) return;
    select_unit<kSelectThreads>(a, (int64_t)blockIdx.x);
}
hipError_t launch_step_rest(const DecodeArgs& d, const SelectArgs& a, int64_t U, hipStream_t stream) {
    hipLaunchKernelGGL(step_rest_kernel, dim3((unsigned)U), dim3(kSelectThreads), 0, stream, d.ws_m, a);
    return hipGetLastError();
}

template <int NT, int G>
static hipError_t launch_step_tail_g(const DecodeArgs& d, const SelectArgs& a, int64_t U, int32_t hd,
                                     hipStream_t stream) {
    const dim3 grid((unsigned)U), block(NT);
    if (hd == 64) hipLaunchKernelGGL((step_tail_kernel<64, NT, G>), grid, block, 0, stream, d, a);
    else if (hd == 128) hipLaunchKernelGGL((step_tail_kernel<128, NT, G>), grid, block, 0, stream, d, a);
    else if (hd == 256) hipLaunchKernelGGL((step_tail_kernel<256, NT, G>), grid, block, 0, stream, d, a);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

template <int NT>
static hipError_t launch_step_tail_nt(const DecodeArgs& d, const SelectArgs& a, int64_t U, int32_t hd,
                                      hipStream_t stream) {
    switch (d.G) {
        case 1: return launch_step_tail_g<NT, 1>(d, a, U, hd, stream);
        case 2: return launch_step_tail_g<NT, 2>(d, a, U, hd, stream);
        case 4: return launch_step_tail_g<NT, 4>(d, a, U, hd, stream);
        case 8: return launch_step_tail_g<NT, 8>(d, a, U, hd, stream);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_step_tail(const DecodeArgs& d, const SelectArgs& a, int64_t U, int32_t hd, hipStream_t stream) {
    if (a.layout == KF_LAYOUT_SLOT) return launch_step_tail_nt<kSelectThreadsSlot>(d, a, U, hd, stream);
    return launch_step_tail_nt<kSelectThreads>(d, a, U, hd, stream);
}

// Survivor lists alone, for the eviction into another cache: the selection of select_unit with the unit's keys held
// in registers.  A thread owns KPT neighbouring slots, so the stable ranks take one wave scan and one exchange
// between the waves instead of a sweep with two barriers per NT slots, and the radix passes read no memory.  Each
// pass has a histogram of its own and every wave finds the digit by itself: one barrier a pass.  select_kernel spent
// 96 us on 2048 units of 2048 tokens (sixteen waves a unit, two units a CU at a time, five reads of the scores, some
// thirty barriers each); this takes 24, next to a row copy of 374 (one unit-layer of 32 heads x 32768 tokens: the call
// 211 -> 113 us).
template <int NT, int KPT>
__global__ void __launch_bounds__(NT) select_list_kernel(const SelectArgs a) {
    constexpr int NW = NT / kWave;
    __shared__ __attribute__((aligned(16))) uint32_t hist[4][256];
    __shared__ uint32_t wtot[NW];
    const int64_t u = (int64_t)blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int n = a.len[u];
    const int k = a.k, w = a.w;
    int32_t* idx = a.idx + (size_t)u * k;
    if (n <= k) {  // under budget: nothing leaves
        for (int i = tid; i < k; i += NT) idx[i] = (i < n) ? i : -1;
        return;
    }
    const int ncand = n - w, nkey = k - w;
    const float* fu = a.score + (size_t)u * a.cap;
    const int j0 = tid * KPT;
    uint32_t key[KPT];
#pragma unroll
    for (int i = 0; i < KPT; ++i) key[i] = (j0 + i < ncand) ? float_key(fu[j0 + i]) : 0u;
    for (int i = tid; i < 4 * 256; i += NT) (&hist[0][0])[i] = 0u;
    __syncthreads();

    // ---- threshold T = the nkey-th largest key, need = how many candidates equal to it survive
    uint32_t T = 0xFFFFFFFFu, need = 0;
    if (nkey > 0) {
        uint32_t prefix = 0, mask = 0, remaining = (uint32_t)nkey;
#pragma unroll
        for (int pass = 0; pass < 4; ++pass) {
            const int shift = 24 - 8 * pass;
#pragma unroll
            for (int i = 0; i < KPT; ++i)
                if (j0 + i < ncand && (key[i] & mask) == prefix) atomicAdd(&hist[pass][(key[i] >> shift) & 255u], 1u);
            __syncthreads();
            // lane owns bins 255-4*lane .. 252-4*lane: highest digits first
            const uint4 h = *(const uint4*)&hist[pass][252 - 4 * lane];
            const uint32_t c[4] = {h.w, h.z, h.y, h.x};
            const uint32_t tot = c[0] + c[1] + c[2] + c[3];
            uint32_t above = wave_scan(tot) - tot;
            uint32_t digit = 0, rem = 0;
            bool mine = false;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if (above < remaining && remaining <= above + c[i]) {
                    digit = (uint32_t)(255 - 4 * lane - i);
                    rem = remaining - above;
                    mine = true;
                }
                above += c[i];
            }
            const unsigned long long owner = __ballot(mine);  // exactly one lane
            const int src = owner ? __ffsll((long long)owner) - 1 : 0;
            prefix |= (uint32_t)__builtin_amdgcn_readlane((int)digit, src) << shift;
            remaining = (uint32_t)__builtin_amdgcn_readlane((int)rem, src);
            mask |= 0xFFu << shift;
        }
        T = prefix;
        need = remaining;
    }

    // ---- stable ranks: survivors above T and candidates equal to it before this thread's slots (16 bits each)
    uint32_t mine = 0;
#pragma unroll
    for (int i = 0; i < KPT; ++i)
        if (j0 + i < ncand && nkey > 0) mine += (key[i] > T ? 1u : 0u) + (key[i] == T ? 0x10000u : 0u);
    const uint32_t upto = wave_scan(mine);
    if (lane == 63) wtot[wv] = upto;
    __syncthreads();
    uint32_t before = upto - mine;
#pragma unroll
    for (int i = 0; i < NW; ++i) before += i < wv ? wtot[i] : 0u;
    uint32_t gt = before & 0xFFFFu, eq = before >> 16;
#pragma unroll
    for (int i = 0; i < KPT; ++i) {
        if (j0 + i < ncand && nkey > 0) {
            const bool above = key[i] > T, same = key[i] == T;
            if (above || (same && eq < need)) {
                const uint32_t dst = gt + min(eq, need);
                if (dst < (uint32_t)nkey) idx[dst] = j0 + i;  // always true; keeps a logic error in bounds
            }
            gt += above ? 1u : 0u;
            eq += same ? 1u : 0u;
        }
    }
    for (int i = tid; i < w; i += NT) idx[nkey + i] = ncand + i;  // the recent window
}

// Units of up to `cap` tokens: two waves' worth of latency per unit matters as little as their number is large, so
// short units take four waves (eight of them fit a CU), longer ones sixteen; beyond 32768 tokens select_kernel.
hipError_t launch_select_list(const SelectArgs& a, int64_t U, hipStream_t stream) {
    const dim3 grid((unsigned)U);
    if (a.cap <= 256 * 8) hipLaunchKernelGGL((select_list_kernel<256, 8>), grid, dim3(256), 0, stream, a);
    else if (a.cap <= 1024 * 8) hipLaunchKernelGGL((select_list_kernel<1024, 8>), grid, dim3(1024), 0, stream, a);
    else if (a.cap <= 1024 * 32) hipLaunchKernelGGL((select_list_kernel<1024, 32>), grid, dim3(1024), 0, stream, a);
    else return launch_select(a, U, stream);
    return hipGetLastError();
}

// Out-of-place compaction: survivor i of unit u (slot idx[u][i] of the source
// cache) goes to slot i of the destination cache.  Source and destination do
// not overlap, so any number of workgroups can share a unit: a workgroup copies
// kGatherRows rows, a lane one 16-byte piece of K or V.
constexpr int kGatherThreads = 256;
constexpr int kGatherRows = 64;

__global__ void __launch_bounds__(kGatherThreads) gather_kernel(const GatherArgs g) {
    const int64_t u = blockIdx.y + (int64_t)blockIdx.z * gridDim.y;
    if (u >= g.units) return;
    const int64_t ud = u + g.dst_unit0;
    const int tid = threadIdx.x;
    const int k = g.k;
    const int32_t* idx = g.idx + (size_t)u * k;
    const int row0 = blockIdx.x * kGatherRows;
    const int PPR = g.row_bytes >> 4;
    const uint4* Ks = (const uint4*)((const char*)g.src_K + (size_t)u * g.src_cap * g.row_bytes);
    const uint4* Vs = (const uint4*)((const char*)g.src_V + (size_t)u * g.src_cap * g.row_bytes);
    uint4* Kd = (uint4*)((char*)g.dst_K + (size_t)ud * g.dst_cap * g.row_bytes);
    uint4* Vd = (uint4*)((char*)g.dst_V + (size_t)ud * g.dst_cap * g.row_bytes);
    const int pieces = kGatherRows * PPR;  // per tensor
    for (int p = tid; p < 2 * pieces; p += kGatherThreads) {
        const int t = p >= pieces, q = t ? p - pieces : p;
        const int i = row0 + q / PPR, piece = q % PPR;
        if (i < k) {
            const int s = idx[i];
            if (s >= 0 && s < g.src_cap) {
                const uint4 v = stream_load((t ? Vs : Ks) + (size_t)s * PPR + piece);
                stream_store((t ? Vd : Kd) + (size_t)i * PPR + piece, v);
            }
        }
    }
    if (tid < kGatherRows) {
        const int i = row0 + tid;
        if (i < k) {
            const int s = idx[i];
            if (s >= 0 && s < g.src_cap) {
                g.dst_score[(size_t)ud * g.dst_cap + i] = g.src_score[(size_t)u * g.src_cap + s];
                g.dst_pos[(size_t)ud * g.dst_cap + i] = g.src_pos[(size_t)u * g.src_cap + s];
            }
        }
    }
    if (blockIdx.x == 0 && tid == 0) g.dst_len[ud] = min(g.src_len[u], k);
}

hipError_t launch_gather(const GatherArgs& g, hipStream_t stream) {
    const unsigned gy = (unsigned)(g.units < 32768 ? g.units : 32768);
    const unsigned gz = (unsigned)((g.units + gy - 1) / gy);
    const dim3 grid((unsigned)((g.k + kGatherRows - 1) / kGatherRows), gy, gz);
    hipLaunchKernelGGL(gather_kernel, grid, dim3(kGatherThreads), 0, stream, g);
    return hipGetLastError();
}

// Beam fork (beam search, one cache per beam): gridDim.x workgroups share the live rows of a destination unit
// and copy them from the parent beam's unit -- a lane one 16-byte piece of K or V at a time, four in flight --
// with their scores and positions.  The parent's row of the batch is only read in this launch (it continues
// itself), so source and destination never meet.  Few, looping workgroups per unit rather than one per 64
// rows: most calls fork few beams or none, and a workgroup that finds nothing to do still costs its launch.
constexpr int kForkDepth = 4;
__global__ void __launch_bounds__(kGatherThreads) fork_kernel(const ForkArgs f) {
    const int64_t u = blockIdx.y + (int64_t)blockIdx.z * gridDim.y;  // destination unit
    const int64_t units = (int64_t)f.L * f.B * f.H;
    if (u >= units) return;
    const int h = (int)(u % f.H), b = (int)((u / f.H) % f.B);
    const int64_t l = u / ((int64_t)f.H * f.B);
    const int pb = f.parent[b];
    if (pb == b) return;
    if (pb < 0 || pb >= f.B || f.parent[pb] != pb) {
        if (blockIdx.x == 0 && threadIdx.x == 0) atomicAdd(f.ws_err, 1);
        return;
    }
    const int64_t us = (l * f.B + pb) * f.H + h;  // source unit
    const int n = min(max(f.len[us], 0), f.cap);
    if (blockIdx.x == 0 && threadIdx.x == 0) f.len[u] = n;
    const int per = (n + (int)gridDim.x - 1) / (int)gridDim.x;
    const int row0 = (int)blockIdx.x * per, row1 = min(n, row0 + per);
    if (row0 >= row1) return;
    const int tid = threadIdx.x;
    const int PPR = f.row_bytes >> 4;
    const size_t so = (size_t)us * f.cap * PPR + (size_t)row0 * PPR, dof = (size_t)u * f.cap * PPR + (size_t)row0 * PPR;
    const int pieces = (row1 - row0) * PPR;  // per tensor; the rows of a slice are contiguous
    for (int p0 = tid; p0 < 2 * pieces; p0 += kForkDepth * kGatherThreads) {
        uint4 v[kForkDepth];
#pragma unroll
        for (int i = 0; i < kForkDepth; ++i) {
            const int p = p0 + i * kGatherThreads;
            v[i] = make_uint4(0u, 0u, 0u, 0u);
            if (p < 2 * pieces) v[i] = stream_load((p >= pieces ? (const uint4*)f.V + so + (p - pieces) : (const uint4*)f.K + so + p));
        }
#pragma unroll
        for (int i = 0; i < kForkDepth; ++i) {
            const int p = p0 + i * kGatherThreads;
            if (p < 2 * pieces) stream_store((p >= pieces ? (uint4*)f.V + dof + (p - pieces) : (uint4*)f.K + dof + p), v[i]);
        }
    }
    for (int r = row0 + tid; r < row1; r += kGatherThreads) {
        f.score[(size_t)u * f.cap + r] = f.score[(size_t)us * f.cap + r];
        f.pos[(size_t)u * f.cap + r] = f.pos[(size_t)us * f.cap + r];
    }
}

hipError_t launch_fork(const ForkArgs& f, hipStream_t stream) {
    const int64_t units = (int64_t)f.L * f.B * f.H;
    const unsigned gy = (unsigned)(units < 32768 ? units : 32768);
    const unsigned gz = (unsigned)((units + gy - 1) / gy);
    // slices per unit: about 64 KB of rows each, at most 16, fewer when the units alone fill the chip
    const int64_t unit_bytes = 2 * (int64_t)f.cap * f.row_bytes;
    int64_t slices = (unit_bytes + 65535) / 65536;
    if (slices > 16) slices = 16;
    while (slices > 1 && units * slices > 4096) slices >>= 1;
    const dim3 grid((unsigned)slices, gy, gz);
    hipLaunchKernelGGL(fork_kernel, grid, dim3(kGatherThreads), 0, stream, f);
    return hipGetLastError();
}

hipError_t launch_select(const SelectArgs& a, int64_t U, hipStream_t stream) {
    const dim3 grid((unsigned)U);
    if (a.presel && !a.presel_done) {
        hipLaunchKernelGGL(presel_kernel, dim3((unsigned)(U * a.presel)), dim3(kPreselThreads), 0, stream, a, U);
        const hipError_t e0 = hipGetLastError();
        if (e0 != hipSuccess) return e0;
    }
    if (a.layout == KF_LAYOUT_SLOT)
        hipLaunchKernelGGL((select_kernel<kSelectThreadsSlot>), grid, dim3(kSelectThreadsSlot), 0, stream, a);
    else
        hipLaunchKernelGGL((select_kernel<kSelectThreads>), grid, dim3(kSelectThreads), 0, stream, a);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess && a.wide) e = launch_shift(a, U, stream);
    return e;
}

// Second launch of the two-launch eviction: every chunk of rows behind the evicted slot moves down by one.
hipError_t launch_shift(const SelectArgs& a, int64_t U, hipStream_t stream) {
    const int nchunks = (a.k + a.chunk_rows - 1) / a.chunk_rows;
    const int lds = U * nchunks <= kShiftLdsMaxWorkgroups || U <= kShiftLdsMaxUnits ? kShiftLds : 0;
    hipLaunchKernelGGL(shift_chunk_kernel, dim3((unsigned)(U * nchunks)), dim3(kWideThreads), lds, stream, a, nchunks, U);
    return hipGetLastError();
}

}  // namespace kf
