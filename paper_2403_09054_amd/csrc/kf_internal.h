// Host-side declarations shared by the API layer and the kernel files.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "../../include/keyformer.h"

namespace kf {

// ------------------------------------------------------------------ decode
struct DecodeArgs {
    void* K;
    void* V;
    float* score;
    int32_t* pos;
    int32_t* len;
    const void* q;
    const void* k_new;
    const void* v_new;
    float* out;
    const uint64_t* seeds;
    const float* slopes;
    float* ws_part;    // [U][S][G][D+4] partial outputs and softmax statistics of each split and query head
    float* ws_e;       // [U][G][cap]    un-normalised score increments of each token
    int32_t* ws_err;   // [1]         skipped-unit counter
    int32_t* ws_m;     // [U]         tokens this launch scored in each unit (0: skipped); written when split or shared
    int32_t B, H, cap, layer0;
    int32_t G;         // query heads per cached head (q and out hold H*G heads)
    int32_t S;         // splits of a unit's token range
    int32_t chunk;     // tokens per split
    int32_t q_pos;
    int32_t noise;
    int32_t new_pos;   // position bias from slot indices instead of original positions
    int32_t shared;    // one score for all layers: leave the normalised increments in ws_e, do not touch score
    // Step taken from device memory (non-NULL `step`): t = *step, q_pos = n0 + t - 1,
    // tau = tau_init + min(t, T)*dtau; q_pos and inv_tau above are then ignored.
    const int32_t* step;
    int32_t n0, T;
    float tau_init, dtau;
    // Per-sequence query position / temperature (either may be NULL): [B], override the above.
    const int32_t* seq_q_pos;
    const float* seq_tau;
    // Whole step in this launch (single split): after the scores are updated the workgroup
    // evicts for its unit.  Slot layout: it stores the new token straight into the freed slot.  fuse_k = 0: off.
    int32_t fuse_k, fuse_w;
    int32_t fuse_ordered;  // ordered layout (a few small units, cap == k + 1): it moves the rows behind the evicted slot down itself
    int32_t* fuse_idx;  // NULL, or [U][k] survivor list as the selection kernel writes it
    int32_t* step_inc;   // NULL, or the device step counter the launch's last workgroup advances (whole-step launch)
    int32_t* ws_ticket;  // [1] workgroups of this launch that are done (zero between launches)
    // Fused step of few, long units: the merge launch (pre_slices workgroups per unit) also leaves, per
    // workgroup, the smallest eviction candidate among the tokens it updated -- what the selection's own
    // candidate scan launch would compute from the finished scores.  pre_slices = 0: off.
    int32_t pre_slices, pre_k, pre_w, pre_layout;
    unsigned long long* pre_min;  // [U][pre_slices] (score key, tie-break) pack, ~0 if the slice has no candidate
    int32_t* pre_slot;            // [U][pre_slices] its slot
    int32_t keep_w;  // the last keep_w rows of a unit are loaded into the caches: the step's eviction moves them; 0: none
    float inv_tau;
    float scale;
    // Small launch (FEW form of the decode kernel).  With few_f the splits also leave copies of what the
    // eviction launch overwrites while its other workgroups still read it.
    int32_t few;
    int32_t few_rows;   // R: slots per workgroup of the eviction launch
    int32_t few_nb;     // boundary slots kept per unit
    float* few_f;       // NULL, or [U][cap]: the scores before this step
    void* few_brow;     // [U][few_nb][2][row_bytes] K and V rows at slots R, 2R, ...
    int32_t* few_bpos;  // [U][few_nb] their positions
};
constexpr int32_t kFuseOrderedBytes = 64 * 1024;  // of K, and as much of V, that the workgroup of a unit moves itself

// Limits of the FEW form: tokens per split (old scores and boundary rows are held in registers) and splits.  The ordered
// step at other values, up to 130 shapes each, of the speed at these: 256 workgroups 0.75 to 1.09, 1024 0.80 to 1.08
// (1.24 where only they bring a split below its limit), 32 KB 0.75 to 0.92, 128 KB 0.96 to 1.05 (1.21 likewise), 64 rows
// with 4 or 8 heads 0.75 to 0.94, 256 rows 0.88 to 1.15, 32 splits 0.87 to 1.08.
constexpr int32_t kFewTokens = 2;    // per thread of 256
constexpr int32_t kFewPieces = 2;    // 16-byte pieces of boundary rows per thread
constexpr int32_t kFewMaxChunk = 512;
constexpr int32_t kFewMaxChunkGrouped = 128;     // with 4 or 8 query heads
constexpr int32_t kFewChunkBytes = 64 * 1024;    // of K, and as much of V
constexpr int32_t kFewWorkgroups = 512;          // splits of all units together
constexpr int32_t kFewMaxSplits = 64;            // of a unit, times its query heads
constexpr int32_t kFewMaxRowPieces = 32;         // 16-byte pieces of the longest row
constexpr int32_t kWideChunkBytes = 32 * 1024;   // see wide_chunk_rows

// Launch shape of the decode kernel for U units of up to m tokens.
struct DecodePlan {
    int32_t S, chunk;
    size_t lds_bytes;
};
DecodePlan plan_decode(int64_t U, int32_t m, int32_t d, int32_t dtype, int32_t G);
bool plan_decode_few(int64_t U, int32_t m, int32_t d, int32_t dtype, int32_t G, DecodePlan* plan);
int32_t few_max_splits(int64_t U, int32_t G);  // of any m
hipError_t launch_decode(const DecodeArgs& a, int64_t U, int32_t d, int32_t dtype, size_t lds_bytes,
                         hipStream_t stream);
// Workgroups per unit of the merge launch that follows a split decode launch.
int32_t decode_merge_slices(int32_t S, int32_t chunk);

// Shared score function: adds up the layers' contributions and gives every layer the same score.
//   inc != NULL (decode): score[l][bh][j] += sum_l' inc[l'][bh][j] for the m[.][bh] tokens just scored
//   inc == NULL (prompt): score[l][bh][j]  = sum_l' score[l'][bh][j] for j < n
struct ShareArgs {
    float* score;
    const float* inc;
    const int32_t* m;   // decode: [L][BH] tokens scored per unit;  prompt: the caches' len
    int32_t* ws_err;
    int32_t L, BH, cap;
    int32_t inc_unit;   // floats between the increments of consecutive units (G*cap)
};
hipError_t launch_share(const ShareArgs& a, hipStream_t stream);

// ------------------------------------------------------------------ select
struct SelectArgs {
    void* K;
    void* V;
    float* score;
    int32_t* pos;
    int32_t* len;
    int32_t* idx;       // [U][k] source slot of every survivor (caller's kept_idx or workspace)
    int32_t cap, k, w;
    int32_t row_bytes;  // d * sizeof(element)
    int32_t idx_is_output;  // idx is the caller's kept_idx (must be complete), not scratch
    int32_t layout;         // kf_layout
    int32_t move;           // 0: only write the survivor index list (rows are gathered elsewhere)
    int32_t* ws_err;        // [1] skipped-unit counter
    int32_t* step_inc;      // NULL, or the device step counter this launch advances by one when it is done
    // Ordered layout, decode shape, rows moved by a second launch of several workgroups per unit
    // ("wide"): the selection launch only finds the evicted slot and saves the chunk-boundary entries.
    int32_t wide;           // 0: the selection workgroup moves the rows itself
    int32_t chunk_rows;     // R: rows a workgroup of the second launch moves
    int32_t nb;             // boundary slots kept per unit: cap / R
    int32_t* ws_evict;      // [U]                  evicted slot, or -1 (nothing for the second launch)
    void* ws_brow;          // [U][nb][2][row_bytes] K and V rows at slots R, 2R, ... saved before anything moves
    float* ws_bscore;       // [U][nb]              their scores
    int32_t* ws_bpos;       // [U][nb]              their positions
    // Long units in the decode shape: a launch ahead of the selection cuts the candidate scan of a unit
    // into `presel` slices, one workgroup each, and leaves every slice's smallest candidate here.
    int32_t presel;             // 0: the selection workgroup scans the candidates itself
    int32_t presel_done;        // the slices' minima are there already (left by the decode merge launch)
    unsigned long long* ws_pmin;  // [U][presel] smallest (score key, tie-break) pack of the slice, ~0 if none
    int32_t* ws_pslot;          // [U][presel] its slot
    int32_t rest;               // launch_step_finish: units not exactly one token over the budget are left to launch_step_rest
};
constexpr int32_t kPreselMaxSlices = 16;
// rows per workgroup of the wide shift: 2048 16-byte pieces per tensor, i.e. 32 KB of K and 32 KB of V
inline int32_t wide_chunk_rows(int32_t row_bytes) { return kWideChunkBytes / row_bytes; }
hipError_t launch_select(const SelectArgs& a, int64_t U, hipStream_t stream);
// the survivor lists alone (a.move == 0)
hipError_t launch_select_list(const SelectArgs& a, int64_t U, hipStream_t stream);
struct GatherArgs {
    const void* src_K;
    const void* src_V;
    const float* src_score;
    const int32_t* src_pos;
    const int32_t* src_len;
    void* dst_K;
    void* dst_V;
    float* dst_score;
    int32_t* dst_pos;
    int32_t* dst_len;
    const int32_t* idx;  // [units][k] survivor slots in the source
    int64_t units;       // units of the source cache
    int64_t dst_unit0;   // first destination unit (dst_layer0 * B * H)
    int32_t src_cap, dst_cap, k, row_bytes;
};
hipError_t launch_gather(const GatherArgs& g, hipStream_t stream);

// Beam fork: row b of the batch takes over the state of row parent[b] (see kf_beam_fork).
struct ForkArgs {
    void* K;
    void* V;
    float* score;
    int32_t* pos;
    int32_t* len;
    const int32_t* parent;  // [B]
    int32_t* ws_err;
    int32_t L, B, H, cap, row_bytes;
};
hipError_t launch_fork(const ForkArgs& f, hipStream_t stream);
// decode merge + select + compact of every unit in one launch (after the split kernel of a fused step)
hipError_t launch_step_tail(const DecodeArgs& d, const SelectArgs& a, int64_t U, int32_t hd, hipStream_t stream);
// merge + selection + compaction of a small launch, several workgroups per unit (after a FEW split launch with few_f)
constexpr int32_t kFinishMaxTokens = 4096;
hipError_t launch_step_finish(const DecodeArgs& d, const SelectArgs& a, int64_t U, int32_t hd, hipStream_t stream);
// selection and compaction of the units that launch_step_finish left with a.rest set
hipError_t launch_step_rest(const DecodeArgs& d, const SelectArgs& a, int64_t U, hipStream_t stream);
// the row-shifting launch of the two-launch eviction (after a selection launch that ran with a.wide set)
hipError_t launch_shift(const SelectArgs& a, int64_t U, hipStream_t stream);
// the split kernel alone (no merge launch): first half of a fused step
hipError_t launch_decode_split(const DecodeArgs& a, int64_t U, int32_t d, int32_t dtype, size_t lds_bytes,
                               hipStream_t stream);

// ------------------------------------------------------------------ prefill
struct PrefillArgs {
    const void* Q;
    const void* K;
    float* score;
    int32_t* pos;
    int32_t* len;
    const uint64_t* seeds;
    const float* slopes;
    const int32_t* seq_n;  // [B] per-sequence prompt length, or null: every sequence has n rows
    int32_t* ws_err;       // device error counter
    float* ws_c;        // [U][n_pad] per-row log2 normaliser            (U = L*B*H query units)
    uint32_t* ws_r;     // [U][n_pad] per-row noise key
    float* ws_f;        // [U][parts][n_pad] column sums per query head and part (G > 1 or parts > 1 only)
    float2* ws_part;    // [U][parts][n_pad] reference exponent and sum of a row's parts (parts > 1 only)
    float* ws_kn;       // NULL, or [U/G][n_pad/32] largest key norm of a tile: far tiles are left out with a position bias
    float4* ws_tile;    // [U][n_pad/32] bounds of a tile's query rows (with ws_kn)
    int32_t B, H, cap, layer0, n, n_pad;  // H counts QUERY heads; the caches hold H/G heads
    int32_t G;          // query heads per cached head
    int32_t parts;      // workgroups that share the tile walk of a 128-row block, at most ...
    int32_t part_tiles; // ... and the tiles each of them walks
    int32_t noise;
    float inv_tau;
    float scale;
};
// Parts of the blocks' tile walks for U query units of up to n rows.
constexpr int32_t kPrefillMaxPartTiles = 64;
constexpr int32_t kPrefillMaxParts = 32;  // bounds the scratch: 12 bytes per row and part
constexpr int64_t kPrefillPartsRowLimit = 2 * 1024 * 128;  // U * n from which no prompt is cut
constexpr int32_t kPrefillPartsMaxRows = 144 * 128;        // n above which none is
static_assert(kPrefillPartsMaxRows / 32 <= kPrefillMaxParts * kPrefillMaxPartTiles, "the longest cut walk fits the most parts");
struct PrefillParts {
    int32_t parts, tiles;
};
constexpr PrefillParts kPrefillWhole{1, 1 << 26};
PrefillParts plan_prefill(int64_t U, int32_t n);
hipError_t launch_prefill(const PrefillArgs& a, int64_t U, int32_t d, int32_t dtype, hipStream_t stream);

// Prompts with a position bias whose far tiles are looked for (see kf_prefill.hip): the search takes a launch and a trip to
// memory ahead of each walk.  Slopes 2^(-8h/H), d = 128, against walks over all tiles: 32 x 2048 rows 1.07 to 1.1 times as
// fast, 16 x 4096 1.2, 128 x 1300 1.06, 32 x 4096 1.3, 256 x 2048 1.27 to 1.3, 128 x 4096 1.5; below these limits 32 x 1300
// 0.96, 8 x 4096 0.94 to 0.98, 128 x 1000 0.98 to 1.  Slopes too flat for anything to be left out cost 0.5 % at 256 x 2048
// and 3 % (a launch) at 32 x 2048.
constexpr int32_t kPrefillSkipMinRows = 1025;
constexpr int64_t kPrefillSkipMinAllRows = 65536;
constexpr int32_t kPrefillRowPad = 128;  // n is padded to this for the row-statistics arrays

// Prompts whose logits are evaluated once (kf_strips.hip): Gumbel adjustment.
constexpr int32_t kStripSmallRows = 1024;  // up to here workgroups of 4 waves
constexpr int32_t kStripMaxRows = 2048;
// Workgroups per query unit (their column sums take as many floats a row, ws_f; one alone of an ungrouped head writes the
// score itself), or 0: not this way.
int32_t plan_strips(int64_t U, int32_t n, int32_t d, int32_t dtype, bool bias);
hipError_t launch_strips(const PrefillArgs& a, int64_t U, int32_t d, int32_t dtype, hipStream_t stream);

}  // namespace kf
