// Internal declarations shared by the kernels and the C-ABI layer of the SIDCo library.
#ifndef SIDCO_INTERNAL_H
#define SIDCO_INTERNAL_H

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "sidco.h"

namespace sidco {

constexpr int kBlock = 512;                       // threads per block: 8 wave64
constexpr int kWavesPerBlock = kBlock / 64;
constexpr int kTile = 256;                        // elements per wave step: 64 lanes x float4
constexpr int kGrid = 32;                         // tiles sit on the grid of 128-byte lines of the vector (see WaveTiles)
constexpr int kMaxBlocks = 512;                   // 2 blocks per CU on 256 CUs
constexpr int kMaxWaves = kMaxBlocks * kWavesPerBlock;
// A batch's launch: its vectors share kMaxBlocks blocks' worth of tiles evenly, and each may leave one block
// that is not full, so up to twice as many.
constexpr int kMaxBatch = kMaxBlocks;  // vectors per batch
constexpr int kBatchBlocks = kMaxBlocks + kMaxBatch;
// A non-final stage whose source is still the dense vector writes survivor lists only if the expected
// fraction of the vector that goes into them is at most this; otherwise it only counts and sums, and
// the next stage scans the dense vector again (4 B/element read, against 16 B per list entry written
// + read, writes being the dearer half).
constexpr double kMaterializeBelow = 0.16;
// Default position of a dense stage's candidate threshold between this stage's target ratio and the
// next one's, on the log scale: log(1/ratio_w) = L_m + kSpeculation * L_{m+1}.  At 0.5 the candidate
// lists serve the next stage as long as the mean excess over eta_m is at least about half of what the
// fitted law predicts (a Gaussian tail under an exponential fit still passes).
constexpr double kSpeculation = 0.5;
// A call that repeats the previous call's shape on the device (same d, law and ratios: the next
// training iteration) starts from where the previous call's next threshold really fell on that scale,
// minus this margin, and never above kHintMax: gradients change slowly from one iteration to the
// next, so the candidate lists shrink to a little more than the next stage's exceedances.
constexpr float kHintMargin = 0.1f;
constexpr float kHintMax = 0.95f;
static_assert(kMaxBlocks <= kBlock, "a thread for every producer block, in gather_body and for compact_body's folded sums");

constexpr int kDistExp = SIDCO_DIST_EXP;
constexpr int kDistGamma = SIDCO_DIST_GAMMA_GPD;
constexpr int kDistGpd = SIDCO_DIST_GPD;

constexpr uint32_t kStNonfinite = SIDCO_ST_NONFINITE;
constexpr uint32_t kStVarZero = SIDCO_ST_VAR_ZERO;
constexpr uint32_t kStGammaS = SIDCO_ST_GAMMA_S;
constexpr uint32_t kStGammaClamp = SIDCO_ST_GAMMA_CLAMP;
constexpr uint32_t kStStopped = SIDCO_ST_STOPPED;
constexpr uint32_t kStOverflow = SIDCO_ST_OVERFLOW;
constexpr uint32_t kStFallback = SIDCO_ST_FALLBACK;

// A fitted law as the kernels use it (see Fit in the kernel source), with the location it sits on.
struct FitRecord {
    int gpd;
    float loc;
    double s, c, a, b;
};

constexpr int kBandsNone = 0, kBandsRecord = 1, kBandsUse = 2;
// Bands of a first pass (see k_fit_bands): what it looks for besides the sums of the fit.  Stage m < M: magnitudes in
// (lo[m-1], hi[m-1]] are listed, those above hi[m-1] summed up; the last stage: everything above lo[M-1] is listed.
constexpr int kBandStages = 3;  // calls of 2 and 3 stages
// Widest band, of a stage before the last, that the next call goes by (see bands_record).  In a batch the lists have less
// room (kChunkList), and with 0.15 for the first stage they overflowed on the first call after each rest (66 M elements in 50 tensors, gamma law, 3
// stages, ratio 0.001: every tensor's).
constexpr float kBandMaxWidth = 0.15f, kBandMaxWidthBatch = 0.08f;
struct Bands {
    uint32_t on;  // stages of the calls they are for; 0: the edges mean nothing, the first pass only forms the fit's sums
    float lo[kBandStages], hi[kBandStages];
};

// Calls since the thresholds last jumped, and calls between the two jumps before.  After a jump the next call goes
// without bands (or Top-k's edge); after one that came less than kCalmRun calls behind the one before it so do
// kCalmMost calls: bands that serve two calls and then miss gain nothing.  A training step, us, without bands, with eight
// calls without them after any jump, and so.  Jumps in every 8th call: 25.6 M elements, 3 stages 84.4, 86.5 and 79.3; 40 M,
// ratio 0.01 116.6, 118.7 and 110.8; 100 M 258, 273 and 243; 138 M 515, 535 and 445; 66 M in 50 tensors 187, 190 and 161.
// In every 5th, without and so: 25.6 M 84.6 and 81.6, 40 M 117 and 115, 138 M 515 and 470, 161 tensors 84.2 and 84.3.
constexpr uint32_t kCalmRun = 4, kCalmMost = 8;
struct Calm {
    uint32_t run, last;
};

// Device-resident state of one call.  Stage m's kernel reads the entries stage m-1 wrote and
// writes its own, so no entry is read and written inside one kernel.
struct DevState {
    sidco_diag diag;
    uint32_t status_after[SIDCO_MAX_STAGES + 1];  // status bits accumulated up to and including stage m
    uint32_t frozen_after[SIDCO_MAX_STAGES + 1];  // 1 once an empty exceedance set stopped the refinement
    float list_eta[SIDCO_MAX_STAGES + 1];         // the lists written by stage m's kernel hold every entry above this
    FitRecord cand_fit[SIDCO_MAX_STAGES + 1];     // stage m wrote candidate lists: its fitted law and location
    // Survives from call to call (k_fit does not clear it): where stage m+1's threshold fell between
    // stage m's target ratio and its own, on the log scale of stage m's fitted law; NaN if unknown.
    float theta_seen[SIDCO_MAX_STAGES + 1];
    // Adapt_Stages bookkeeping (Algorithm 1): pairs reported by the calls since the controller last
    // looked, not counting the call in flight; k_fit folds the previous call's count in (or starts over)
    unsigned long long khat_sum;
    long long prev_cap;                           // output capacity of the previous call (clips its count)
    unsigned long long selected_ctr;              // pairs selected by the last stage (cleared by k_fit)
    uint32_t overflow;                            // 1 if selected_ctr exceeded the output capacity
    uint32_t bad_index;                           // sidco_scatter_add met an index outside [0, d) since the last check
    // who made the last call with this state (id of a stage controller, 0 otherwise), and whether a call
    // of someone else fell into the current window of the controller's count
    unsigned long long owner;
    uint32_t disturbed;
    // Bands of the call in flight (copied by its first pass) and of the next one (written by the last stage); whether
    // stage m's threshold, and those before it, fell into their bands; the last call's thresholds and half-widths
    Bands band, band_next;
    uint32_t band_live[kBandStages + 1];
    uint32_t band_over;     // a batch's first pass found more entries for a chunk's list than it has room for, or another's
                            // more than are worth listing
    float band_eta[kBandStages], band_w[kBandStages];
    Calm band_calm;
};

// Rows of kMaxWaves tiles from which on the waves of a first pass change places (see acc_tile).  Shorter vectors gain nothing, and those
// that the caches serve lose (one stage on 8 M 27.8 and 28.4 us).  Calls without it and with it, us: 2 stages 19 M 59.3 and 59.2,
// 25.6 M 74.1 and 73.5, 3 stages 82.1 and 81.5, calls that do not repeat a shape, 25.6 M 83.5 and 82.1, 40 M 122 and 118.7; DGC 19 M
// 77.1 and 76.5, 25.6 M 93.0 and 92.9, 40 M 133 and 129.  A call of one stage reads the vector again at its own places, and 19 M take
// 50.8 and 52.3, 25.6 M 65.9 and 67.1, 40 M 98.3 and 99.8, and longer ones have the flat shape: it never does.  Top-k, whose first pass
// lists as well or is read again, with its scatter: fp32 19 M 66.2 and 67.1, 22.5 M 75.6 and 76.4, 25.6 M 73.1 and 72.2 (the training-step
// case), 33 M, k of a hundredth 134.5 and 131.8, 38 M 154.6 and 149.4, a thousandth 113.2 and 113.3; bf16 25.6 M 73.3 and 74.2, 29 M 80.5
// and 80.6, 38 M, a hundredth 129.0 and 126.6.
constexpr uint32_t kTurnRowsTopk = 24, kTurnRowsTopk16 = 28;
constexpr uint32_t kTurnRows = 18;

// element type of the gradient buffer (the accumulated vector and the residual are always fp32)
constexpr int kGradF32 = 0, kGradF16 = 1, kGradBf16 = 2;

// Kernel arguments: the first three 64-byte lines are what a stage's kernel asks for before its threshold, in the order of
// need.  A line that is not in the scalar cache yet, and after a kernel's start none is, costs 0.2 us and more.
struct Params {
    DevState* st;
    const double* part_in;  // [4][kBatchBlocks] partial sums written by the previous kernel
    const uint32_t* blk_in; // [kMaxBlocks] per-block sums of cnt
    double* band_part;      // [3 * (kBandStages - 1)][kMaxBlocks] sums of y, y^2 and 1 above each band's upper edge
    int stage;              // 1-based stage a k_compact launch works for
    uint32_t nblocks;       // grid size of the kernels that read the dense vector or write partial sums
    int dist;
    uint32_t nwaves;        // waves that own tiles
    uint32_t tq, tr;        // T / nwaves and T % nwaves, T = ceil((d + shift) / kTile) tiles (see WaveTiles)
    float theta;            // > 0: the lists of this kernel are candidate lists (see stage_prologue); else 0
    int use_hint;           // the previous call on the device had this call's shape: theta_seen applies

    int2* band_seg;         // lists of a first pass with bands
    uint32_t* band_cnt;     // [kMaxWaves] their lengths
    const int2* seg_in;     // survivor lists (index, value bits); wave w's list starts at seg_begin(w)
    const uint32_t* cnt_in; // [kMaxWaves] survivor-list lengths written by the previous kernel
    int2* seg_out;
    const float* acc;       // dense working vector read by stage 1's compaction: acc_w, else grad
    uint32_t shift;         // elements between the 128-byte boundary before acc[0] and acc[0] (see WaveTiles)
    uint32_t nfull;         // (d + shift) / kTile: tiles below this index are complete (tile 0 only if shift = 0)
    int reverse;            // a dense stage kernel walks the tiles from the last to the first
    int M;

    double L_stage, L_next; // log(1/delta_m) of the stage and of the next one
    int64_t d;
    float theta_min;        // lowest theta a hint may lead to: below it the lists would exceed kMaterializeBelow
    int cand_stage;         // the stage of this call that wrote candidate lists; 0: none so far
    double* part_out;
    uint32_t* cnt_out;
    uint32_t* blk_out;
    float* residual;        // NULL: memoryless

    const void* grad;       // d elements of type `gt`
    float* acc_w;           // where k_fit stores acc: residual; for a 16-bit gradient without residual a
                            // workspace buffer; NULL when acc is the fp32 gradient itself
    int gt;                 // kGrad*
    uint32_t turn;          // k_fit: the waves change places from row to row (see acc_tile)
    int acc_reset;          // k_fit: start the controller's count of reported pairs over instead of adding to it
    unsigned long long owner;  // id of the stage controller that makes the call, 0 otherwise
    int32_t* out_idx;
    float* out_val;
    int32_t* out_count;
    float* out_eta;
    int64_t out_cap;
    uint32_t* status_out;   // NULL, or a device word that receives the call's status bits as well
    int bands;              // kBands*
    float band_w[kBandStages];  // least half-widths of the bands; the last stage's 0 if it reads no lists
    float band_max;             // and the first one's widest
    double L[SIDCO_MAX_STAGES];  // log(1/delta_m)
};

// ---- exact Top-k comparator (sidco_topk.hip) ----
constexpr int kTopkBins = 2048;  // digit 0 = magnitude bits 30..20; digits 1 and 2 have 1024 bins
// The blocks of k_topk_hist add their histograms of digit 0 to one of this many global copies: few of the 2048 bins
// hold nearly all of a gradient, and same-address atomics of 512 blocks serialise at 11 ns each.  With the sweeps in
// address order (see WaveTiles) and a search in the histogram that takes 3 barriers instead of 20, a call and its
// scatter, us: 1 M elements 35.6 -> 26.7, 4 M 46.1 -> 36.9, 25.6 M 100.7 -> 90.2, 60 M 226.7 -> 182.8; bf16 off the
// line grid 12 M 106.7 -> 64.0, 60 M 380.1 -> 222.3.
constexpr int kTopkCopies = 8;
constexpr int kTopkHist = (kTopkCopies + 2) * kTopkBins;  // words of all digits
constexpr int kTopkLater = 2 * kTopkBins;                 // those of digits 1 and 2

struct TopkState {
    uint32_t prefix[3];            // bin of the k-th largest key in digit 0, 1, 2
    uint32_t k_rem[3];             // rank of that key inside the bin (k_rem[2] = ties still needed)
    uint32_t kth_key;              // the k-th largest magnitude as its bit pattern
    uint32_t k_eff;                // k when the device decides it (TopkParams::k_from_state)
    unsigned long long gt_ctr;     // output places reserved for entries above the k-th key
    unsigned long long eq_ctr;     // entries equal to the k-th key seen so far
    // Survive from call to call: the first pass lists the entries whose key is `edge` or more (of this call; the next one;
    // kNoEdge: none); the last k-th magnitude, and the share that the next one may fall below it
    uint32_t edge, edge_next;
    float last_kth, margin;
    Calm calm;
};
constexpr uint32_t kNoEdge = 0xffffffffu;

struct TopkParams {
    const void* grad;       // d elements of type `gt`
    int gt;                 // kGrad*
    float* residual;        // NULL: memoryless
    float* acc_w;           // where the first kernel stores acc: residual; a workspace buffer for a 16-bit gradient
                            // without residual; NULL when acc is the fp32 gradient itself
    const float* acc;       // acc_w, else grad
    int64_t d;
    int64_t k;
    int k_from_state;       // the last kernel takes k from st->k_eff (may be 0) instead of `k`
    uint32_t clear0;        // words of hist0 that the last kernel clears for the next call
    int bands;              // kBands*: whether the call leaves an edge for the next one, and whether it has one itself
    uint32_t shift, nfull, nwaves, tq, tr, nblocks, turn;  // see Params
    uint32_t* hist0;        // [kTopkCopies][kTopkBins]
    uint32_t* hist1;        // [1024]
    uint32_t* hist2;        // [1024]
    TopkState* st;
    uint32_t* cnt;          // [kMaxWaves] list lengths
    int2* seg;              // per-wave lists
    int32_t* out_idx;
    float* out_val;
    int32_t* out_count;
    float* out_kth;
};

void launch_topk_zero(const TopkParams& p, hipStream_t s);
void launch_topk_hist(const TopkParams& p, hipStream_t s);
void launch_topk_compact(const TopkParams& p, hipStream_t s);
void launch_topk_refine(const TopkParams& p, uint32_t grid, hipStream_t s);
void launch_topk_final(const TopkParams& p, uint32_t grid, hipStream_t s);

// ---- DGC comparator: threshold from a radix select on a random subset, first pass over the vector,
// second radix select on the first pass's entries ----
struct DgcState {
    TopkState sample;               // select of the k_s-th largest magnitude of the subset
    TopkState lists;                // select among the entries of the first pass
    unsigned long long first_pass;  // entries above the subset's threshold
    float eta;                      // that threshold
    float kth;                      // smallest magnitude that stayed
};

struct DgcParams {
    const void* grad; // d elements of type `gt`
    int gt;           // kGrad*
    float* residual;  // NULL: memoryless
    float* acc_w;     // where the dense pass stores acc: residual, or nowhere
    int64_t d;
    int64_t k;        // target number of entries
    uint32_t shift, nfull, nwaves, tq, tr, nblocks, turn;  // see Params
    uint64_t seed;
    uint32_t n_s, k_s;  // subset size, rank of the threshold in it
    uint32_t* keys;     // [n_s] magnitude keys of the subset
    uint32_t* hist_s;   // [3][kTopkBins] digit histograms of the subset
    uint32_t* hist_l;   // [3][kTopkBins] digit histograms of the first pass's entries
    DgcState* st;
    uint32_t* cnt;      // [kMaxWaves] list lengths
    int2* seg;          // per-wave lists
    float* out_eta;
};

void launch_dgc_zero(const DgcParams& p, hipStream_t s);
void launch_dgc_sample(const DgcParams& p, hipStream_t s);
void launch_dgc_digit(const DgcParams& p, int digit, hipStream_t s);
void launch_dgc_dense(const DgcParams& p, hipStream_t s);
void launch_dgc_lists(const DgcParams& p, uint32_t grid, hipStream_t s);

// A block's place in its vector's grid (the whole launch for a single call, a slice of it in a batch).
struct Blk {
    uint32_t id;  // block index within the vector's grid
    uint32_t n;   // size of that grid
    uint32_t none;  // 0 (see stage_grid)
    bool records;   // the block that keeps what the vector's call leaves in its state
};

// ---- batched calls: several vectors (the tensors of one flat buffer) in one launch sequence ----
// One vector of a batch, relative to the call's base pointers (so that the table on the device depends on
// the layout alone and survives a change of buffers).
struct TensorDesc {
    int64_t offset;         // first element in grad / residual
    int64_t d;
    int64_t out_offset;     // first pair in out_idx / out_val
    int64_t out_cap;
    uint64_t seg_off;       // first slot of the vector in the survivor-list buffers
    uint32_t first_block;   // the vector's blocks in the dense grids: [first_block, first_block + nblocks)
    uint32_t nblocks;
    uint32_t first_final;   // ... and in the last stage's grid
    uint32_t nfinal;
    uint32_t index;         // position in out_counts / out_etas
    uint32_t nwaves;        // waves that own tiles of the vector
    uint32_t tq, tr;        // T / nwaves and T % nwaves, T the tiles at any alignment of the buffers (see max_tiles)
};

struct BatchTable {
    DevState st[kMaxBatch];
    TensorDesc desc[kMaxBatch];
    uint16_t map[kBatchBlocks];   // block of a dense grid -> vector
    uint16_t fmap[kBatchBlocks];  // block of the last stage's grid -> vector
};

// Kernel arguments of a batched launch (by value): what all vectors share.
struct BatchArgs {
    BatchTable* tb;
    const void* grad;       // base pointers of the call; the gradient's elements are of type `gt`
    int gt;                 // kGrad*
    float* residual;
    float* acc_own;         // workspace copy of acc for a 16-bit gradient without residual, else NULL
    int32_t* out_idx;
    float* out_val;
    int32_t* out_counts;
    float* out_etas;
    double* part[2];
    uint32_t* cnt[2];
    uint32_t* blk[2];
    int2* seg[2];
    int in, out;            // which half of the double buffers the kernel reads / writes
    int dist, M, stage, reverse;
    double L[SIDCO_MAX_STAGES];
    double L_stage, L_next;
    float theta, theta_min;
    int use_hint, cand_stage;
    double* flat;           // partial sums of a flat first pass (see k_fit_flat_batched), chunks per block and blocks
    uint32_t flat_gx, flat_blocks;
    int pieces;             // k_fit_flat_batched: whether blocks go by piece_order
    int bands;              // as in Params, and if used: lengths of the chunks' lists, and the lists, kChunkList entries each
    float band_w[kBandStages];
    uint32_t* chunk_cnt;
    int2* chunk_list;
};
// Room in a chunk's list: an eighth of its entries.  A stage's wave that takes the lists of its share of a block's chunks
// never has more entries than the elements its own list has room for: of a block with n <= 8 waves of at most q + 1 and at
// least q >= 1 tiles, chunks of 8 tiles shared out over the n, that is ceil((q + 1) / 8) lists of one tile's length.
constexpr uint32_t kChunkList = kTile;

void launch_fit_batched(const BatchArgs& a, bool ec, uint32_t blocks, uint32_t flat_gx, bool fold, hipStream_t s);
void launch_compact_batched(const BatchArgs& a, bool stats, bool write, bool flat, bool keep, uint32_t blocks, hipStream_t s);
void launch_lists_batched(const BatchArgs& a, uint32_t blocks, hipStream_t s);
void launch_final_lists_batched(const BatchArgs& a, uint32_t final_blocks, hipStream_t s);
void launch_gather_batched(const BatchArgs& a, uint32_t blocks, hipStream_t s);

void launch_clear_u32(uint32_t* p, hipStream_t s);
void launch_scatter_add(float* dense, int64_t d, const int32_t* idx, const float* val, const int32_t* count,
                        int64_t capacity, float scale, uint32_t* bad, hipStream_t s);
// k_fit's shape for large vectors (see k_fit_flat): one float4 per thread, 256-thread blocks.  Waves that walk
// interleaved tiles drift apart, the more the longer they run, and the window of addresses widens with them; the
// flat shape's blocks start in address order, but it needs a kernel that folds its partial sums.  A two-stage call
// in the per-wave shape and in the flat one, us: 25.6 M elements 84.3 and 87.5, 41 M 111.2 and 113.7, 50 M 133.2
// and 135.0, 58 M 154.2 and 155.1, 62 M 164.5 and 161.2, 80 M 217.0 and 205.7; with a bf16 gradient 50 M 120.1 and
// 126.8, 62 M 148.7 and 150.8, 80 M 193.3 and 191.2; one stage, with both shapes' tiles in pieces (acc_tile, piece_order), 40 M
// 100.7 and 101.2, 50 M 123.9 and 123.8, 58 M 147.7 and 146.9, 66 M 164.9 and 163.0, 80 M 202.5 and 197.5.  The shapes meet between 58 and 62 M with fp32 gradients and
// between 62 and 80 M with 16-bit ones, which share the line: it costs them at most 1.4 % of a call around 62 M.
constexpr int kFlatBlock = 256;
constexpr int kFlatTiles = 2;                                // tiles per wave of a batch's flat first pass
constexpr uint32_t kFlatChunk = kFlatBlock / 64 * kFlatTiles;  // and per block
constexpr int64_t kFlatMinD = 58000000;
// That line for calls that clear much of the residual (see keeps_much), us per wave and flat: 2 stages, 50 M elements,
// ratio 0.08 308 and 302, 0.1 321 and 315; 40 M, 0.1 263 and 260; 25 M, 0.1 169 and 167; 15 M, 0.1 100.9 and 101.2;
// 1 stage, 15 M, 0.1 89.4 and 91.2.
constexpr int64_t kFlatMinMuch = 20000000;
// A batch's waves walk the tiles of their own vector, so that its window is as many as it has vectors, and the flat
// shape pays earlier: 25.6 M elements in 161 tensors 96.6 us per wave and 90.6 flat, 66 M in 50 tensors 236.6 and 204.
constexpr int64_t kFlatMinBatch = 12000000;
// From this length on the blocks of that shape go by piece_order; shorter batches with many tensors, of whose chunks some are
// empty, lose by it.  A call in address order and so, us: 66 M elements in 50 tensors 145.4 and 143.2, in 20 of 64 elements
// up 150.7 and 148.5, in 300 208.4 and 206.2, in 161 of 64 elements up 151.8 and 151.7; 40 M in 50 99.3 and 98.8, in 100 of 64
// up 100.5 and 101.7; 25.6 M in 161 72.6 and 75.5, in 50 70.5 and 70.5; 14 M in 20 50.0 and 51.0.
constexpr int64_t kPiecesMinBatch = 60000000;
// A batch whose longest vector has at most this many flat partial sums leaves them to the prologue of the first
// stage's kernel, 4 loads per thread and quantity; beyond it a kernel folds them first, 4.8 us against 1 to 2.5 in that
// prologue: 161 tensors, 25.6 M elements 83.5 -> 81.6 us, 200 tensors, 14 M 49.0 -> 47.0.
constexpr uint32_t kFlatDirect = 4 * kBlock;
inline bool fit_uses_flat(int64_t d, bool much) { return d >= (much ? kFlatMinMuch : kFlatMinD); }
inline uint32_t fit_flat_blocks(int64_t d, uint32_t shift)
{
    return (uint32_t)(((d + shift + 3) / 4 + kFlatBlock - 1) / kFlatBlock);
}
// k_small's block, its threads that hold data, the longest vector that goes through it, and the pairs that a data wave's
// list has room for with N float4s per lane: all and a step of the wave more, or what 150 of the 160 KB of LDS hold.  A
// training step's call and its scatter, one kernel against the kernels of a longer vector, us: 12000 elements 13.3 and 18.2
// (the host's launches), with three stages 20.6; 36864, one stage 13.8 and 20.2, three 18.1 to 19.7 and 23.5; 36864, two stages, ratio
// 0.1 17.5 and 20.3; the gamma law there, of which it keeps 31 %, 23.1 and 21.5.
constexpr int kSmallBlock = 1024, kSmallWaves = kSmallBlock / 64, kSmallData = kSmallBlock - 64;
constexpr int kSmallMaxD = 36864;
template <int N>
constexpr uint32_t kSmallList = 256 * N + 64 < 1280 ? 256 * N + 64 : 1280;
void launch_small(const Params& p, hipStream_t s);
void launch_fit(const Params& p, bool flat, double* scratch, hipStream_t s);
// A call that repeats a shape but has no bands (its thresholds jump) sweeps past the caches from this length on.  A training
// step of that kind with ordinary accesses and past the caches, us: 100 M elements, 2 stages 276 and 284, 120 M 339 and 342,
// 138 M, 3 stages, ratio 0.01 559 and 541, 0.1 965 and 943.
constexpr int64_t kBandPastMinD = 130000000;
void launch_fit_bands(const Params& p, hipStream_t s);
void launch_compact(const Params& p, bool stats, bool write, bool keep, hipStream_t s);
void launch_lists(const Params& p, hipStream_t s);
void launch_final_lists(const Params& p, uint32_t grid_blocks, hipStream_t s);
constexpr int kSelectBlock = 256, kSelectTiles = 16;  // k_select's block, and its tiles per wave
void launch_select(const Params& p, bool keep, hipStream_t s);
void launch_gather(const Params& p, hipStream_t s);

}  // namespace sidco
#endif
