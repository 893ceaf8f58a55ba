// Exact Top-k by magnitude on MI355X (gfx950): the comparator the paper measures its threshold
// estimators against (arXiv 2101.10761, Sec. 1: Top-k keeps the k entries of largest magnitude and is
// found on a GPU by a radix select that reads the vector once per digit; footnote of Sec. 2.3: the
// threshold operator C_eta equals Top-k at k = khat).
//
// Radix select on the 31 magnitude bits of the fp32 values (|x| as an unsigned integer orders like |x|
// itself; NaN patterns lie above infinity and therefore count as the largest entries), most
// significant digit first, digits of 11 + 10 + 10 bits.  Only the first digit needs the whole vector:
//
//   k_topk_zero      clears the histograms of digit 0, for a workspace's first call: the last kernel of a call leaves
//                    them clear, and the first one clears what only later kernels use
//   k_topk_hist      acc = g + residual (App. B.2), stored back; histogram of digit 0 of |acc|
//                    (per-block histogram in LDS, merged into the global one with atomics on 2048
//                    distinct addresses)                                         [12 B / element]
//                    A call that repeats a shape also lists the entries above an edge under the last k-th key
//   k_topk_compact   prologue: every block finds the digit-0 bin b0 that holds the k-th largest key
//                    (suffix sums of the histogram).  Body: entries with digit 0 >= b0 go to per-wave
//                    lists; those with digit 0 == b0 are binned by digit 1       [4 B / element]
//   k_topk_refine    prologue: bin b1 of digit 1; body (lists only): digit-2 histogram of the entries
//                    that match b0 and b1
//   k_topk_final     prologue: bin b2, i.e. the exact k-th largest key kappa and the number of entries
//                    equal to it that are still needed.  Body (lists only): entries above kappa and
//                    the needed number of entries equal to kappa go to the output; residual update.
//
// The k-th largest magnitude, the set of selected entries above it and every value are deterministic.
// Which of the entries that EQUAL the k-th largest magnitude complete the set is decided by the
// order in which blocks reserve their share and may differ between runs.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "sidco_internal.h"
#include "sidco_device.h"
#include "sidco_select.h"

namespace sidco {

__global__ __launch_bounds__(kBlock) void k_topk_zero(TopkParams p)
{
    const uint32_t i = blockIdx.x * kBlock + threadIdx.x;
    if (i < (uint32_t)(kTopkHist - kTopkLater)) p.hist0[i] = 0;
}

// ---------------------------------------------------------------------------------------------
// k_topk_hist: error-compensation add + digit-0 histogram
// ---------------------------------------------------------------------------------------------
struct DigitHist {
    uint32_t* sh_hist;
    __device__ __forceinline__ void tile(f4 c, uint32_t)
    {
        atomicAdd(&sh_hist[mag_key(c.x) >> 20], 1u);
        atomicAdd(&sh_hist[mag_key(c.y) >> 20], 1u);
        atomicAdd(&sh_hist[mag_key(c.z) >> 20], 1u);
        atomicAdd(&sh_hist[mag_key(c.w) >> 20], 1u);
    }
    __device__ __forceinline__ void one(bool valid, float c, int64_t)
    {
        if (valid) atomicAdd(&sh_hist[mag_key(c) >> 20], 1u);
    }
    __device__ __forceinline__ void end() {}
};

// The same behind a call of the same shape: also lists the entries at or above the edge that call left.
struct DigitHistLists {
    DigitHist h;
    ListWriter lw;
    uint32_t edge;
    int lane;
    uint32_t shift;
    __device__ __forceinline__ void tile(f4 c, uint32_t t)
    {
        h.tile(c, t);
        const int32_t i0 = (int32_t)(t * kTile + lane * 4 - shift);
#pragma unroll
        for (int j = 0; j < 4; ++j) list_push(lw, mag_key(c[j]) >= edge, i0 + j, c[j], lane);
        list_flush(lw, lane);
    }
    __device__ __forceinline__ void one(bool valid, float c, int64_t i)
    {
        h.one(valid, c, i);
        list_push(lw, valid && mag_key(c) >= edge, (int32_t)i, c, lane);
    }
    __device__ __forceinline__ void end() { list_flush(lw, lane); }
};

// BANDS: behind a call of the same shape (see k_topk_compact); the residual goes past the caches then, as nothing reads
// the vector again if the k-th magnitude falls where it is expected.
template <bool EC, int GT, bool BANDS>
__global__ __launch_bounds__(kBlock) void k_topk_hist(TopkParams p)
{
    // a 16-bit gradient is widened as it is read, and acc is always stored then (every later kernel reads fp32)
    constexpr bool WRITE = EC || GT != kGradF32;
    __shared__ uint32_t sh_hist[kTopkBins];
    for (int i = threadIdx.x; i < kTopkBins; i += kBlock) sh_hist[i] = 0;
    AccTile first;
    uint32_t edge = kNoEdge;
    if constexpr (BANDS) {
        first = acc_first<EC, WRITE, GT, EC>(p, blockIdx.x * kWavesPerBlock + (threadIdx.x >> 6), threadIdx.x & 63);
        edge = __builtin_amdgcn_readfirstlane(p.st->edge_next);
    }
    if (blockIdx.x == 0) {
        for (int i = threadIdx.x; i < kTopkLater; i += kBlock) p.hist1[i] = 0;  // digits 1 and 2, one piece
        if (threadIdx.x == 0) {
            p.st->gt_ctr = 0;
            p.st->eq_ctr = 0;
            p.st->prefix[0] = p.st->prefix[1] = p.st->prefix[2] = 0;
            p.st->k_rem[0] = p.st->k_rem[1] = p.st->k_rem[2] = 0;
            p.st->kth_key = 0;
            p.st->k_eff = 0;
            p.st->edge = edge;
        }
    }
    __syncthreads();
    const uint32_t w = blockIdx.x * kWavesPerBlock + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    DigitHist h{sh_hist};
    if constexpr (BANDS) {
        __shared__ int2 ring[kWavesPerBlock][kRingSize];
        if (edge != kNoEdge) {
            DigitHistLists v;
            v.h = h;
            v.lw.list = p.seg + seg_begin(p, w < p.nwaves ? w : 0);
            v.lw.ring = ring[threadIdx.x >> 6];
            v.lw.run = v.lw.fill = 0;
            v.edge = edge;
            v.lane = lane;
            v.shift = p.shift;
            if (w < p.nwaves) {
                acc_sweep<EC, WRITE, GT, EC>(p, w, lane, v, &first);
                const uint32_t n = list_finish(v.lw, lane);
                if (lane == 0) p.cnt[w] = n;
            }
        } else if (w < p.nwaves) {
            acc_sweep<EC, WRITE, GT>(p, w, lane, h, &first);
        }
    } else if (w < p.nwaves) {
        acc_sweep<EC, WRITE, GT>(p, w, lane, h);
    }
    __syncthreads();
    merge_hist(sh_hist, p.hist0 + (blockIdx.x % kTopkCopies) * kTopkBins, kTopkBins);
}

// ---------------------------------------------------------------------------------------------
// k_topk_compact: dense pass.  Entries whose digit 0 is at least b0 go to the wave's list; digit-1
// histogram of those whose digit 0 equals b0.
// ---------------------------------------------------------------------------------------------
__device__ __forceinline__ void topk_emit(bool valid, float x, int32_t idx, uint32_t b0, ListWriter& lw, int lane,
                                          uint32_t* sh_hist)
{
    const uint32_t key = mag_key(x);
    const uint32_t d0 = key >> 20;
    list_push(lw, valid && d0 >= b0, idx, x, lane);
    if (valid && d0 == b0) atomicAdd(&sh_hist[(key >> 10) & 1023u], 1u);
}

// BANDS: the first pass has listed all entries from an edge on, below which the k-th magnitude of the last call was not,
// less a margin.  If the boundary bin is not below the edge, the lists hold all that is asked for, and something more
// that the kernels after this one pass over, and this kernel bins them instead of reading the vector; else it writes its
// own lists in their place.
template <bool BANDS>
__global__ __launch_bounds__(kBlock, 4) void k_topk_compact(TopkParams p)
{
    __shared__ uint32_t sh_hist[1024];
    __shared__ uint32_t sh_wave[kWavesPerBlock];
    __shared__ uint32_t sh_out[2];
    __shared__ int2 ring[kWavesPerBlock][kRingSize];
    const int lane = threadIdx.x & 63, wib = threadIdx.x >> 6;
    const uint32_t w = blockIdx.x * kWavesPerBlock + wib;
    const bool active = w < p.nwaves;
    uint32_t bins[kTopkBins / kBlock];
    load_bins<kTopkBins / kBlock, kTopkCopies>(p.hist0, bins);
    // from the last tile to the first: k_topk_hist left the end of the vector in the caches
    const WaveTiles wt = wave_tiles(p, active ? w : 0);
    const DenseSweep ds = dense_sweep(p, wt, true, p.seg);
    f4 a = dense_load(ds, 0, lane);  // behind the histogram's loads, ahead of the search in it
    const int2* list = p.seg + seg_begin(p, active ? w : 0);
    int2 head[2];
    uint32_t n_in = 0, edge = kNoEdge;
    if constexpr (BANDS) {
        head[0] = list[lane];  // a wave owns several tiles
        head[1] = list[64 + lane];
        n_in = active ? p.cnt[w] : 0u;
        edge = p.st->edge;
    }
    for (int i = threadIdx.x; i < 1024; i += kBlock) sh_hist[i] = 0;
    uint32_t b0, k1;
    pick_bin<kTopkBins / kBlock>(bins, (unsigned long long)p.k, sh_wave, sh_out, b0, k1);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        p.st->prefix[0] = b0;
        p.st->k_rem[0] = k1;
    }
    if (BANDS && edge <= b0 << 20) {  // kNoEdge is above all bins
        n_in = __builtin_amdgcn_readfirstlane(n_in);
        auto entry = [&](bool in, int2 e) {
            const uint32_t key = mag_key(__int_as_float(e.y));
            if (in && key >> 20 == b0) atomicAdd(&sh_hist[(key >> 10) & 1023u], 1u);
        };
        entry((uint32_t)lane < n_in, head[0]);
        entry((uint32_t)lane + 64 < n_in, head[1]);
        for (uint32_t c = 128; c < n_in; c += 256) {
            int2 e[4];
#pragma unroll
            for (uint32_t u = 0; u < 4; ++u) e[u] = list[c + u * 64 + lane < n_in ? c + u * 64 + lane : 0u];
#pragma unroll
            for (uint32_t u = 0; u < 4; ++u) entry(c + u * 64 + lane < n_in, e[u]);
        }
    } else if (active) {
        ListWriter lw;
        lw.list = p.seg + seg_begin(p, w);
        lw.ring = ring[wib];
        lw.run = lw.fill = 0;
#pragma unroll 1
        for (uint32_t j = 0; j < ds.nb; ++j) {
            const f4 c = a;
            a = dense_load(ds, j + 1, lane);
            const int32_t i0 = (int32_t)(dense_tile(ds, j) * kTile + lane * 4 - p.shift);
            topk_emit(true, c.x, i0 + 0, b0, lw, lane, sh_hist);
            topk_emit(true, c.y, i0 + 1, b0, lw, lane, sh_hist);
            topk_emit(true, c.z, i0 + 2, b0, lw, lane, sh_hist);
            topk_emit(true, c.w, i0 + 3, b0, lw, lane, sh_hist);
            list_flush(lw, lane);
        }
        for (uint32_t g = 0; g < wt.n - wt.nb; ++g) {
            const uint32_t t = w + guarded_tile(wt, g) * wt.W;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int64_t i = (int64_t)t * kTile + lane * 4 + j - p.shift;
                const bool valid = i >= 0 && i < p.d;
                topk_emit(valid, valid ? p.acc[i] : 0.0f, (int32_t)i, b0, lw, lane, sh_hist);
            }
            list_flush(lw, lane);
        }
        const uint32_t n = list_finish(lw, lane);
        if (lane == 0) p.cnt[w] = n;
    }
    __syncthreads();
    merge_hist(sh_hist, p.hist1, 1024);
}

// k_topk_refine: digit-2 histogram of the list entries whose digits 0 and 1 are b0 and b1
__global__ __launch_bounds__(kBlock) void k_topk_refine(TopkParams p)
{
    __shared__ uint32_t sh_hist[1024];
    __shared__ uint32_t sh_wave[kWavesPerBlock];
    __shared__ uint32_t sh_out[2];
    const ListGroup lists = load_lists(p);
    for (int i = threadIdx.x; i < 1024; i += kBlock) sh_hist[i] = 0;
    const uint32_t b0 = p.st->prefix[0];
    const uint32_t k1 = p.st->k_rem[0];
    uint32_t b1, k2;
    pick_bin<1024 / kBlock>(p.hist1, (unsigned long long)k1, sh_wave, sh_out, b1, k2);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        p.st->prefix[1] = b1;
        p.st->k_rem[1] = k2;
    }
    const uint32_t want = (b0 << 10) | b1;  // key >> 10
    for_lists(lists, [&](bool in, int2 e) {
        const uint32_t key = mag_key(__int_as_float(e.y));
        if (in && (key >> 10) == want) atomicAdd(&sh_hist[key & 1023u], 1u);
    });
    __syncthreads();
    merge_hist(sh_hist, p.hist2, 1024);
}

// Edge for the next call: the k-th magnitude less a margin of 2 % and one and a half times its last change (which later
// calls let shrink by 13 % each), down to the start of its bin of digit 0 (an eighth of an octave at most).  Beyond
// kTopkMargin the lists would grow long: that is a jump, and the next call goes without an edge (see Calm).
constexpr float kTopkMargin = 0.3f;
__device__ void topk_record(const TopkParams& p, float kth)
{
    float m = 0.02f;
    Calm calm = {kCalmMost, kCalmMost};
    if (p.bands == kBandsUse) {
        const float moved = 0.02f + 1.5f * __builtin_fabsf(kth - p.st->last_kth) / p.st->last_kth;
        if (moved <= kTopkMargin) m = moved;
        // a captured call that has not run yet may have left no margin at all
        m = __builtin_fmaxf(m, 0.87f * __builtin_fminf(p.st->margin, kTopkMargin));
        calm = calm_after(p.st->calm, !(moved <= kTopkMargin));
    }
    const float e = kth * (1.0f - m);
    p.st->edge_next = calm_enough(calm) && e > 0.0f && e < __builtin_inff() ? mag_key(e) & ~((1u << 20) - 1u) : kNoEdge;
    p.st->last_kth = kth;
    p.st->margin = m;
    p.st->calm = calm;
}

// k_topk_final: the k-th largest key, the output and the residual update
__global__ __launch_bounds__(kBlock) void k_topk_final(TopkParams p)
{
    __shared__ uint32_t sh_wave[kWavesPerBlock];
    __shared__ uint32_t sh_out[2];
    __shared__ uint32_t sh_gt[kWavesPerBlock], sh_eq[kWavesPerBlock];
    __shared__ unsigned long long sh_base[2];
    const ListGroup lists = load_lists(p);
    // digit 0's histograms are done with: a kernel of its own before every call took 4.7 us
    for (uint32_t i = blockIdx.x * kBlock + threadIdx.x; i < p.clear0; i += gridDim.x * kBlock) p.hist0[i] = 0;
    const uint32_t b0 = p.st->prefix[0], b1 = p.st->prefix[1];
    const uint32_t k2 = p.st->k_rem[1];
    uint32_t b2, need;
    pick_bin<1024 / kBlock>(p.hist2, (unsigned long long)k2, sh_wave, sh_out, b2, need);
    const uint32_t kappa = (b0 << 20) | (b1 << 10) | b2;
    const unsigned long long K = p.k_from_state ? (unsigned long long)p.st->k_eff : (unsigned long long)p.k;
    const int lane = threadIdx.x & 63, wib = threadIdx.x >> 6;

    // pass A: entries above kappa and entries equal to it, per wave
    uint32_t n_gt = 0, n_eq = 0;
    for_lists(lists, [&](bool in, int2 e) {
        const uint32_t key = mag_key(__int_as_float(e.y));
        n_gt += (uint32_t)__popcll(__ballot(in && key > kappa));
        n_eq += (uint32_t)__popcll(__ballot(in && key == kappa));
    });
    if (lane == 0) {
        sh_gt[wib] = n_gt;
        sh_eq[wib] = n_eq;
    }
    __syncthreads();
    uint32_t off_gt = 0, off_eq = 0, tot_gt = 0, tot_eq = 0;
#pragma unroll
    for (int i = 0; i < kWavesPerBlock; ++i) {
        if (i < wib) {
            off_gt += sh_gt[i];
            off_eq += sh_eq[i];
        }
        tot_gt += sh_gt[i];
        tot_eq += sh_eq[i];
    }
    if (threadIdx.x == 0) {
        // one reservation per block and counter (same-address atomics are slow: keep them few)
        sh_base[0] = tot_gt ? atomicAdd(&p.st->gt_ctr, (unsigned long long)tot_gt) : 0ull;
        sh_base[1] = tot_eq ? atomicAdd(&p.st->eq_ctr, (unsigned long long)tot_eq) : 0ull;
        if (blockIdx.x == 0) {
            p.st->prefix[2] = b2;
            p.st->k_rem[2] = need;
            p.st->kth_key = kappa;
            *p.out_count = (int32_t)K;
            *p.out_kth = __int_as_float((int)kappa);
            if (p.bands != kBandsNone) topk_record(p, __int_as_float((int)kappa));
        }
    }
    __syncthreads();
    // the k - need entries above kappa fill the front of the output, the ties the last `need` places
    unsigned long long pos_gt = sh_base[0] + off_gt;
    unsigned long long pos_eq = sh_base[1] + off_eq;
    const unsigned long long tie_base = K - need;

    // pass B: same traversal, writing
    for_lists(lists, [&](bool in, int2 e) {
        const uint32_t key = mag_key(__int_as_float(e.y));
        const bool gt = in && key > kappa, eq = in && key == kappa;
        const unsigned long long m_gt = __ballot(gt), m_eq = __ballot(eq);
        unsigned long long at = 0;
        bool take = false;
        if (gt) {
            at = pos_gt + lane_prefix(m_gt);
            take = at < tie_base;  // always true; keeps a corrupted histogram from writing out of bounds
        } else if (eq) {
            const unsigned long long rank = pos_eq + lane_prefix(m_eq);
            take = rank < need;
            at = tie_base + rank;
        }
        if (take) {
            p.out_idx[at] = e.x;
            p.out_val[at] = __int_as_float(e.y);
            if (p.residual) p.residual[e.x] = 0.0f;
        }
        pos_gt += (unsigned long long)__popcll(m_gt);
        pos_eq += (unsigned long long)__popcll(m_eq);
    });
}

// ---------------------------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------------------------
void launch_topk_zero(const TopkParams& p, hipStream_t s)
{
    hipLaunchKernelGGL(k_topk_zero, dim3((kTopkHist + kBlock - 1) / kBlock), dim3(kBlock), 0, s, p);
}

template <int GT>
static void launch_topk_hist_type(const TopkParams& p, hipStream_t s)
{
    const dim3 grid(p.nblocks), block(kBlock);
    const bool bands = p.bands == kBandsUse;
    if (p.residual && bands) hipLaunchKernelGGL((k_topk_hist<true, GT, true>), grid, block, 0, s, p);
    else if (p.residual) hipLaunchKernelGGL((k_topk_hist<true, GT, false>), grid, block, 0, s, p);
    else if (bands) hipLaunchKernelGGL((k_topk_hist<false, GT, true>), grid, block, 0, s, p);
    else hipLaunchKernelGGL((k_topk_hist<false, GT, false>), grid, block, 0, s, p);
}

void launch_topk_hist(const TopkParams& p, hipStream_t s)
{
    switch (p.gt) {
        case kGradF16: launch_topk_hist_type<kGradF16>(p, s); break;
        case kGradBf16: launch_topk_hist_type<kGradBf16>(p, s); break;
        default: launch_topk_hist_type<kGradF32>(p, s); break;
    }
}

void launch_topk_compact(const TopkParams& p, hipStream_t s)
{
    if (p.bands == kBandsUse) hipLaunchKernelGGL(k_topk_compact<true>, dim3(p.nblocks), dim3(kBlock), 0, s, p);
    else hipLaunchKernelGGL(k_topk_compact<false>, dim3(p.nblocks), dim3(kBlock), 0, s, p);
}

void launch_topk_refine(const TopkParams& p, uint32_t grid, hipStream_t s)
{
    hipLaunchKernelGGL(k_topk_refine, dim3(list_grid(p.nwaves, grid)), dim3(kBlock), 0, s, p);
}

void launch_topk_final(const TopkParams& p, uint32_t grid, hipStream_t s)
{
    hipLaunchKernelGGL(k_topk_final, dim3(list_grid(p.nwaves, grid)), dim3(kBlock), 0, s, p);
}

}  // namespace sidco
