// Radix-select building blocks shared by the exact Top-k comparator and the DGC comparator: the
// magnitude key of an fp32 value, the search of a digit histogram for the bin that holds the k-th
// largest key, the merge of a block's LDS histogram into the global one, and the split of the
// per-wave lists over a small grid.
#ifndef SIDCO_SELECT_H
#define SIDCO_SELECT_H

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "sidco_internal.h"
#include "sidco_device.h"

namespace sidco {

__device__ __forceinline__ uint32_t mag_key(float x) { return (uint32_t)__float_as_int(x) & 0x7fffffffu; }

// A thread's PER bins of a digit histogram of kBlock * PER bins, summed over its COPIES copies.
template <int PER, int COPIES = 1>
__device__ __forceinline__ void load_bins(const uint32_t* __restrict__ hist, uint32_t (&local)[PER])
{
    typedef uint32_t bins __attribute__((ext_vector_type(PER)));
    bins c[COPIES];
#pragma unroll
    for (int k = 0; k < COPIES; ++k)
        c[k] = *reinterpret_cast<const bins*>(hist + k * (kBlock * PER) + threadIdx.x * PER);
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        local[j] = 0;
#pragma unroll
        for (int k = 0; k < COPIES; ++k) local[j] += c[k][j];
    }
}

// Bin of a digit histogram that holds the k-th largest entry, counted from the top bin downwards, and the rank the
// entry has inside that bin; `local` are the thread's bins (load_bins).  Every thread of the block returns the
// same pair.  Needs sum(hist) >= k >= 1.
template <int PER>
__device__ __forceinline__ void pick_bin(const uint32_t (&local)[PER], unsigned long long k, uint32_t* sh_wave,
                                         uint32_t* sh_out, uint32_t& bin, uint32_t& k_in_bin)
{
    const uint32_t t = threadIdx.x, lane = t & 63, wib = t >> 6;
    uint32_t tsum = 0;
#pragma unroll
    for (int j = 0; j < PER; ++j) tsum += local[j];
    // inclusive suffix sums over the threads (counts are at most d < 2^31: no overflow): within the wave, then
    // the totals of the waves behind it
    uint32_t s = tsum;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t other = __shfl_down(s, o, 64);
        s += lane + o < 64 ? other : 0u;
    }
    __syncthreads();  // protects sh_wave / sh_out against a previous use
    if (lane == 0) sh_wave[wib] = s;
    if (t == 0) sh_out[0] = sh_out[1] = 0;  // only reached if the histogram holds fewer than k entries
    __syncthreads();
#pragma unroll
    for (uint32_t i = 1; i < (uint32_t)kWavesPerBlock; ++i) s += i > wib ? sh_wave[i] : 0u;
    const unsigned long long above = (unsigned long long)s - tsum;  // entries in the bins of later threads
    if (above < k && k <= (unsigned long long)s) {                  // exactly one thread
        unsigned long long acc = above;
#pragma unroll
        for (int j = PER - 1; j >= 0; --j) {
            if (acc < k && k <= acc + local[j]) {
                sh_out[0] = t * PER + j;
                sh_out[1] = (uint32_t)(k - acc);
            }
            acc += local[j];
        }
    }
    __syncthreads();
    bin = sh_out[0];
    k_in_bin = sh_out[1];
}

// the same from the histogram in memory
template <int PER>
__device__ __forceinline__ void pick_bin(const uint32_t* __restrict__ hist, unsigned long long k, uint32_t* sh_wave,
                                         uint32_t* sh_out, uint32_t& bin, uint32_t& k_in_bin)
{
    uint32_t local[PER];
    load_bins<PER>(hist, local);
    pick_bin<PER>(local, k, sh_wave, sh_out, bin, k_in_bin);
}

// adds a block's LDS histogram to the global one
__device__ __forceinline__ void merge_hist(const uint32_t* sh_hist, uint32_t* __restrict__ hist, int nb)
{
    for (int i = threadIdx.x; i < nb; i += kBlock) {
        const uint32_t c = sh_hist[i];
        if (c) atomicAdd(&hist[i], c);
    }
}

// ---------------------------------------------------------------------------------------------
// The per-wave lists split over a small grid: a wave takes the lists first, first + 8, ... below last, at most
// kListGroup of them (list_grid), and requests the length and the first 64 entries of each at once:
// one list after the other is two dependent round trips for a handful of entries each.
// ---------------------------------------------------------------------------------------------
constexpr uint32_t kListGroup = 4;
inline uint32_t list_grid(uint32_t nwaves, uint32_t wanted)
{
    const uint32_t least = (nwaves + kListGroup * kWavesPerBlock - 1) / (kListGroup * kWavesPerBlock);
    return wanted > least ? wanted : least;
}
struct ListGroup {
    const int2* list[kListGroup];
    uint32_t n[kListGroup];   // entries
    int2 head[kListGroup];    // the lane's entry among the first 64; stale past the end
};
template <typename P>
__device__ __forceinline__ ListGroup load_lists(const P& p)
{
    const uint32_t per_block = (p.nwaves + gridDim.x - 1) / gridDim.x;
    const uint32_t first = blockIdx.x * per_block + (threadIdx.x >> 6);
    const uint32_t end = (blockIdx.x + 1) * per_block, last = end < p.nwaves ? end : p.nwaves;
    ListGroup g;
#pragma unroll
    for (uint32_t k = 0; k < kListGroup; ++k) {
        const uint32_t sw = first + k * kWavesPerBlock;
        const uint32_t w = sw < last ? sw : 0u;
        g.list[k] = p.seg + seg_begin(p, w);  // room for at least a tile
        g.n[k] = sw < last ? p.cnt[w] : 0u;
        g.head[k] = g.list[k][threadIdx.x & 63];
    }
    return g;
}
// f(in, entry) for every group of 64 entries of the wave's lists, the wave together
template <typename F>
__device__ __forceinline__ void for_lists(const ListGroup& g, F f)
{
    const uint32_t lane = threadIdx.x & 63;
#pragma unroll
    for (uint32_t k = 0; k < kListGroup; ++k) {
        const uint32_t n = __builtin_amdgcn_readfirstlane(g.n[k]);
        if (n > 0) f(lane < n, g.head[k]);
        for (uint32_t c = 64; c < n; c += 64) {
            const bool in = c + lane < n;
            f(in, in ? g.list[k][c + lane] : make_int2(0, 0));
        }
    }
}

}  // namespace sidco
#endif
