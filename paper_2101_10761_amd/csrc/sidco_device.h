// Device-side helpers shared by the kernels of the SIDCo library: wave primitives, the split of the
// vector into per-wave tiles, the sweeps over them, and the LDS-staged writer of per-wave survivor lists.
#ifndef SIDCO_DEVICE_H
#define SIDCO_DEVICE_H

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "sidco_internal.h"

namespace sidco {

typedef float f4 __attribute__((ext_vector_type(4)));

// The value `v` as a lane finds it through one DPP move, zero where the move has no source: within rows of 16 lanes
// from the lane CTRL below (row_shr:1 .. 15 = 0x111 .. 0x11f), or from the last lane of the row(s) before
// (row_bcast:15 = 0x142 into the rows of ROWS = 0xa, row_bcast:31 = 0x143 into those of 0xc).
template <int CTRL, int ROWS, typename T>
__device__ __forceinline__ T dpp_or_zero(T v)
{
    static_assert(sizeof(T) == 8, "two registers");
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, CTRL, ROWS, 0xf, true);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), CTRL, ROWS, 0xf, true);
    return __builtin_bit_cast(T, (uint64_t)hi << 32 | lo);
}

// Sums over the wave in a fixed order, the same in every lane.  Six DPP moves and adds: a shuffle through LDS costs
// several times the latency, and these sums stand in the serial chain of every kernel's prologue and epilogue
// (25.6 M elements, three stages: dense stage 21.6 -> 20.8 us, the two list stages 8.6 -> 6.8 and 7.7 -> 7.0;
// 14.7 M, two stages: dense stage 16.1 -> 14.7, last stage 10.1 -> 9.4).  Several values take every step together: one
// value's moves fill the wait for the adds of the others.
template <int CTRL, int ROWS, int Q, typename T>
__device__ __forceinline__ void wave_step(T (&v)[Q])
{
#pragma unroll
    for (int q = 0; q < Q; ++q) v[q] += dpp_or_zero<CTRL, ROWS>(v[q]);
}
template <int Q, typename T>
__device__ __forceinline__ void wave_totals(T (&v)[Q])
{
    wave_step<0x111, 0xf>(v);
    wave_step<0x112, 0xf>(v);
    wave_step<0x114, 0xf>(v);
    wave_step<0x118, 0xf>(v);  // lane 15 of each row: the row's sum
    wave_step<0x142, 0xa>(v);
    wave_step<0x143, 0xc>(v);  // lane 63: the wave's sum
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const uint64_t u = __builtin_bit_cast(uint64_t, v[q]);
        const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)u, 63);
        const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), 63);
        v[q] = __builtin_bit_cast(T, (uint64_t)hi << 32 | lo);
    }
}
template <typename T>
__device__ __forceinline__ T wave_total(T v)
{
    T a[1] = {v};
    wave_totals(a);
    return a[0];
}

__device__ __forceinline__ double wave_sum(double v) { return wave_total(v); }
__device__ __forceinline__ unsigned long long wave_sum_u64(unsigned long long v) { return wave_total(v); }

__device__ __forceinline__ Calm calm_after(Calm c, bool jumped)
{
    if (jumped) return Calm{0, c.run};
    return Calm{c.run < kCalmMost ? c.run + 1 : kCalmMost, c.last};
}
__device__ __forceinline__ bool calm_enough(Calm c) { return c.run >= (c.last >= kCalmRun ? 1u : kCalmMost); }

// Four elements of 16 bits in two words as fp32 (widening either type is exact).
template <int GT, typename W>
__device__ __forceinline__ f4 widen4(W w)
{
    const uint32_t w0 = w.x, w1 = w.y;  // elements 0,1 and 2,3
    f4 c;
    if constexpr (GT == kGradBf16) {
        c.x = __uint_as_float(w0 << 16);
        c.y = __uint_as_float(w0 & 0xffff0000u);
        c.z = __uint_as_float(w1 << 16);
        c.w = __uint_as_float(w1 & 0xffff0000u);
    } else {
        typedef _Float16 h2 __attribute__((ext_vector_type(2)));
        const h2 lo = __builtin_bit_cast(h2, w0), hi = __builtin_bit_cast(h2, w1);
        c.x = (float)lo.x;
        c.y = (float)lo.y;
        c.z = (float)hi.x;
        c.w = (float)hi.y;
    }
    return c;
}

// Four consecutive gradient elements as fp32, from element e on: one 16-byte load of an fp32 buffer, one 8-byte
// load of an fp16 / bf16 buffer (widening either type is exact).  The address need only be aligned for one
// element: tiles follow the alignment of the accumulated vector, the gradient's may be another one (the load
// instruction is the same; a misaligned stream measured within 2 % of an aligned one).  STREAM: the
// buffer is read once per call, keep it out of the caches' way (a template parameter: as a run-time
// flag the two loads are merged and the non-temporal hint is lost).
template <int GT, bool STREAM>
__device__ __forceinline__ f4 load_grad4(const void* __restrict__ g, size_t e)
{
    if constexpr (GT == kGradF32) {
        typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));
        const f4u* q = reinterpret_cast<const f4u*>(reinterpret_cast<const float*>(g) + e);
        if constexpr (STREAM) return __builtin_nontemporal_load(q);
        else return *q;
    } else {
        typedef uint32_t u2 __attribute__((ext_vector_type(2), aligned(2)));
        const u2* q = reinterpret_cast<const u2*>(reinterpret_cast<const uint16_t*>(g) + e);
        u2 w;
        if constexpr (STREAM) w = __builtin_nontemporal_load(q);
        else w = *q;
        return widen4<GT>(w);
    }
}

// one gradient element as fp32
template <int GT>
__device__ __forceinline__ float load_grad1(const void* __restrict__ g, int64_t i)
{
    if constexpr (GT == kGradF32) return reinterpret_cast<const float*>(g)[i];
    else if constexpr (GT == kGradBf16)
        return __uint_as_float((uint32_t) reinterpret_cast<const uint16_t*>(g)[i] << 16);
    else return (float)reinterpret_cast<const _Float16*>(g)[i];
}

// number of set bits of `mask` below this lane
__device__ __forceinline__ uint32_t lane_prefix(unsigned long long mask)
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// The tiles of one wave of the sparsifier's sweeps: wave w of W takes the tiles w, w + W, w + 2W, ... (in long vectors the sweep
// that forms acc takes others, see acc_tile, as many).  All waves
// then work in one narrow window of the vector that moves through it in address order, which DRAM and the
// memory-side cache serve better than thousands of separate streams (a statistics-only sweep right after k_fit,
// contiguous ranges against this: 16.2 and 13.0 us at 25.6 M elements, 38 and 29 us at 66 M, 106 and 88 us at
// 138 M), and values of a different scale in one part of the vector spread over all lists.  The counts come
// ready from the host (q = T / W, r = T % W): a 64-bit division in every kernel cost 0.5 us each.
// Tiles sit on the grid of 128-byte lines of the accumulated vector, wherever it starts: tile t holds the elements
// 256 t - shift .. 256 t + 255 - shift, `shift` being the number of elements between the boundary before acc[0]
// and acc[0].  On the 16-byte grid alone a tile began and ended inside a line, and that line was fetched, and
// written back in part, by the L2s of two XCDs: 50 tensors of odd lengths, 66 M elements in all, 129 us for the
// first pass and 65 for the dense stage against 124 and 51 now (kGrid of 64 and 256 measured the same as 32).  So tile 0
// is incomplete if shift > 0 and the last tile may be; those two take guarded scalar accesses, every other one whole
// 16-byte accesses.
struct WaveTiles {
    uint32_t w, W;
    uint32_t n;       // tiles of the wave
    uint32_t k0, nb;  // its tiles number k0 .. k0 + nb - 1 are complete
};
template <typename P>  // Params, TopkParams or DgcParams
__device__ __forceinline__ WaveTiles wave_tiles(const P& p, uint32_t w)
{
    WaveTiles t;
    t.w = w;
    t.W = p.nwaves;
    t.n = p.tq + (w < p.tr ? 1u : 0u);
    t.k0 = (w == 0 && p.shift > 0) ? 1u : 0u;
    uint32_t k1 = t.n;
    if (k1 > 0 && w + (k1 - 1) * t.W >= p.nfull) --k1;
    t.nb = k1 > t.k0 ? k1 - t.k0 : 0u;
    return t;
}

// number of the wave's g-th incomplete tile, g < n - nb
__device__ __forceinline__ uint32_t guarded_tile(const WaveTiles& t, uint32_t g)
{
    return (t.nb == 0 || g < t.k0) ? g : g + t.nb;
}

// First tile of wave w if the waves took contiguous ranges of the same lengths.
template <typename P>
__device__ __forceinline__ uint32_t tile_begin(const P& p, uint32_t w)
{
    return w * p.tq + (w < p.tr ? w : p.tr);
}

// Survivor list of wave w: its first slot and the slots it has (one per element of the wave's tiles).
template <typename P>
__device__ __forceinline__ size_t seg_begin(const P& p, uint32_t w) { return (size_t)tile_begin(p, w) * kTile; }
template <typename P>
__device__ __forceinline__ uint32_t seg_slots(const P& p, uint32_t w) { return (p.tq + (w < p.tr ? 1u : 0u)) * kTile; }

// Number of the wave's k-th tile in the sweep that forms acc; they ascend.  In long vectors (`turn`, see kTurnRows)
// the waves do not keep their place in the row.  Blocks go to the eight XCDs in turn, b and b + 256 share a CU and the later
// one ends 1.5 % behind the other, and every other XCD ends 5 % behind its neighbours; where places stay, an XCD has the same
// 8 KB of every 64 KB all the way.  Here the halves of the waves change places from row to row, and in each half of a
// row an XCD has 256 KB in one piece, the piece behind its last one.  A training step, us, places that stay, halves that
// change and this: 14.7 M elements, 2 stages 45.3, 45.3 and 45.1; 25.6 M, 3 stages 72.3, 72.0 and 71.9; 32 M, 2 stages -, 78.1
// and 77.1; 40 M 94.4, 93.6 and 92.3; 66 M, gamma 146.5, 143.8 and 142.0; 78 M, 3 stages -, 188.5 and 186.7; 90 M, 2 stages
// 203, 198.8 and 195.9; 138 M, 3 stages 405.8, 393.0 and 392.2 (first pass 292 and 278).  Pieces of 128 and of 64 KB or that
// move on every other row are slower (66 M 142.7, 147.6, 145.1), and so are places that move on by one, two, four or eight
// blocks a row (138 M 394, 401, 405, 405).  The lists and sums are the wave's whichever its tiles are.
template <typename P>
__device__ __forceinline__ uint32_t acc_tile(const P& p, uint32_t w, uint32_t k)
{
    static_assert(kMaxBlocks == 512 && kWavesPerBlock == 8, "halves of 8 pieces of 32 blocks");
    if (p.turn && k < p.tq) {
        const uint32_t b = w / kWavesPerBlock, half = (b >> 8) ^ (k & 1u), piece = (b + k) & 7u;
        w = ((half * 8 + piece) * 32 + (b >> 3 & 31u)) * kWavesPerBlock + w % kWavesPerBlock;
    }
    return k * p.nwaves + w;
}

// One wave's share of the sweep that forms acc = g + residual (EC; else acc = g) and stores it (WRITE) to p.acc_w.
// The wave requests its next tile before it works on the one it has: one tile (1 KB of each operand) per wave in
// flight is what 16 waves per CU need to keep HBM busy, and more only widens the window of addresses that the chip
// works in (2 and 4 tiles ahead, and 32 waves per CU, were 1 to 5 % slower at 25.6 M to 138 M elements).
// `v` sees every complete tile (v.tile(values, tile number)), every lane of the others (v.one(valid, value, index),
// the wave together) and the end of each of those (v.end()).
// PAST: the residual is read and written past the caches, for a pass whose result is not read again soon.
struct AccTile {
    f4 g, r;
};
template <bool EC, bool WRITE, int GT, bool PAST, typename P>
__device__ __forceinline__ AccTile acc_load(const P& p, size_t i)
{
    AccTile a = {};
    a.g = load_grad4<GT, WRITE>(p.grad, i);
    if constexpr (EC && PAST) a.r = __builtin_nontemporal_load(reinterpret_cast<const f4*>(p.acc_w + i));
    else if constexpr (EC) a.r = *reinterpret_cast<const f4*>(p.acc_w + i);
    return a;
}
template <bool PAST>
__device__ __forceinline__ void acc_store(float* acc, size_t i, f4 c)
{
    if constexpr (PAST) __builtin_nontemporal_store(c, reinterpret_cast<f4*>(acc + i));
    else *reinterpret_cast<f4*>(acc + i) = c;
}
// The first tile of a wave that has a complete one, for a kernel that has something to wait for before its sweep.
template <bool EC, bool WRITE, int GT, bool PAST, typename P>
__device__ __forceinline__ AccTile acc_first(const P& p, uint32_t w, int lane)
{
    const uint32_t t = acc_tile(p, w, (w == 0 && p.shift > 0) ? 1u : 0u);
    return acc_load<EC, WRITE, GT, PAST>(p, (size_t)t * kTile + lane * 4 - p.shift);
}
// `first`: NULL, or that tile
template <bool EC, bool WRITE, int GT, bool PAST = false, typename P, typename V>
__device__ __forceinline__ void acc_sweep(const P& p, uint32_t w, int lane, V& v, const AccTile* first = nullptr)
{
    w = __builtin_amdgcn_readfirstlane(w);
    WaveTiles wt = wave_tiles(p, w);
    // the wave with the vector's last, incomplete tile may be another one than in the other sweeps
    wt.nb = wt.n - wt.k0 - (wt.n > wt.k0 && acc_tile(p, w, wt.n - 1) >= p.nfull ? 1u : 0u);
    if (wt.nb > 0) {
        float* acc = p.acc_w;
        uint32_t t = acc_tile(p, w, wt.k0);
        size_t i = (size_t)t * kTile + lane * 4 - p.shift;
        AccTile a = first ? *first : acc_load<EC, WRITE, GT, PAST>(p, i);
#pragma unroll 1
        for (uint32_t k = 1; k < wt.nb; ++k) {
            f4 c = a.g;
            if (EC) c = a.g + a.r;
            const uint32_t t1 = acc_tile(p, w, wt.k0 + k);
            const size_t i1 = (size_t)t1 * kTile + lane * 4 - p.shift;
            a = acc_load<EC, WRITE, GT, PAST>(p, i1);
            if (WRITE) acc_store<PAST>(acc, i, c);
            v.tile(c, t);
            t = t1;
            i = i1;
        }
        if (EC) a.g = a.g + a.r;
        if (WRITE) acc_store<PAST>(acc, i, a.g);
        v.tile(a.g, t);
    }
    for (uint32_t k = 0; k < wt.n - wt.nb; ++k) {
        const uint32_t t = acc_tile(p, w, guarded_tile(wt, k));
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int64_t i = (int64_t)t * kTile + lane * 4 + j - p.shift;
            const bool valid = i >= 0 && i < p.d;
            float c = 0.0f;
            if (valid) {
                c = load_grad1<GT>(p.grad, i);
                if (EC) c = c + p.acc_w[i];
                if (WRITE) p.acc_w[i] = c;
            }
            v.one(valid, c, i);
        }
        v.end();
    }
}

// The sweep of one wave over its tiles of the dense vector.  `reverse` walks them from the last to the first: the
// kernel before this one left the end of what it touched last in the caches, and the host alternates the
// direction from pass to pass so that each pass starts where the one before it stopped.
// The loads are non-temporal: the vector has just been written by the first pass and much of it is still dirty in the
// memory-side cache; reads that do not allocate behind it neither push those lines out early nor wait for them
// (first pass and a statistics-only sweep together, plain against non-temporal loads: 65.7 and 63.9 us at 25.6 M
// elements, 160 and 153 us at 66 M, 366 and 334 us at 138 M).  Calls that clear much of the residual right after such a
// sweep take ordinary loads (see keeps_much in the host code).
struct DenseSweep {
    const float* x;   // element 0 of tile 0, or a readable stand-in if the wave has no complete tile
    uint32_t nb;      // complete tiles of the wave
    uint32_t first;   // the first one in walking order
    int32_t step;     // from one tile to the next in walking order
    uint32_t any;     // a complete tile, the same one for every wave
};

template <typename P>
__device__ __forceinline__ DenseSweep dense_sweep(const P& p, const WaveTiles& wt, bool reverse, const int2* stand_in)
{
    DenseSweep d;
    d.nb = wt.nb;
    d.x = d.nb > 0 ? p.acc - p.shift : reinterpret_cast<const float*>(stand_in);
    const uint32_t k = wt.k0 + (reverse ? d.nb - 1 : 0u);
    d.first = d.nb > 0 ? wt.w + k * wt.W : 0u;
    d.step = reverse ? -(int32_t)wt.W : (int32_t)wt.W;
    d.any = (d.nb > 0 && p.shift > 0) ? 1u : 0u;
    return d;
}

// Tile number of the wave's j-th complete tile in walking order.
__device__ __forceinline__ uint32_t dense_tile(const DenseSweep& d, uint32_t j)
{
    return d.first + (uint32_t)((int32_t)j * d.step);
}

// That tile's values.  Past the wave's last tile the same tile for every wave: the load is unconditional (loads under
// a run-time condition come with waits on the spot), but costs no HBM traffic.  KEEP: an ordinary load.
template <bool KEEP = false>
__device__ __forceinline__ f4 dense_load(const DenseSweep& d, uint32_t j, int lane)
{
    const uint32_t t = j < d.nb ? dense_tile(d, j) : d.any;
    const f4* q = reinterpret_cast<const f4*>(d.x + (size_t)t * kTile) + lane;
    if constexpr (KEEP) return *q;
    else return __builtin_nontemporal_load(q);
}

// A wave's survivor list under construction.  Entries are collected in LDS and written out in long
// contiguous runs: global stores complete in order with the wave's loads, so a store issued between
// two batches of streaming loads holds the next batch back by its own round trip; few, large,
// full-line stores cost a fraction of one small partial-line store per tile component (measured:
// 1.6 M entries out of 25.6 M elements add 9 us as they come and 3 us staged).
constexpr uint32_t kRingFlush = 512;                // staged entries that trigger a write-out
constexpr uint32_t kRingSize = kRingFlush + kTile;  // a whole tile can arrive between two checks
template <typename T>
struct ListWriterT {
    T* __restrict__ list;  // the wave's list in global memory (room for every element of its tiles)
    T* ring;               // the wave's staging area in LDS, kRingSize entries
    uint32_t run;          // entries already written to `list` (wave-uniform)
    uint32_t fill;         // entries staged in `ring` (wave-uniform, < kRingFlush after list_flush)
};
typedef ListWriterT<int2> ListWriter;  // (index, value bits) pairs

template <typename T>
__device__ __forceinline__ void list_push_entry(ListWriterT<T>& lw, bool keep, T e, int lane)
{
    const unsigned long long mask = __ballot(keep);
    if (keep) lw.ring[lw.fill + lane_prefix(mask)] = e;
    lw.fill += (uint32_t)__popcll(mask);
}

__device__ __forceinline__ void list_push(ListWriter& lw, bool keep, int32_t idx, float x, int lane)
{
    list_push_entry(lw, keep, make_int2(idx, __float_as_int(x)), lane);
}

// After at most kTile pushes: writes out kRingFlush entries at a time while that many are staged.
template <typename T>
__device__ __forceinline__ void list_flush(ListWriterT<T>& lw, int lane)
{
    if (lw.fill < kRingFlush) return;  // wave-uniform
    const uint32_t whole = lw.fill & ~(kRingFlush - 1);
#pragma unroll 1
    for (uint32_t c = 0; c < whole; c += 64) lw.list[lw.run + c + lane] = lw.ring[c + lane];
    // the leftover (fewer than kRingFlush entries) moves to the front; LDS accesses of a wave stay in order
    const uint32_t left = lw.fill - whole;
#pragma unroll 1
    for (uint32_t c = 0; c < left; c += 64)
        if (c + lane < left) lw.ring[c + lane] = lw.ring[whole + c + lane];  // source and destination are disjoint
    lw.run += whole;
    lw.fill = left;
}

// writes out what is still staged; returns the list's length
template <typename T>
__device__ __forceinline__ uint32_t list_finish(ListWriterT<T>& lw, int lane)
{
#pragma unroll 1
    for (uint32_t c = 0; c < lw.fill; c += 64)
        if (c + lane < lw.fill) lw.list[lw.run + c + lane] = lw.ring[c + lane];
    lw.run += lw.fill;
    lw.fill = 0;
    return lw.run;
}

}  // namespace sidco
#endif
