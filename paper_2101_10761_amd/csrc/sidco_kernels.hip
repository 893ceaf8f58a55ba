// SIDCo gradient sparsifier for MI355X (gfx950): device kernels and their launchers.
//
// Pipeline of one call (arXiv 2101.10761; Algorithm 1 "Sparsify", Sec. 2.3-2.4, App. B.2-B.3):
//
//   k_fit        acc = g + residual, stored back to residual; per-block fp64 partial sums of
//                |acc|, acc^2, log2|acc| (whichever the chosen law needs)       [reads 8 B, writes 4 B / element]
//                Two launch shapes: every wave walks its own tiles (short vectors), or
//                k_fit_flat, one float4 per thread in address order, followed by k_fit_reduce, which
//                folds the per-block sums into the 512 slots the next kernel expects (long vectors, and from a
//                lower length on calls that clear much of the residual; see fit_uses_flat).
//                The gradient may be fp16 / bf16; it is widened as it is read.
//   k_fit_bands  the same for a call that repeats a shape: it also sums up and lists what the stages will ask for if
//                the thresholds fall near the last call's.
//   stage m      m = 1..M, one kernel each.  Prologue: the first wave of every block reduces the previous kernel's
//                partial sums in a fixed order and evaluates the closed-form threshold eta_m in
//                fp64 (the same arithmetic, hence identical bits, in every block).
//                k_compact: the stage whose source is the dense acc (m = 1; also later stages while the
//                exceedances are still a large part of the vector).  It forms n and the sums of
//                (|x| - eta_m) and its square over the exceedances for the next stage's fit, and writes
//                per-wave lists of the entries above a candidate threshold at or above eta_m - high enough
//                that the lists stay short, low enough (judged from the fit and from where the previous
//                call's next threshold fell) that the next stage can select from them alone.  A wave requests
//                its first tile before its threshold is known and stays a tile ahead.
//                k_lists: a middle stage whose source is those lists (or, if they turn out not to reach
//                down to its threshold, the dense acc again): same sums, exact exceedance lists out.
//                k_final_lists: the last stage for M >= 2; it selects, writes the contiguous
//                (index, value) output and zeroes the residual at those indices in one kernel, each
//                block reserving its output range with one atomic.
//                k_eta, k_select: the last stage of a call that keeps a large part of a long vector: it selects from the
//                dense vector and writes the residual back whole.
//   k_small      the whole call in one block, for a vector of at most kSmallMaxD elements.
//   k_gather     M = 1 only (last stage read the dense vector): exclusive prefix over the per-block
//                survivor counts, copy of the lists into the output, residual zeroing.
//
// Design rules, from measurement on this chip: same-address atomics serialise at ~11 ns each and a
// device-scope fence in a write-heavy kernel forces an L2 write-back, so the big kernels have
// neither.  Kernel boundaries are the only global synchronisation; every wave owns one of every nwaves
// 256-element tiles and a survivor list with room for all of its own, so list positions need no atomics,
// and thresholds, selected set and values are deterministic.
// The *_batched kernels run the same bodies for the vectors of a batch, each block on the vector that a
// table on the device assigns to it.
//
// All floating-point accumulation is fp64 (full rate on CDNA4 vector ALUs); comparisons are fp32
// against the fp32 threshold, so the decision |x| > eta is the same one an fp32 reference takes.
#include <hip/hip_runtime.h>
#include <float.h>
#include <math.h>
#include <stdint.h>

#include <type_traits>

#include "sidco_internal.h"
#include "sidco_device.h"

namespace sidco {

// Sums of `v[q]` over the block, in a fixed order; every thread returns the same values.
template <int Q>
__device__ __forceinline__ void block_sum(double (&v)[Q], double (*sh)[4])
{
    const int lane = threadIdx.x & 63, wib = threadIdx.x >> 6;
    wave_totals(v);
    __syncthreads();  // protects sh against a previous use
    if (lane == 0) {
#pragma unroll
        for (int q = 0; q < Q; ++q) sh[wib][q] = v[q];
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        double t = 0.0;
#pragma unroll
        for (int i = 0; i < kWavesPerBlock; ++i) t += sh[i][q];
        v[q] = t;
    }
}

// ---------------------------------------------------------------------------------------------
// closed-form thresholds (fp64, evaluated redundantly by every thread of every block)
// ---------------------------------------------------------------------------------------------

// A fitted law, reduced to what its quantile above the stage's location needs:
//   linear : t(L) = s * L + c   exponential (eqs. (6), (10)-(11)): s = mean, c = 0
//                               gamma (Corollary 1.2): s = beta, c = -beta * log Gamma(alpha)
//                               degenerate fits: s = 0, c = the limit of the closed form
//   gpd    : t(L) = (b / a) * (exp(a L) - 1)   moment-matched GPD (eqs. (7)-(9); Corollary 1.3):
//                               a = (1 - mu^2/var) / 2, b = mu (mu^2/var + 1) / 2
// with L = log(1/ratio).  The parameters are computed once in fp64; the stage's own threshold is the
// fp64 quantile, the candidate threshold (any value at or above it would do) a cheaper fp32 one.
struct Fit {
    bool gpd;
    double s, c, a, b;
};

__device__ __forceinline__ Fit fit_linear(double s, double c)
{
    Fit f;
    f.gpd = false;
    f.s = s;
    f.c = c;
    f.a = f.b = 0.0;
    return f;
}

__device__ __forceinline__ Fit fit_gpd(double mu, double var, uint32_t& status)
{
    if (!(var > 0.0)) {  // all magnitudes equal: limit of the closed form as var -> 0+
        status |= kStVarZero;
        return fit_linear(0.0, mu);
    }
    const double q = (mu * mu) / var;
    Fit f;
    f.gpd = true;
    f.a = 0.5 * (1.0 - q);
    f.b = 0.5 * mu * (q + 1.0);
    f.s = f.c = 0.0;
    if (f.a == 0.0) return fit_linear(f.b, 0.0);  // the exponential limit
    return f;
}

// Stage-1 fit of the chosen law to |acc| (Corollary 1 / eq. (6); Corollaries 1.2, 1.3).
// `var` is only used for the GPD law, `mulog` only for the gamma law.
__device__ Fit stage1_fit(int dist, double mu, double var, double mulog, uint32_t& status)
{
    if (dist == kDistExp) return fit_linear(mu, 0.0);  // eq. (6)
    if (dist == kDistGpd) return fit_gpd(mu, var, status);
    // gamma law: closed-form shape from s = log(mean) - mean(log), threshold -beta (log delta + log Gamma(alpha))
    const double s = log(mu) - mulog;
    if (!(s > 0.0)) {  // the closed form tends to -infinity here and negative thresholds clamp to 0
        status |= kStGammaS;
        return fit_linear(0.0, 0.0);
    }
    const double a = (3.0 - s + sqrt((s - 3.0) * (s - 3.0) + 24.0 * s)) / (12.0 * s);
    const double b = mu / a;
    return fit_linear(b, -b * lgamma(a));
}

// Stage m >= 2 fit of the exceedances over eta_{m-1}
// (Lemma 2 / eqs. (7)-(9) for the GPD chains, Corollary 2 / eqs. (10)-(11) for the exponential chain).
__device__ Fit pot_fit(int dist, double ybar, double yvar, uint32_t& status)
{
    if (dist == kDistExp) return fit_linear(ybar, 0.0);
    return fit_gpd(ybar, yvar, status);
}

// the stage's threshold above its location, fp64
__device__ __forceinline__ double fit_quantile(const Fit& f, double L)
{
    return f.gpd ? (f.b / f.a) * expm1(f.a * L) : f.s * L + f.c;
}

// a candidate threshold above the location, fp32 arithmetic (its accuracy does not matter)
__device__ __forceinline__ float fit_quantile_fast(const Fit& f, double L)
{
    if (!f.gpd) return (float)(f.s * L + f.c);
    return (float)(f.b / f.a) * expm1f((float)(f.a * L));
}

// log(1/delta_i) of stage i+1.  A chain of selects rather than an index: the arguments of a batched launch
// are assembled in registers, and an indexed array there would be spilled to scratch memory.
__device__ __forceinline__ double stage_L(const Params& p, int i)
{
    double v = 0.0;
#pragma unroll
    for (int j = 0; j < SIDCO_MAX_STAGES; ++j)
        if (j == i) v = p.L[j];
    return v;
}

__device__ __forceinline__ Blk whole_grid() { return Blk{blockIdx.x, gridDim.x, 0u, blockIdx.x == 0}; }
// The same for a stage's kernel.  `none` is zero, but the compiler does not know: it comes with the arguments that the
// kernel needs ahead of its threshold, and what is loaded with it waits for all of them at once.  Fetched one by one as
// they come up they are a chain of round trips, 0.2 us each.
__device__ __forceinline__ Blk stage_grid(const Params& p)
{
    uint32_t none;
    asm("s_mov_b32 %0, 0"
        : "=s"(none)
        : "s"(p.st), "s"(p.part_in), "s"(p.blk_in), "s"(p.band_part), "s"(p.stage), "s"(p.nblocks), "s"(p.dist), "s"(p.nwaves),
          "s"(p.tq), "s"(p.tr), "s"(p.theta), "s"(p.use_hint), "s"(p.band_seg), "s"(p.band_cnt), "s"(p.seg_in), "s"(p.cnt_in),
          "s"(p.seg_out), "s"(p.acc), "s"(p.shift), "s"(p.nfull), "s"(p.reverse), "s"(p.M), "s"(p.L_stage), "s"(p.L_next),
          "s"(p.d), "s"(p.theta_min));
    return Blk{blockIdx.x, gridDim.x, none, blockIdx.x == 0};
}

// What the prologue of a stage's kernel hands to its body.
struct StageEta {
    float eta;      // eta_m: the stage's threshold (statistics of the next fit; selection in the last stage)
    float eta_w;    // the lists this kernel writes hold every entry above eta_w (eta_w >= eta)
    bool lists_ok;  // the producer's lists hold every entry above eta: they can stand in for the dense vector
    bool hit;       // eta fell into the stage's band: the first pass's sums and lists serve the stage
};

// Prologue of every stage kernel (prologue_load, prologue_finish): reduce the producer's per-block partial sums (fixed
// order) and evaluate eta for stage p.stage.
//
// Speculative candidate lists.  A stage that reads the dense vector and keeps a large fraction
// (delta_1 = 0.25) would have to write a quarter of it as 8-byte pairs, or make the next stage read the
// dense vector again.  Instead it evaluates the SAME fitted law a second time at a smaller ratio,
// log(1/ratio) = L_m + theta * L_{m+1}, and writes only the entries above that candidate threshold
// eta_w.  theta is the host's setting (0.5: halfway between this stage's target and the next one's) or,
// when the previous call on the device had the same shape, the place where that call's next
// threshold really fell, less a margin (and not so low that the lists would outgrow what the host
// planned for: theta_min).  The next stage's eta is computed from the exact statistics as
// always; if it lands at or above eta_w the candidate lists contain every entry it can select and
// replace the dense vector, else that kernel falls back to the dense vector.  Either way the result is
// the same: only the time depends on the guess.
//
// What a stage's prologue reads from memory: issued as early as possible, and BEFORE any bulk loads of
// the kernel's body - the wave's memory counter retires in order, so a wait for these few values would
// otherwise also wait for every load issued ahead of them.
// The partial sums are the first wave's: it adds them up alone, eight of each kind per lane, and goes on to the closed
// form without waiting for the rest of the block.  A prologue is a chain of latencies - arguments, partial sums, the sums,
// the closed form - and sets the time of every stage that reads only lists.  With a value per thread, a sum over the block,
// arguments and state fetched as they came up, the lists' loads ahead of the partial sums' and the bookkeeping of block 0
// ahead of the threshold's way to the other waves, a training step took, us, and so: 2.6 M elements, 2 stages 22.7 and 21.5;
// 14.7 M, 2 stages 46.8 and 44.8; 25.6 M, 3 stages 76.0 and 72.4, with a bf16 gradient 67.9 and 64.8.
typedef double d2 __attribute__((ext_vector_type(2), aligned(8)));
typedef uint32_t u2 __attribute__((ext_vector_type(2), aligned(4)));
constexpr int kPartLoads = kMaxBlocks / 128;
static_assert(kMaxBlocks % 128 == 0, "every partial sum is loaded");
struct PrologueLoads {
    d2 a[kPartLoads], b[kPartLoads];  // the lane's share of the producer's partial sums: the first quantity's, the second's
    u2 n[kPartLoads];                 // and of the counts
    float eta_prev;     // eta_{m-1}
    uint32_t status;    // status bits accumulated up to stage m-1
    bool frozen;        // an empty exceedance set has stopped the refinement
    float list_eta;     // the producer's lists hold every entry above this
    float seen;         // where the next stage's threshold fell last time (hint), NaN if unknown
};

// Whether all thresholds so far fell into their bands (see k_fit_bands), and then the stage's own band; the last stage's
// has no upper edge.
struct BandEdges {
    bool live;
    bool over;   // they did, but the first pass found more entries than its lists have room for
    float lo, hi;
    float cand;  // > 0: what the stage's lists are to start from then (a batch's first stage)
};

// The quantity that the law adds to the plain sum: rows of the partial sums of the first pass and of a stage.
__device__ __forceinline__ int second_row(int dist, int m)
{
    if (dist == kDistExp) return 0;  // none: the first once more
    return m == 1 && dist == kDistGamma ? 2 : 1;
}

// How a block gets at the partial sums: its first wave loads them; every thread has a share, which the block adds up; or every
// thread loads one, and the first wave adds them up from LDS, with the same bits as in the first way.
constexpr int kSumsWave = 0, kSumsBlock = 1, kSumsStaged = 2;

template <int SUMS = kSumsWave>
__device__ __forceinline__ PrologueLoads prologue_load(const Params& p, Blk b, bool auto_src)
{
    const int m = p.stage;  // 1-based
    PrologueLoads g;
    if (SUMS == kSumsWave && threadIdx.x < 64) {
        const double* first = p.part_in;
        const double* second = p.part_in + (size_t)second_row(p.dist, m) * kBatchBlocks;
        const uint32_t most = ((p.nblocks - 1) & ~1u) + b.none;  // pairs past the last block's are that one's again: an unused value at most
#pragma unroll
        for (int k = 0; k < kPartLoads; ++k) {
            const uint32_t i = min((uint32_t)(128 * k) + 2 * threadIdx.x, most);
            g.a[k] = *reinterpret_cast<const d2*>(first + i);
            g.b[k] = *reinterpret_cast<const d2*>(second + i);
            g.n[k] = *reinterpret_cast<const u2*>(p.blk_in + i);  // in stage 1 too: under a condition 0.3 % of a call slower
        }
    }
    g.seen = (p.theta > 0.0f && p.use_hint) ? p.st->theta_seen[m] : __builtin_nanf("");
    g.list_eta = auto_src ? p.st->list_eta[m - 1] : 0.0f;
    g.eta_prev = 0.0f;
    g.status = 0;
    g.frozen = false;
    if (m > 1) {
        g.eta_prev = p.st->diag.eta[m - 2];
        g.status = p.st->status_after[m - 1];
        g.frozen = p.st->frozen_after[m - 1] != 0;
    }
    return g;
}

// What the stage's fit is made from, by the first wave: sums of |x| (stage 1) or y = |x| - eta_{m-1} over the exceedances,
// the law's second quantity, and the exceedances' number (anything in stage 1, where nothing asks for it).
struct StageSums {
    double first, second, n;
};
__device__ __forceinline__ StageSums prologue_sums_staged(const double* staged)
{
    double v[2] = {0.0, 0.0};
#pragma unroll
    for (int k = 0; k < kPartLoads; ++k) {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            v[0] += staged[128 * k + 2 * threadIdx.x + j];
            v[1] += staged[kMaxBlocks + 128 * k + 2 * threadIdx.x + j];
        }
    }
    wave_totals(v);
    return StageSums{v[0], v[1], 0.0};
}
__device__ __forceinline__ StageSums prologue_sums(const Params& p, const PrologueLoads& g)
{
    double v[3] = {0.0, 0.0, 0.0};
#pragma unroll
    for (int k = 0; k < kPartLoads; ++k) {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const bool have = (uint32_t)(128 * k + j) + 2 * threadIdx.x < p.nblocks;
            v[0] += have ? g.a[k][j] : 0.0;
            v[1] += have ? g.b[k][j] : 0.0;
            v[2] += have ? (double)g.n[k][j] : 0.0;  // counts < 2^31: exact in fp64
        }
    }
    wave_totals(v);
    return StageSums{v[0], v[1], v[2]};
}

// Behind an unfolded flat first pass (stage 1 of a batch) a thread's share of the partial sums is several values:
// loaded together with the prologue's other loads, added up once the bulk loads are on their way.
struct FlatPart {
    const double* part;  // the vector's partial sums
    uint32_t n;          // their number for each quantity, at most kFlatDirect
    uint32_t stride;     // from one quantity's to the next one's
};
struct FlatLoads {
    double a[kFlatDirect / kBlock], b[kFlatDirect / kBlock];
};
__device__ __forceinline__ FlatLoads flat_load(const FlatPart& fp, int dist)
{
    FlatLoads f;
    // the law's second quantity, if it has one
    const double* second = fp.part + (size_t)(dist == kDistGamma ? 2 : dist == kDistGpd ? 1 : 0) * fp.stride;
#pragma unroll
    for (uint32_t k = 0; k < kFlatDirect / kBlock; ++k) {
        const uint32_t i = k * kBlock + threadIdx.x;
        const uint32_t at = i < fp.n ? i : 0u;
        f.a[k] = fp.part[at];
        f.b[k] = second[at];
    }
    return f;
}
// the thread's share: of the sum of magnitudes, of the second quantity, and 0 exceedances
__device__ __forceinline__ void flat_sums(const FlatPart& fp, const FlatLoads& f, double (&v)[3])
{
    double a = 0.0, b = 0.0;
#pragma unroll
    for (uint32_t k = 0; k < kFlatDirect / kBlock; ++k) {
        if (k * kBlock + threadIdx.x < fp.n) {
            a += f.a[k];
            b += f.b[k];
        }
    }
    v[0] = a;
    v[1] = b;
    v[2] = 0.0;
}

// What block 0 keeps of a stage.
struct StageRecord {
    double stats[3];
    unsigned long long n;
    uint32_t status;  // accumulated, this stage's bits among them
    bool frozen;
    Fit fit;
    float loc;
};

// Evaluates eta for stage p.stage from the reduced sums; called by the first wave of a block.
__device__ __forceinline__ StageEta stage_eval(const Params& p, bool auto_src, const PrologueLoads& g, const StageSums& sums,
                                               StageRecord& rec, const BandEdges& band = BandEdges{})
{
    const int m = p.stage;  // 1-based
    const double L = p.L_stage;
    // candidate threshold of this kernel's lists: log-ratio Lw > L, or none
    double Lw = 0.0;
    if (p.theta > 0.0f) {
        float theta = p.theta;
        if (g.seen == g.seen) theta = fminf(fmaxf(g.seen - kHintMargin, p.theta_min), kHintMax);
        Lw = L + (double)theta * p.L_next;
    }
    Fit fit = fit_linear(0.0, 0.0);
    float loc = 0.0f;
    uint32_t status = g.status;
    double stats[3] = {0.0, 0.0, 0.0};
    StageEta r;
    bool frozen = g.frozen;
    unsigned long long n;
    r.eta = r.eta_w = 0.0f;
    r.lists_ok = false;
    r.hit = false;
    if (m == 1) {
        n = (unsigned long long)p.d;
        const double d = (double)p.d;
        const double mu = sums.first / d;
        double var = 0.0, mulog = 0.0;
        bool finite = isfinite(mu);
        if (p.dist == kDistGpd) {
            var = sums.second / d - mu * mu;
            finite = finite && isfinite(var);
        } else if (p.dist == kDistGamma) {
            mulog = (sums.second / d) * 0.6931471805599453094;  // log2 -> natural log
            finite = finite && isfinite(mulog);
        }
        stats[0] = mu;
        stats[1] = var;
        stats[2] = mulog;
        if (!finite) {
            status |= kStNonfinite;
            r.eta = r.eta_w = __builtin_nanf("");
        } else {
            fit = stage1_fit(p.dist, mu, var, mulog, status);
            double tq = fit_quantile(fit, L);
            if (tq < 0.0) {  // only the gamma form can be negative: delta_1 * Gamma(alpha) > 1
                status |= kStGammaClamp;
                tq = 0.0;
            }
            r.eta = r.eta_w = (float)tq;
            if (Lw > L) {
                const float c = fit_quantile_fast(fit, Lw);
                if (c > r.eta) r.eta_w = c;
            }
        }
    } else {
        const float eta_prev = g.eta_prev;
        n = (unsigned long long)sums.n;
        r.eta = r.eta_w = eta_prev;
        if (!frozen) {
            if (n == 0) {  // nothing exceeds eta_prev: keep it for all later stages
                frozen = true;
                status |= kStStopped;
            } else {
                const double ybar = sums.first / (double)n;
                const double yvar = p.dist == kDistExp ? 0.0 : sums.second / (double)n - ybar * ybar;
                stats[0] = ybar;
                stats[1] = yvar;
                fit = pot_fit(p.dist, ybar, yvar, status);
                loc = eta_prev;
                r.eta = r.eta_w = (float)((double)eta_prev + fit_quantile(fit, L));
                if (Lw > L) {
                    const float c = eta_prev + fit_quantile_fast(fit, Lw);
                    if (c > r.eta) r.eta_w = c;
                }
            }
        }
    }
    // both false for a NaN threshold, which selects nothing anyway
    r.hit = band.live && r.eta >= band.lo && r.eta <= band.hi;
    r.lists_ok = auto_src && !band.live && r.eta >= g.list_eta;
    if (r.hit && band.cand > 0.0f) r.eta_w = band.cand;
    if (!r.hit && (band.live || band.over || (auto_src && !r.lists_ok))) status |= kStFallback;
    rec.stats[0] = stats[0];
    rec.stats[1] = stats[1];
    rec.stats[2] = stats[2];
    rec.n = n;
    rec.status = status;
    rec.frozen = frozen;
    rec.fit = fit;
    rec.loc = loc;
    return r;
}

// Block 0's first thread: the stage in the diagnostics and for the stages behind it.
__device__ __forceinline__ void stage_record(const Params& p, const StageEta& r, const StageRecord& rec)
{
    const int m = p.stage;
    p.st->diag.eta[m - 1] = r.eta;
    p.st->diag.n[m - 1] = (int64_t)rec.n;
    p.st->diag.stats[m - 1][0] = rec.stats[0];
    p.st->diag.stats[m - 1][1] = rec.stats[1];
    p.st->diag.stats[m - 1][2] = rec.stats[2];
    p.st->status_after[m] = rec.status;
    p.st->frozen_after[m] = rec.frozen ? 1u : 0u;
    p.st->list_eta[m] = r.eta_w;
    if (p.theta > 0.0f) {
        FitRecord f;
        f.gpd = rec.fit.gpd ? 1 : 0;
        f.loc = rec.loc;
        f.s = rec.fit.s;
        f.c = rec.fit.c;
        f.a = rec.fit.a;
        f.b = rec.fit.b;
        p.st->cand_fit[m] = f;
    }
}

// One thread of the last stage's kernel: where the threshold fell for which stage p.cand_stage wrote candidate lists, for
// the next call.  Inverts that stage's quantile function at the next one's threshold: eta = loc + Q(L_s + theta L_{s+1}).
// Here, beside the reservation's round trip, and not where the threshold is evaluated: a logarithm and two divisions more
// than the other blocks have, 0.6 us in the chain of block 0.
__device__ __forceinline__ void hint_record(const Params& p, float eta_last)
{
    const int s = p.cand_stage;
    if (s == 0) return;
    const FitRecord f = p.st->cand_fit[s];
    const float eta = s + 1 == p.M ? eta_last : p.st->diag.eta[s];
    const bool frozen = p.st->frozen_after[s + 1] != 0;
    const double tq = (double)eta - (double)f.loc;
    const double Lq = f.gpd ? log1p(tq * f.a / f.b) / f.a : (tq - f.c) / f.s;
    const float seen = (float)((Lq - stage_L(p, s - 1)) / stage_L(p, s));
    p.st->theta_seen[s] = (frozen || !(fabsf(seen) < 1.0e6f)) ? __builtin_nanf("") : seen;
}

template <typename T>
__device__ __forceinline__ void present(T x) { asm volatile("" ::"v"(x)); }

// Reduces the partial sums (fixed order) and evaluates eta for stage p.stage.  Returns the same values
// in every thread of every block.  Block 0 records the stage in the diagnostics.  `v`: the thread's share of the
// sums, `staged`: LDS for kMaxBlocks of each kind (see kSumsWave).
template <int SUMS = kSumsWave>
__device__ __forceinline__ StageEta prologue_finish(const Params& p, Blk b, bool auto_src, const PrologueLoads& g, const BandEdges& band = BandEdges{},
                                                    double (*v)[3] = nullptr, double (*sh)[4] = nullptr, double* staged = nullptr)
{
    __shared__ float sh_eta[4];
    const uint32_t t = threadIdx.x;
    // have what the closed form asks for loaded by now: the compiler would put the loads where it is used, a round trip
    // behind the sums
    present(g.eta_prev);
    present(g.list_eta);
    present(g.seen);
    present(g.status);
    present(g.frozen ? 1u : 0u);
    present(band.lo);
    present(band.hi);
    present(band.cand);
    if constexpr (SUMS == kSumsBlock) block_sum<3>(*v, sh);
    if constexpr (SUMS == kSumsStaged) {
        static_assert(kMaxBlocks == kBlock, "a place for every thread");
        staged[t] = (*v)[0];
        staged[kMaxBlocks + t] = (*v)[1];
        __syncthreads();
    }
    // One wave per block evaluates the closed form - a few hundred dependent fp64 instructions, more for
    // the gamma law - and the others wait: with every wave at it, four per SIMD take turns on the same
    // arithmetic and the prologue lasts that much longer (measured).
    StageEta r;
    StageRecord rec;
    if (t < 64) {
        StageSums sums;
        if constexpr (SUMS == kSumsBlock) sums = StageSums{(*v)[0], (*v)[1], (*v)[2]};
        else if constexpr (SUMS == kSumsStaged) sums = prologue_sums_staged(staged);
        else sums = prologue_sums(p, g);
        r = stage_eval(p, auto_src, g, sums, rec, band);
        if (t == 0) {
            sh_eta[0] = r.eta;
            sh_eta[1] = r.eta_w;
            sh_eta[2] = r.lists_ok ? 1.0f : 0.0f;
            sh_eta[3] = r.hit ? 1.0f : 0.0f;
        }
    }
    __syncthreads();
    if (b.records && t == 0) stage_record(p, r, rec);
    r.eta = sh_eta[0];
    r.eta_w = sh_eta[1];
    r.lists_ok = sh_eta[2] != 0.0f;
    r.hit = sh_eta[3] != 0.0f;
    return r;
}

// both halves back to back, for kernels whose body loads little before the threshold is known
__device__ __forceinline__ StageEta stage_prologue(const Params& p, Blk b, bool auto_src, const BandEdges& band = BandEdges{})
{
    const PrologueLoads g = prologue_load(p, b, auto_src);
    return prologue_finish(p, b, auto_src, g, band);
}

// ---------------------------------------------------------------------------------------------
// k_fit: error-compensation add (App. B.2) fused with the sums of the stage-1 fit
// ---------------------------------------------------------------------------------------------
template <int DIST>
__device__ __forceinline__ void fit_accum(float x, double& s1, double& s2, double& sl, int& se)
{
    const float a = __builtin_fabsf(x);
    const double da = (double)a;
    s1 += da;
    if constexpr (DIST == kDistGpd) s2 = __builtin_fma(da, da, s2);  // a*a is exact in fp64
    if constexpr (DIST == kDistGamma) {
        // log2 max(|x|, 2^-126) = exponent + log2(mantissa in [0.5,1)): the exponents are summed
        // exactly as integers, the hardware log2 only sees [0.5,1) where its error is <= 1 ulp of a
        // value in [-1,0).  NaN compares false and is replaced by 2^-126 here; s1 carries the NaN.
        const float c = __builtin_fmaxf(a, FLT_MIN);
        se += __builtin_amdgcn_frexp_expf(c);
        sl += (double)__builtin_amdgcn_logf(__builtin_amdgcn_frexp_mantf(c));
    }
}

// EC: acc = g + residual, stored back.  A 16-bit gradient is widened to fp32 first and acc is always stored (into
// the residual, or, without one, into the workspace's own buffer), because every later kernel reads fp32.
template <bool EC, int GT>
constexpr bool fit_writes() { return EC || GT != kGradF32; }

// Whether edges are for calls of M stages.  They ascend in every record; memory that holds none is refused here, and what
// ascends by chance serves a call as well as any.
__device__ __forceinline__ bool bands_usable(const Bands& e, int M)
{
    const float inf = __builtin_inff();
    const bool first = e.on == (uint32_t)M && e.lo[0] > 0.0f && e.lo[0] < e.hi[0] && e.hi[0] <= e.lo[1] && e.hi[0] < inf;
    const bool rest = M == 2 ? e.hi[1] == inf : e.lo[1] < e.hi[1] && e.hi[1] <= e.lo[2] && e.hi[1] < inf && e.hi[2] == inf;
    return first && rest;
}

// start of a call: per-call device state, by one thread
__device__ __forceinline__ void fit_reset_state(const Params& p)
{
    p.st->status_after[0] = 0;
    p.st->frozen_after[0] = 0;
    p.st->diag.stages = p.M;
    // Adapt_Stages bookkeeping: the pairs the previous call reported join the running count
    const unsigned long long prev_sel = p.st->selected_ctr;
    const unsigned long long prev_cap = (unsigned long long)p.st->prev_cap;
    p.st->khat_sum = p.acc_reset ? 0ull : p.st->khat_sum + (prev_sel < prev_cap ? prev_sel : prev_cap);
    // a window of a controller's count is only its own if every call since its start was that controller's
    if (p.acc_reset) p.st->disturbed = 0;
    else if (p.st->owner != p.owner) p.st->disturbed = 1;
    p.st->owner = p.owner;
    p.st->prev_cap = (long long)p.out_cap;
    p.st->selected_ctr = 0;
    p.st->overflow = 0;
    if (p.out_count) *p.out_count = 0;
    if (p.status_out) *p.status_out = 0;
    if (p.bands == kBandsUse) {
        p.st->band = p.st->band_next;
        if (!bands_usable(p.st->band_next, p.M)) p.st->band.on = 0;
    }
}

// one element through the guarded scalar path
template <int DIST, bool EC, int GT>
__device__ __forceinline__ float fit_one(const Params& p, int64_t i, double& s1, double& s2, double& sl, int& se)
{
    float c = load_grad1<GT>(p.grad, i);
    if (EC) c = c + p.acc_w[i];
    if (fit_writes<EC, GT>()) p.acc_w[i] = c;
    fit_accum<DIST>(c, s1, s2, sl, se);
    return c;
}

// the sums of one lane
template <int DIST>
struct FitSums {
    double s1 = 0.0, s2 = 0.0, sl = 0.0;
    int se = 0;
    __device__ __forceinline__ void tile(f4 c, uint32_t)
    {
        fit_accum<DIST>(c.x, s1, s2, sl, se);
        fit_accum<DIST>(c.y, s1, s2, sl, se);
        fit_accum<DIST>(c.z, s1, s2, sl, se);
        fit_accum<DIST>(c.w, s1, s2, sl, se);
    }
    __device__ __forceinline__ void one(bool valid, float c, int64_t)
    {
        if (valid) fit_accum<DIST>(c, s1, s2, sl, se);
    }
    __device__ __forceinline__ void end() {}
};

template <int DIST, bool EC, int GT, bool PAST = false>
__device__ __forceinline__ void fit_body(const Params& p, Blk b, const AccTile* first = nullptr)
{
    __shared__ double sh[kWavesPerBlock][4];
    const int lane = threadIdx.x & 63, wib = threadIdx.x >> 6;
    const uint32_t w = b.id * kWavesPerBlock + wib;
    FitSums<DIST> f;
    if (w < p.nwaves) acc_sweep<EC, fit_writes<EC, GT>(), GT, PAST>(p, w, lane, f, first);
    double v[3] = {f.s1, f.s2, f.sl + (double)f.se};
    wave_totals(v);
    if (lane == 0) {
        sh[wib][0] = v[0];
        sh[wib][1] = v[1];
        sh[wib][2] = v[2];
    }
    __syncthreads();
    if (threadIdx.x < 3) {
        double tot = 0.0;
#pragma unroll
        for (int i = 0; i < kWavesPerBlock; ++i) tot += sh[i][threadIdx.x];
        p.part_out[threadIdx.x * kBatchBlocks + b.id] = tot;
    }
    if (b.id == 0 && threadIdx.x == 0) fit_reset_state(p);
}

// ---------------------------------------------------------------------------------------------
// k_fit_flat + k_fit_reduce: the same pass for large vectors.  One float4 per thread and a grid that
// covers the vector in address order: the blocks in flight at any time touch one narrow window of each
// buffer, however long the vector is (see kFlatMinD for both shapes' times).
// Of every 2 MB an XCD has 256 KB in one piece, the piece behind its last one (piece_order; see acc_tile).  A training step
// with blocks in address order and so, us: 1 stage, 66 M elements 167.2 and 162.8, 138 M 373 and 361.5; 2 stages, 40 M, ratio 0.1
// 257.0 and 254.4; 3 stages, 25 M, 0.1 180.9 and 180.3; 4 stages, 66 M 274.1 and 271.9.  Pieces that stay 138 M 376, of 32 KB 389.
// The price is one partial sum per 256-thread block - far too many for every block of the next
// kernel to add up - so a second, small kernel folds them into the usual 512 slots, in a fixed order.
// ---------------------------------------------------------------------------------------------
// Place in address order of block i of n, GROUP of which cover 2 MB.
template <uint32_t GROUP>
__device__ __forceinline__ uint32_t piece_order(uint32_t i, uint32_t n)
{
    if ((i | (GROUP - 1)) >= n) return i;  // the last ones, which do not fill 2 MB
    return (i & ~(GROUP - 1)) + ((i + i / GROUP) & 7u) * (GROUP / 8) + (i & (GROUP - 1)) / 8;
}

template <int DIST, bool EC, int GT>
__global__ __launch_bounds__(kFlatBlock) void k_fit_flat(Params p, double* __restrict__ flat_part, uint32_t nflat)
{
    __shared__ double sh[kFlatBlock / 64][4];
    const int lane = threadIdx.x & 63, wib = threadIdx.x >> 6;
    const uint32_t place = piece_order<512>(blockIdx.x, nflat);
    const int64_t i = ((int64_t)place * kFlatBlock + threadIdx.x) * 4 - p.shift;  // first of the thread's 4 elements
    double s1 = 0.0, s2 = 0.0, sl = 0.0;
    int se = 0;
    if (i >= 0 && i + 4 <= p.d) {
        constexpr bool WRITE = fit_writes<EC, GT>();
        f4 c = load_grad4<GT, WRITE>(p.grad, (size_t)i);
        f4* a4 = reinterpret_cast<f4*>(p.acc_w + i);
        if (EC) c = c + *a4;
        if (WRITE) *a4 = c;
        fit_accum<DIST>(c.x, s1, s2, sl, se);
        fit_accum<DIST>(c.y, s1, s2, sl, se);
        fit_accum<DIST>(c.z, s1, s2, sl, se);
        fit_accum<DIST>(c.w, s1, s2, sl, se);
    } else {  // the vector's ends
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (i + j >= 0 && i + j < p.d) fit_one<DIST, EC, GT>(p, i + j, s1, s2, sl, se);
    }
    double v[3] = {s1, s2, sl + (double)se};
    wave_totals(v);
    if (lane == 0) {
        sh[wib][0] = v[0];
        sh[wib][1] = v[1];
        sh[wib][2] = v[2];
    }
    __syncthreads();
    if (threadIdx.x < 3) {
        double tot = 0.0;
#pragma unroll
        for (int w = 0; w < kFlatBlock / 64; ++w) tot += sh[w][threadIdx.x];
        flat_part[(size_t)threadIdx.x * nflat + place] = tot;
    }
}

// Slot s of the 512 receives the partial sums of the flat blocks [s * per, (s + 1) * per): one wave
// per slot, every lane adds its share in order, then the lanes are combined in a fixed order.
__global__ __launch_bounds__(kBlock) void k_fit_reduce(Params p, const double* __restrict__ flat_part, uint32_t nflat,
                                                       uint32_t per)
{
    const int lane = threadIdx.x & 63;
    const uint32_t slot = blockIdx.x * kWavesPerBlock + (threadIdx.x >> 6);
    const uint32_t b0 = slot * per, b1 = b0 + per < nflat ? b0 + per : nflat;
    double v[3] = {0.0, 0.0, 0.0};
    for (uint32_t b = b0 + lane; b < b1; b += 64) {
        v[0] += flat_part[b];
        if (p.dist == kDistGpd) v[1] += flat_part[(size_t)nflat + b];
        if (p.dist == kDistGamma) v[2] += flat_part[2 * (size_t)nflat + b];
    }
    wave_totals(v);
    if (lane == 0 && slot < (uint32_t)kMaxBlocks) {
        p.part_out[0 * kBatchBlocks + slot] = v[0];
        p.part_out[1 * kBatchBlocks + slot] = v[1];
        p.part_out[2 * kBatchBlocks + slot] = v[2];
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) fit_reset_state(p);
}

// ---------------------------------------------------------------------------------------------
// k_fit_bands: the first pass of a call that repeats the call before it in shape.  That call's thresholds, plus and
// minus a few times what they moved by between the calls before, are a band in which each of this call's thresholds is
// expected.  Besides the sums of the fit this pass forms, for every stage but the last, the sums of y = |x| - hi over the
// magnitudes above the band, and lists the entries inside the bands and above the last stage's lower edge.  If the stage's
// threshold then falls into its band - the stage's kernel checks - the exceedances are those sums, shifted to the
// threshold, and the band's entries above it: the vector is not read again.  If not, the kernel reads the vector as it
// would without bands.  The thresholds come from exact sums either way.
// Bound by HBM: the ten or so instructions more per element hide behind 12 bytes.  Since nothing reads the vector again
// soon, the residual goes past the caches, loads and stores: 25.6 M elements, three stages, three vectors in turn, first
// pass alone 50.7 us against 57.0 (with the loads or the stores alone 58.2 and 57.0), 66 M 135 against 142; a dense stage
// after such a pass would lose more than that (25.6 M, a call without bands 84.5 and 89.5).  A training step without and
// with bands, us: 14.7 M, 2 stages, ratio 0.001 55.5 and 46.3; 25.6 M, 3 stages 84.2 and 75.5, bf16 77.4 and 67.1; 30 M,
// fp16, 2 stages, 0.01 96.8 and 68.5; 66 M, gamma 171 and 148; 138 M, 3 stages, 0.01 518 and 409.  A call whose
// thresholds fall out of the bands pays for them, the more the longer the lists get; where the thresholds double or halve
// 25.6 M 88 and 100, 66 M 173 and 203, 100 M, 2 stages, 0.01 295 and 359, 138 M, 3 stages, 0.01 515 and 645, 0.001 405 and 461.
// ---------------------------------------------------------------------------------------------
// A band's half-width is the least one (see band_width in the host code) or, where that is more, kBandDrift times the
// threshold's last relative change, which later calls let shrink by kBandDecay each: what moves by 10 % every third
// call stays inside.  What would take more than kBandMaxWidth - a tenth of the vector in lists costs what the dense pass
// does, kBandLastWidest for the last stage, whose band has no upper edge - is a jump: the next call goes without bands (see
// Calm), and the widths do not grow by it.  Where a band would reach the next threshold (a carried residual grows light
// tails, in which the later thresholds draw together) the two meet half way, if that leaves both of them more room than
// their thresholds moved by: 138 M elements, 3 stages, ratio 0.001, one residual over 400 fresh gradients, us a call at the
// end 384 without bands, 416 when such calls went without them, 339 so.
constexpr float kBandDrift = 1.5f, kBandDecay = 0.87f, kBandLastWidest = 0.4f;
// A wave that lists more than one in kBandCrowd of its elements - their 16 bytes, written and read, are then what a dense
// pass reads - makes the vector rest as after jumps that come often: many entries share one magnitude near a threshold.
// Magnitudes 0 and s, 71.5 % of them s, without a residual, 66 M elements: 251 us a call without bands, 642 and with the
// rest 291.
constexpr uint32_t kBandCrowd = 4;
// The least width for short vectors (in a batch), whose thresholds are noisy: 99 % of the changes from call to call,
// relative and times the square root of the length, were within 4.4 (exponential) and 4 (GPD) for the first threshold and 6.6
// and 7.8 for the second, 6 to 19 and 8 to 20 with the gamma law (12 M to 66 M elements in 50 to 300 tensors).
constexpr float kBandNoise = 6.0f, kBandNoiseLater = 8.0f, kBandNoiseGamma = 3.0f;

// One thread of the last stage's kernel: bands for the next call from this one's thresholds.
__device__ void bands_record(const Params& p, float eta_last)
{
    if (p.bands == kBandsNone) return;
    DevState* st = p.st;
    Bands b;
    b.on = (uint32_t)p.M;
    float below = 0.0f;
    bool met = false;  // `below` is where the band before met this one
    const bool over = p.bands == kBandsUse && st->band_over != 0;
    st->band_over = 0;
    float eta_now[kBandStages], moved[kBandStages], most[kBandStages];
    bool jumped = false;
#pragma unroll
    for (int m = 0; m < kBandStages; ++m) {
        if (m >= p.M) continue;
        const bool last = m + 1 == p.M;
        eta_now[m] = last ? eta_last : st->diag.eta[m];
        most[m] = last ? kBandLastWidest : m == 0 ? p.band_max : kBandMaxWidth;
        moved[m] = 0.0f;
        if (p.bands == kBandsUse) moved[m] = kBandDrift * __builtin_fabsf(eta_now[m] - st->band_eta[m]) / st->band_eta[m];
        if (!(moved[m] <= most[m])) jumped = true;  // also what is not a number
    }
#pragma unroll
    for (int m = 0; m < kBandStages; ++m) {
        b.lo[m] = b.hi[m] = __builtin_inff();
        if (m >= p.M) continue;
        const bool last = m + 1 == p.M;
        const float eta = eta_now[m];
        const float spread = (m == 0 ? kBandNoise : kBandNoiseLater) * (p.dist == kDistGamma ? kBandNoiseGamma : 1.0f);
        float w = spread / __builtin_sqrtf((float)p.d);
        const float need = eta * __builtin_fmaxf(w, moved[m]);
        if (!last) w = __builtin_fminf(w, m == 0 ? kBandMaxWidthBatch : kBandMaxWidth);  // short vectors are a batch's
        w = __builtin_fmaxf(p.band_w[m], w);
        if (p.bands == kBandsUse) {
            if (!jumped) w = __builtin_fmaxf(w, moved[m]);
            // a captured call that has not run yet may have left no width at all
            w = __builtin_fmaxf(w, kBandDecay * __builtin_fminf(st->band_w[m], most[m]));
        }
        st->band_eta[m] = eta;
        st->band_w[m] = w;
        if (last && p.band_w[m] == 0.0f) continue;
        const float lo = __builtin_fmaxf(eta * (1.0f - w), below);
        float hi = last ? __builtin_inff() : eta * (1.0f + w);
        if (met && !(eta - below >= need)) b.on = 0;
        met = false;
        if (m + 1 < kBandStages && !last) {
            const float next = eta_now[m + 1];
            met = hi >= next && !(m + 2 == p.M && p.band_w[m + 1] == 0.0f);
            if (met) hi = eta + 0.5f * (next - eta);
            if (met && !(hi - eta >= need)) b.on = 0;
        }
        if (!((last || w <= most[m]) && eta > lo && eta < hi)) b.on = 0;  // also a threshold that is 0 or not finite
        below = hi;
        b.lo[m] = lo;
        b.hi[m] = hi;
    }
    Calm calm = {kCalmMost, kCalmMost};
    if (p.bands == kBandsUse) calm = calm_after(st->band_calm, jumped);
    if (over) calm = Calm{0, 0};
    if (!calm_enough(calm)) b.on = 0;
    st->band_calm = calm;
    st->band_next = b;
}

__device__ __forceinline__ float uniform(float v)
{
    return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v)));
}

template <int DIST, int NB>
struct FitBands {
    static constexpr bool kSquares = DIST != kDistExp;  // the later stages' fits are GPD then
    FitSums<DIST> f;
    float lo[NB], hi[NB], last;
    double y[NB], yy[NB];
    uint32_t n[NB];
    ListWriter lw;
    int lane;
    uint32_t shift;
    __device__ __forceinline__ void element(float x, int32_t idx)
    {
        const float a = __builtin_fabsf(x);
        // edges ascend: an entry above lo and not above hi of one band, or above the last edge, is above an odd number
        bool keep = a > last;
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const bool above = a > hi[b];
            keep = keep != ((a > lo[b]) != above);
            n[b] += (uint32_t)__popcll(__ballot(above));
            const double v = (double)(above ? a : hi[b]) - (double)hi[b];
            y[b] += v;
            if (kSquares) yy[b] = __builtin_fma(v, v, yy[b]);
        }
        list_push(lw, keep, idx, x, lane);
    }
    __device__ __forceinline__ void tile(f4 c, uint32_t t)
    {
        f.tile(c, t);
        const int32_t i0 = (int32_t)(t * kTile + lane * 4 - shift);
        element(c.x, i0 + 0);
        element(c.y, i0 + 1);
        element(c.z, i0 + 2);
        element(c.w, i0 + 3);
        list_flush(lw, lane);
    }
    __device__ __forceinline__ void one(bool valid, float c, int64_t i)
    {
        f.one(valid, c, i);
        element(c, (int32_t)i);  // zero where invalid: above no edge
    }
    __device__ __forceinline__ void end() { list_flush(lw, lane); }
};

template <int DIST, bool EC, int GT, int NB>
__device__ __forceinline__ void fit_bands_body(const Params& p, Blk b, const Bands& e, const AccTile* first)
{
    __shared__ double sh[kWavesPerBlock][3 + 3 * NB];
    __shared__ int2 ring[kWavesPerBlock][kRingSize];
    const int lane = threadIdx.x & 63, wib = threadIdx.x >> 6;
    const uint32_t w = b.id * kWavesPerBlock + wib;
    FitBands<DIST, NB> f;
#pragma unroll
    for (int k = 0; k < NB; ++k) {
        f.lo[k] = uniform(e.lo[k]);
        f.hi[k] = uniform(e.hi[k]);
        f.y[k] = f.yy[k] = 0.0;
        f.n[k] = 0;
    }
    f.last = uniform(e.lo[NB]);
    f.lane = lane;
    f.shift = p.shift;
    f.lw.list = p.band_seg + seg_begin(p, w < p.nwaves ? w : 0);
    f.lw.ring = ring[wib];
    f.lw.run = f.lw.fill = 0;
    if (w < p.nwaves) {
        acc_sweep<EC, fit_writes<EC, GT>(), GT, EC>(p, w, lane, f, first);
        const uint32_t n = list_finish(f.lw, lane);
        if (lane == 0) {
            p.band_cnt[w] = n;
            if (n > seg_slots(p, w) / kBandCrowd) p.st->band_over = 1;
        }
    }
    // per band y and y^2, and |x| with the law's second quantity
    constexpr int S = DIST == kDistExp ? 1 : 2;
    double w_sum[S * (NB + 1)];
    w_sum[0] = f.f.s1;
    if constexpr (DIST == kDistGpd) w_sum[1] = f.f.s2;
    if constexpr (DIST == kDistGamma) w_sum[1] = f.f.sl + (double)f.f.se;
#pragma unroll
    for (int k = 0; k < NB; ++k) {
        w_sum[S * (k + 1)] = f.y[k];
        if constexpr (S > 1) w_sum[S * (k + 1) + 1] = f.yy[k];
    }
    wave_totals(w_sum);
    double v[3 + 3 * NB];
    v[0] = w_sum[0];
    v[1] = DIST == kDistGpd ? w_sum[S - 1] : 0.0;
    v[2] = DIST == kDistGamma ? w_sum[S - 1] : 0.0;
#pragma unroll
    for (int k = 0; k < NB; ++k) {
        v[3 + 3 * k] = w_sum[S * (k + 1)];
        v[4 + 3 * k] = S > 1 ? w_sum[S * (k + 1) + S - 1] : 0.0;
        v[5 + 3 * k] = (double)f.n[k];
    }
    if (lane == 0) {
#pragma unroll
        for (int q = 0; q < 3 + 3 * NB; ++q) sh[wib][q] = v[q];
    }
    __syncthreads();
    if (threadIdx.x < 3 + 3 * NB) {
        double tot = 0.0;
#pragma unroll
        for (int i = 0; i < kWavesPerBlock; ++i) tot += sh[i][threadIdx.x];
        if (threadIdx.x < 3) p.part_out[threadIdx.x * kBatchBlocks + b.id] = tot;
        else p.band_part[(threadIdx.x - 3) * kMaxBlocks + b.id] = tot;
    }
    if (b.id == 0 && threadIdx.x == 0) fit_reset_state(p);
}

template <bool BANDS>
__device__ __forceinline__ BandEdges band_load(const Params& p)
{
    if constexpr (!BANDS) return BandEdges{};
    const int m = p.stage;
    return BandEdges{m == 1 ? p.st->band.on != 0 : p.st->band_live[m - 1] != 0, false, p.st->band.lo[m - 1], p.st->band.hi[m - 1],
                     0.0f};
}

// What a block of the first pass summed up above the band of this stage, shifted to the stage's threshold below it.
struct BandAbove {
    double y, yy, n;
};
__device__ __forceinline__ BandAbove band_above_load(const Params& p, Blk b)
{
    const double* q = p.band_part + (size_t)3 * (p.stage - 1) * kMaxBlocks + b.id;
    return BandAbove{q[0], q[kMaxBlocks], q[2 * kMaxBlocks]};
}
__device__ __forceinline__ BandAbove band_above_shift(BandAbove a, float hi, float eta)
{
    const double s = (double)hi - (double)eta;
    return BandAbove{a.y + a.n * s, a.yy + (2.0 * a.y + a.n * s) * s, a.n};
}

// ---------------------------------------------------------------------------------------------
// k_compact: statistics of the exceedances of eta_m for the next fit, and per-wave survivor lists
// ---------------------------------------------------------------------------------------------

// One component of a tile (64 candidates, one per lane).  Entries above eta_w go to the wave's list;
// entries above eta_s are counted (`ns`, wave-uniform) and enter the sums of y = |x| - eta_s.
// Comparisons are strict and fp32; NaN on either side is false.
template <bool STATS, bool WRITE>
__device__ __forceinline__ void emit(bool valid, float x, int32_t idx, float eta_s, float eta_w, ListWriter& lw,
                                     int lane, uint32_t& ns, double& sy, double& syy)
{
    const float a = __builtin_fabsf(x);
    if (WRITE) list_push(lw, valid && (a > eta_w), idx, x, lane);
    if (STATS) {
        // y = |x| - eta_s over the selected entries, exactly, and 0 elsewhere (eta_s - eta_s)
        const bool sel = valid && (a > eta_s);
        ns += (uint32_t)__popcll(__ballot(sel));
        const double y = (double)(sel ? a : eta_s) - (double)eta_s;
        sy += y;
        syy = __builtin_fma(y, y, syy);
    }
}

// one complete tile of the dense vector, already loaded
template <bool STATS, bool WRITE>
__device__ __forceinline__ void compact_tile(f4 a, uint32_t t, uint32_t shift, int lane, float eta_s, float eta_w,
                                             ListWriter& lw, uint32_t& ns, double& sy, double& syy)
{
    const int32_t i0 = (int32_t)(t * kTile + lane * 4 - shift);
    emit<STATS, WRITE>(true, a.x, i0 + 0, eta_s, eta_w, lw, lane, ns, sy, syy);
    emit<STATS, WRITE>(true, a.y, i0 + 1, eta_s, eta_w, lw, lane, ns, sy, syy);
    emit<STATS, WRITE>(true, a.z, i0 + 2, eta_s, eta_w, lw, lane, ns, sy, syy);
    emit<STATS, WRITE>(true, a.w, i0 + 3, eta_s, eta_w, lw, lane, ns, sy, syy);
    if (WRITE) list_flush(lw, lane);
}

// `a` holds the wave's first kAhead tiles, requested before the threshold was known: a stage kernel's prologue is
// a cold round trip for the partial sums plus a few hundred dependent fp64 instructions in which the memory pipes
// would otherwise run dry.  From then on tile j + kAhead is requested before tile j is processed.
// One tile (1 KB per wave, 16 KB per CU) is enough: 1, 2 and 4 measured alike at 14.7 M, 25.6 M and 138 M elements.
constexpr int kAhead = 1;

template <bool STATS, bool WRITE, bool KEEP = false>
__device__ __forceinline__ void compact_dense(const Params& p, const WaveTiles& wt, const DenseSweep& d, f4 (&a)[kAhead],
                                              int lane, float eta_s, float eta_w, ListWriter& lw, uint32_t& ns, double& sy,
                                              double& syy)
{
#pragma unroll 1
    for (uint32_t j = 0; j < d.nb; j += kAhead) {
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            if (j + u < d.nb) {  // wave-uniform
                const f4 c = a[u];
                a[u] = dense_load<KEEP>(d, j + u + kAhead, lane);
                compact_tile<STATS, WRITE>(c, dense_tile(d, j + u), p.shift, lane, eta_s, eta_w, lw,
                                           ns, sy, syy);
            }
        }
    }
    for (uint32_t g = 0; g < wt.n - wt.nb; ++g) {
        const uint32_t t = wt.w + guarded_tile(wt, g) * wt.W;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int64_t i = (int64_t)t * kTile + lane * 4 + j - p.shift;
            const bool valid = i >= 0 && i < p.d;
            const float v = valid ? p.acc[i] : 0.0f;
            emit<STATS, WRITE>(valid, v, (int32_t)i, eta_s, eta_w, lw, lane, ns, sy, syy);
        }
        if (WRITE) list_flush(lw, lane);
    }
}

// Two list entries per lane and load (16 B): slot i of a wave's list holds entries 2i and 2i+1.
// `cap2` is the number of slots the wave's segment has room for; slots past the list's end hold
// stale data and are masked by `n_in`.
template <int U>
__device__ __forceinline__ void load_slots(int4 (&q)[U], const int4* __restrict__ src4, uint32_t c, uint32_t cap2,
                                           int lane)
{
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const uint32_t i = c + u * 64 + lane;
        q[u] = i < cap2 ? src4[i] : make_int4(0, 0, 0, 0);
    }
}

template <bool STATS, int U>
__device__ __forceinline__ void compact_slots(const int4 (&q)[U], uint32_t c, uint32_t n_in, int lane, float eta,
                                              ListWriter& lw, uint32_t& ns, double& sy, double& syy)
{
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const uint32_t e = 2 * (c + u * 64 + lane);
        emit<STATS, true>(e < n_in, __int_as_float(q[u].y), q[u].x, eta, eta, lw, lane, ns, sy, syy);
        emit<STATS, true>(e + 1 < n_in, __int_as_float(q[u].w), q[u].z, eta, eta, lw, lane, ns, sy, syy);
        if (u & 1) list_flush(lw, lane);  // every 4 components = at most kTile entries
    }
    static_assert(U % 2 == 0, "flush check after every second slot group");
}

// End of a stage kernel: per block, the number of exceedances of eta_m (the n of the next fit) - or,
// without statistics (dense last stage), the number of list entries (k_gather's prefix) - and the
// block's partial sums of y and y^2, each in its fixed slot.
// BANDS: `above` joins them.
template <bool STATS, bool BANDS = false>
__device__ __forceinline__ void stage_epilogue(const Params& p, Blk b, int lane, int wib, uint32_t count, double sy,
                                               double syy, double (*sh)[4], uint32_t* sh_cnt, BandAbove above = BandAbove{})
{
    if (lane == 0) sh_cnt[wib] = count;
    if (STATS) {
        double v[2] = {sy, syy};
        wave_totals(v);
        if (lane == 0) {  // the prologue is done with sh
            sh[wib][0] = v[0];
            sh[wib][1] = v[1];
        }
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t tot = 0;
#pragma unroll
        for (int i = 0; i < kWavesPerBlock; ++i) tot += sh_cnt[i];
        if (BANDS) tot += (uint32_t)above.n;
        p.blk_out[b.id] = tot;
    }
    if (STATS && threadIdx.x < 2) {
        double tot = 0.0;
#pragma unroll
        for (int i = 0; i < kWavesPerBlock; ++i) tot += sh[i][threadIdx.x];
        if (BANDS) tot += threadIdx.x == 0 ? above.y : above.yy;
        p.part_out[threadIdx.x * kBatchBlocks + b.id] = tot;
    }
}

// A stage whose threshold fell into its band: the band's entries above the threshold.  `q0` and `q1` hold the list's
// first 64 slots and the 64 after them.
template <int U>
__device__ __forceinline__ void band_sums(const int4* __restrict__ src4, uint32_t cap2, uint32_t n, int4 q0, int4 q1, int lane,
                                          float eta, float hi, uint32_t& ns, double& sy, double& syy)
{
    ListWriter none;
    auto entry = [&](bool in, int v) {
        const float x = __int_as_float(v);
        emit<true, false>(in && __builtin_fabsf(x) <= hi, x, 0, eta, eta, none, lane, ns, sy, syy);
    };
    const uint32_t e = 2 * lane;
    entry(e < n, q0.y);
    entry(e + 1 < n, q0.w);
    entry(e + 128 < n, q1.y);
    entry(e + 129 < n, q1.w);
#pragma unroll 1
    for (uint32_t c = 128; c < (n + 1) / 2; c += 64 * U) {
        int4 q[U];
        load_slots<U>(q, src4, c, cap2, lane);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint32_t f = 2 * (c + u * 64 + lane);
            entry(f < n, q[u].y);
            entry(f + 1 < n, q[u].w);
        }
    }
}

// What a batch's first pass with bands left for a block of the first stage's kernel (see k_fit_flat_batched).
struct ChunkPart {
    const double* above;  // sums of y, y^2 and 1 above the band, `stride` apart, one of each for every chunk
    uint32_t stride, n;   // chunks of the block
    const uint32_t* cnt;
    const int2* list;
};

// k_compact: a stage that reads the dense vector.  STATS: form the sums for the next stage's fit.
// WRITE: append the entries above eta_w to this stage's lists (eta_w = eta_m, or a candidate threshold
// above it); a stage whose candidates would still be a large fraction only counts and sums.  KEEP: with ordinary loads,
// which leave the vector in the memory-side cache (see keeps_much in the host code).  BANDS: behind a first pass with
// bands, which this stage may be able to do with; the head of the wave's list is then requested beside its first tile,
// since waiting to know which of them it will be costs more than reading both.  CHUNKS: the same for a batch, whose first
// pass leaves a list for every chunk of the block's range; their heads are requested only if the tensor has bands, which
// the wave knows by the time its first tiles are on their way.
template <bool STATS, bool WRITE, bool FLAT = false, bool KEEP = false, bool BANDS = false, bool CHUNKS = false>
__device__ __forceinline__ void compact_body(const Params& p, Blk b, const FlatPart& fp = FlatPart{},
                                             const ChunkPart& cp = ChunkPart{})
{
    __shared__ double sh[kWavesPerBlock][4];
    __shared__ uint32_t sh_cnt[kWavesPerBlock];
    __shared__ int2 ring[WRITE ? kWavesPerBlock : 1][kRingSize];
    const int lane = threadIdx.x & 63, wib = threadIdx.x >> 6;
    const uint32_t w = b.id * kWavesPerBlock + wib;
    const bool active = w < p.nwaves;
    const WaveTiles wt = wave_tiles(p, active ? w : 0);

    // Neither the prologue's own loads nor the first loads of the body depend on the threshold.  The
    // prologue's go first (the memory counter retires in order: behind the tiles they would wait for
    // them), then the first tiles, so that the stream runs while the partial sums are reduced and the
    // closed form is evaluated.
    BandEdges band = {};
    if constexpr (BANDS || CHUNKS) band = band_load<true>(p);
    constexpr int SUMS = FLAT ? kSumsBlock : CHUNKS ? kSumsStaged : kSumsWave;
    const PrologueLoads g = prologue_load<SUMS>(p, b, false);
    FlatLoads f;
    if constexpr (FLAT) f = flat_load(fp, p.dist);
    double share[3] = {0.0, 0.0, 0.0};
    if constexpr (SUMS == kSumsStaged) {
        if (threadIdx.x < p.nblocks) {
            share[0] = p.part_in[threadIdx.x];
            share[1] = p.part_in[(size_t)second_row(p.dist, 1) * kBatchBlocks + threadIdx.x];
        }
    }
    if constexpr (CHUNKS) {
        band.over = band.live && p.st->band_over != 0;
        band.live = band.live && !band.over;
        band.cand = p.st->band.lo[1];
    }
    const DenseSweep d = dense_sweep(p, wt, p.reverse != 0, p.seg_out);
    f4 a[kAhead];
#pragma unroll
    for (int u = 0; u < kAhead; ++u) a[u] = dense_load<KEEP>(d, u, lane);
    const int4* src4 = nullptr;
    int4 q0 = {}, q1 = {};
    uint32_t n_in = 0;
    BandAbove above = {};
    if constexpr (BANDS) {
        src4 = reinterpret_cast<const int4*>(p.band_seg + seg_begin(p, active ? w : 0));
        q0 = src4[lane];
        n_in = active ? p.band_cnt[w] : 0u;
        q1 = src4[64 + lane];  // a wave owns several tiles
        above = band_above_load(p, b);
    }
    constexpr int U = CHUNKS ? 4 : 1;  // lists a wave requests at once, the first ones before the threshold is known
    int2 head[U];
    uint32_t len[U];
    uint32_t step = 1;
    auto chunk_heads = [&](uint32_t x0) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint32_t x = x0 + u * step;
            const bool have = active && x < cp.n;
            len[u] = have ? cp.cnt[x] : 0u;
            head[u] = cp.list[(have ? x : 0u) * kChunkList + lane];
        }
    };
    if constexpr (CHUNKS) {
        step = p.nwaves - b.id * kWavesPerBlock;  // the block's waves that have a list to write to
        if (step > kWavesPerBlock) step = kWavesPerBlock;
        if (band.live) {
            chunk_heads(wib);
            for (uint32_t x = threadIdx.x; x < cp.n; x += kBlock) {
                above.y += cp.above[x];
                above.yy += cp.above[x + cp.stride];
                above.n += cp.above[x + 2 * (size_t)cp.stride];
            }
        }
    }
    if constexpr (FLAT) flat_sums(fp, f, share);
    static_assert(!CHUNKS || (WRITE && sizeof(ring) >= 2 * kMaxBlocks * sizeof(double)), "room for the staged sums");
    double* const staged = reinterpret_cast<double*>(ring);  // nobody's before the threshold is known

    const StageEta se = prologue_finish<SUMS>(p, b, false, g, band, &share, sh, staged);

    uint32_t run = 0, ns = 0;
    double sy = 0.0, syy = 0.0;
    if constexpr (BANDS) {
        if (b.id == 0 && threadIdx.x == 0) p.st->band_live[p.stage] = se.hit ? 1u : 0u;
        if (se.hit) {
            if (active)
                band_sums<4>(src4, seg_slots(p, w) / 2, __builtin_amdgcn_readfirstlane(n_in), q0, q1, lane, se.eta, band.hi,
                             ns, sy, syy);
            stage_epilogue<STATS, true>(p, b, lane, wib, ns, sy, syy, sh, sh_cnt, band_above_shift(above, band.hi, se.eta));
            return;
        }
    }
    if constexpr (CHUNKS) {
        if (se.hit) {
            if (active) {
                ListWriter lw;
                lw.list = p.seg_out + seg_begin(p, w);
                lw.ring = ring[wib];
                lw.run = lw.fill = 0;
                auto entry = [&](bool in, int2 e) {
                    const float x = __int_as_float(e.y), m = __builtin_fabsf(x);
                    list_push(lw, in && m > se.eta_w, e.x, x, lane);
                    emit<true, false>(in && m <= band.hi, x, 0, se.eta, se.eta, lw, lane, ns, sy, syy);
                };
                auto chunk = [&](uint32_t x, uint32_t n, int2 first) {
                    n = __builtin_amdgcn_readfirstlane(n);
                    entry((uint32_t)lane < n, first);
                    for (uint32_t c = 64; c < n; c += 64) entry(c + lane < n, cp.list[x * kChunkList + c + lane]);
                    list_flush(lw, lane);
                };
                for (uint32_t x = wib;;) {
#pragma unroll
                    for (int u = 0; u < U; ++u) chunk(x + u * step, len[u], head[u]);
                    x += U * step;
                    if (x >= cp.n) break;
                    chunk_heads(x);
                }
                const uint32_t n = list_finish(lw, lane);
                if (lane == 0) p.cnt_out[w] = n;
            }
            above = band_above_shift(above, band.hi, se.eta);
            ns += (uint32_t)wave_sum(above.n);  // counts: exact
            stage_epilogue<STATS>(p, b, lane, wib, ns, sy + above.y, syy + above.yy, sh, sh_cnt);
            return;
        }
    }
    if (active) {
        ListWriter lw;
        lw.list = p.seg_out + seg_begin(p, w);  // room for every element of the wave's tiles
        lw.ring = ring[WRITE ? wib : 0];
        lw.run = lw.fill = 0;
        compact_dense<STATS, WRITE, KEEP>(p, wt, d, a, lane, se.eta, se.eta_w, lw, ns, sy, syy);
        if (WRITE) run = list_finish(lw, lane);
        if (lane == 0) p.cnt_out[w] = run;
    }
    stage_epilogue<STATS>(p, b, lane, wib, STATS ? ns : run, sy, syy, sh, sh_cnt);
}

// ---------------------------------------------------------------------------------------------
// k_lists: a stage m < M whose source is the producer's survivor lists, or, if those are candidate
// lists that do not reach down to this stage's threshold (see stage_prologue), the dense vector.
// The lists are short (a few per cent of the vector at most) and the kernel is bound by latency and
// by the launch itself: every wave takes the list of the same wave of the kernel before it, and its
// first 128 entries are loaded before the prologue.
// ---------------------------------------------------------------------------------------------
template <bool BANDS = false>
__device__ __forceinline__ void lists_body(const Params& p, Blk b)
{
    __shared__ double sh[kWavesPerBlock][4];
    __shared__ uint32_t sh_cnt[kWavesPerBlock];
    __shared__ int2 ring[kWavesPerBlock][kRingSize];
    constexpr int U = 4;
    const int lane = threadIdx.x & 63, wib = threadIdx.x >> 6;
    const uint32_t w = b.id * kWavesPerBlock + wib;
    const bool active = w < p.nwaves;
    const size_t seg = seg_begin(p, active ? w : 0);
    const int2* src = p.seg_in;
    const uint32_t* cnt = p.cnt_in;
    const BandEdges band = band_load<BANDS>(p);  // names the lists: the first round trip, beside the prologue's
    const PrologueLoads g = prologue_load(p, b, true);
    if (band.live) {
        src = p.band_seg;
        cnt = p.band_cnt;
    }
    const int4* __restrict__ src4 = reinterpret_cast<const int4*>(src + seg);
    const uint32_t cap2 = seg_slots(p, active ? w : 0) / 2;  // at least 128: a wave owns a tile
    uint32_t n_in = active ? cnt[w] : 0u;
    const int4 q0 = src4[lane];
    int4 q1 = {};
    BandAbove above = {};
    if constexpr (BANDS) {
        q1 = src4[64 + lane];
        above = band_above_load(p, b);
    }

    const StageEta se = prologue_finish(p, b, true, g, band);
    const float eta = se.eta;

    uint32_t ns = 0;
    double sy = 0.0, syy = 0.0;
    if constexpr (BANDS) {
        if (b.id == 0 && threadIdx.x == 0) p.st->band_live[p.stage] = se.hit ? 1u : 0u;
        if (se.hit) {
            if (active) band_sums<U>(src4, cap2, __builtin_amdgcn_readfirstlane(n_in), q0, q1, lane, eta, band.hi, ns, sy, syy);
            stage_epilogue<true, true>(p, b, lane, wib, ns, sy, syy, sh, sh_cnt, band_above_shift(above, band.hi, eta));
            return;
        }
    }
    if (active) {
        ListWriter lw;
        lw.list = p.seg_out + seg;
        lw.ring = ring[wib];
        lw.run = lw.fill = 0;
        if (!se.lists_ok) {
            // this stage's exceedances straight from the dense vector
            const WaveTiles wt = wave_tiles(p, w);
            const DenseSweep d = dense_sweep(p, wt, p.reverse != 0, p.seg_out);
            f4 a[kAhead];
#pragma unroll
            for (int u = 0; u < kAhead; ++u) a[u] = dense_load(d, u, lane);
            compact_dense<true, true>(p, wt, d, a, lane, eta, eta, lw, ns, sy, syy);
        } else {
            n_in = __builtin_amdgcn_readfirstlane(n_in);
            const uint32_t nslot = (n_in + 1) / 2;
            const uint32_t e = 2 * lane;
            emit<true, true>(e < n_in, __int_as_float(q0.y), q0.x, eta, eta, lw, lane, ns, sy, syy);
            emit<true, true>(e + 1 < n_in, __int_as_float(q0.w), q0.z, eta, eta, lw, lane, ns, sy, syy);
            // the rest, 256 slots per step
            for (uint32_t c = 64; c < nslot; c += 64 * U) {
                int4 q[U];
                load_slots<U>(q, src4, c, cap2, lane);
                compact_slots<true, U>(q, c, n_in, lane, eta, lw, ns, sy, syy);
            }
        }
        const uint32_t n_out = list_finish(lw, lane);
        if (lane == 0) p.cnt_out[w] = n_out;
    }
    stage_epilogue<true>(p, b, lane, wib, ns, sy, syy, sh, sh_cnt);
}

// ---------------------------------------------------------------------------------------------
// k_final_lists: last stage when its source is a set of survivor lists (M >= 2).
// Threshold eta_M, selection, contiguous output and residual update in one kernel.  If the lists are
// candidate lists that turn out not to reach down to eta_M (see stage_prologue), the same two passes
// run over the dense vector instead: slower, same result.  The lists are
// short by now and the kernel is bound by memory latency, not bandwidth: every wave takes up to
// kFinalGroup lists at a time and issues all their loads together, before the prologue, so that the
// whole kernel is a few dependent round trips.  Each block reserves its output range with ONE atomic
// add on the pair counter (same-address atomics cost ~11 ns each on this chip: a hundred of them are
// cheaper than another kernel boundary).  The set of pairs is deterministic; the order of the
// blocks' ranges in the output is not.
// ---------------------------------------------------------------------------------------------
constexpr int kFinalGroup = 4;

struct FinalList {
    const int4* src4;  // the list, two entries per slot
    uint32_t cap2;     // slots the segment has room for
    uint32_t n;        // entries
};

__device__ __forceinline__ FinalList final_list(const Params& p, const int2* seg, const uint32_t* cnt, uint32_t sw, bool valid)
{
    FinalList l;
    const uint32_t w = valid ? sw : 0;
    l.src4 = reinterpret_cast<const int4*>(seg + seg_begin(p, w));
    l.cap2 = seg_slots(p, w) / 2;
    l.n = valid ? cnt[w] : 0u;
    return l;
}

// exceedances among the two entries of this lane's slot `slot` (wave-wide count)
__device__ __forceinline__ uint32_t final_count(int4 q, uint32_t slot, uint32_t n, float eta)
{
    const uint32_t e = 2 * slot;
    const bool s0 = e < n && __builtin_fabsf(__int_as_float(q.y)) > eta;
    const bool s1 = e + 1 < n && __builtin_fabsf(__int_as_float(q.w)) > eta;
    return (uint32_t)__popcll(__ballot(s0)) + (uint32_t)__popcll(__ballot(s1));
}

// writes the exceedances of this lane's slot at the wave's running position `pos`
__device__ __forceinline__ void final_emit(const Params& p, int4 q, uint32_t slot, uint32_t n, float eta,
                                           unsigned long long cap, unsigned long long& pos)
{
    const uint32_t e = 2 * slot;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int32_t idx = h ? q.z : q.x;
        const float x = __int_as_float(h ? q.w : q.y);
        const bool sel = e + h < n && __builtin_fabsf(x) > eta;
        const unsigned long long mask = __ballot(sel);
        const unsigned long long at = pos + lane_prefix(mask);
        if (sel && at < cap) {  // pairs beyond the capacity stay in the residual
            p.out_idx[at] = idx;
            p.out_val[at] = x;
            if (p.residual) p.residual[idx] = 0.0f;
        }
        pos += (unsigned long long)__popcll(mask);
    }
}

// Dense fallback of the two passes over the tiles of source wave sw.  f(values, index of the first) for four
// consecutive elements per lane, the wave together; elements outside the vector come as zeros, which are never above
// a threshold.  kFallbackAhead tiles are requested at a time: a wave has up to four source waves' tiles to itself here,
// and one round trip per 64 elements, as it was, took 330 us for a tensor of 83 K elements in a batch.
constexpr int kFallbackAhead = 4;

template <typename F>
__device__ __forceinline__ void fallback_sweep(const Params& p, uint32_t sw, int lane, F f)
{
    const WaveTiles wt = wave_tiles(p, sw);
    const DenseSweep d = dense_sweep(p, wt, false, p.seg_out);
#pragma unroll 1
    for (uint32_t j = 0; j < d.nb; j += kFallbackAhead) {
        f4 a[kFallbackAhead];
#pragma unroll
        for (int u = 0; u < kFallbackAhead; ++u) a[u] = dense_load(d, j + u, lane);
#pragma unroll
        for (int u = 0; u < kFallbackAhead; ++u)
            if (j + u < d.nb) f(a[u], (int64_t)dense_tile(d, j + u) * kTile + lane * 4 - p.shift);  // wave-uniform
    }
#pragma unroll 1
    for (uint32_t g = 0; g < wt.n - wt.nb; ++g) {
        const int64_t i = (int64_t)(wt.w + guarded_tile(wt, g) * wt.W) * kTile + lane * 4 - p.shift;
        f4 a;
#pragma unroll
        for (int j = 0; j < 4; ++j) a[j] = i + j >= 0 && i + j < p.d ? p.acc[i + j] : 0.0f;
        f(a, i);
    }
}

__device__ __forceinline__ uint32_t final_count_dense(const Params& p, uint32_t sw, int lane, float eta)
{
    uint32_t c = 0;
    fallback_sweep(p, sw, lane, [&](f4 a, int64_t) {
#pragma unroll
        for (int j = 0; j < 4; ++j) c += (uint32_t)__popcll(__ballot(__builtin_fabsf(a[j]) > eta));
    });
    return c;
}

__device__ __forceinline__ void final_emit_dense(const Params& p, uint32_t sw, int lane, float eta,
                                                 unsigned long long cap, unsigned long long& pos)
{
    fallback_sweep(p, sw, lane, [&](f4 a, int64_t i) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const bool sel = __builtin_fabsf(a[j]) > eta;
            const unsigned long long mask = __ballot(sel);
            const unsigned long long at = pos + lane_prefix(mask);
            if (sel && at < cap) {  // pairs beyond the capacity stay in the residual
                p.out_idx[at] = (int32_t)(i + j);
                p.out_val[at] = a[j];
                if (p.residual) p.residual[i + j] = 0.0f;
            }
            pos += (unsigned long long)__popcll(mask);
        }
    });
}

// The call's threshold and status, by the thread that has recorded the stage.
__device__ __forceinline__ void final_results(const Params& p, float eta)
{
    *p.out_eta = eta;
    const uint32_t status = p.st->status_after[p.M];
    p.st->diag.status = status;
    if (p.status_out && status) atomicOr(p.status_out, status);
}

// The last stage's first block of a single call: it selects nothing, but evaluates the threshold once more and keeps what is
// kept of the call.  The records' own loads and divisions held the block back that made them beside its selection, and the
// kernel ends with its last block: a training step of 25.6 M elements, 3 stages 71.8 -> 71.4 us, with a bf16 gradient 65.0 -> 64.2;
// 2 stages as before.
template <bool BANDS>
__device__ __forceinline__ void final_record(const Params& p, Blk b)
{
    const BandEdges band = band_load<BANDS>(p);
    const float eta = stage_prologue(p, b, true, band).eta;
    if (threadIdx.x == 0) final_results(p, eta);
    __syncthreads();
    if (threadIdx.x == kBlock - 64) bands_record(p, eta);
    if (threadIdx.x == kBlock - 128) hint_record(p, eta);
}

template <bool BANDS = false>
__device__ __forceinline__ void final_body(const Params& p, Blk b)
{
    __shared__ uint32_t sh_cnt[kWavesPerBlock];
    __shared__ unsigned long long sh_base;
    constexpr int K = kFinalGroup;
    const int lane = threadIdx.x & 63, wib = threadIdx.x >> 6;
    // source lists of this wave: first, first + 8, first + 16, first + 24 (below last): the launchers give a
    // block at most kFinalGroup * 8 = 32 source lists, so one group of loads covers them all
    const uint32_t per_block = (p.nwaves + b.n - 1) / b.n;
    const uint32_t first = b.id * per_block + wib;
    const uint32_t last = min(p.nwaves, (b.id + 1) * per_block);

    const BandEdges band = band_load<BANDS>(p);  // names the lists: the first round trip, beside the prologue's
    const PrologueLoads g = prologue_load(p, b, true);
    const int2* seg = band.live ? p.band_seg : p.seg_in;
    const uint32_t* cnt = band.live ? p.band_cnt : p.cnt_in;
    // first group of lists: counts and first 64 slots of each (128 behind a first pass with bands, whose lists hold what
    // the stages before needed as well), all loads issued together and before the threshold (none depends on it)
    constexpr int H = BANDS ? 2 : 1;
    FinalList l0[K];
    int4 q0[K][H];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const uint32_t sw = first + k * kWavesPerBlock;
        l0[k] = final_list(p, seg, cnt, sw, sw < last);
#pragma unroll
        for (int h = 0; h < H; ++h) {
            const uint32_t i = h * 64 + lane;
            q0[k][h] = i < l0[k].cap2 && (h == 0 || band.live) ? l0[k].src4[i] : make_int4(0, 0, 0, 0);
        }
    }

    const StageEta se = prologue_finish(p, b, true, g, band);
    const float eta = se.eta;
    const bool from_lists = se.lists_ok || se.hit;

    // pass A: count
    uint32_t mine = 0;
    if (!from_lists) {
        for (uint32_t sw = first; sw < last; sw += kWavesPerBlock) mine += final_count_dense(p, sw, lane, eta);
    } else {
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const uint32_t n = __builtin_amdgcn_readfirstlane(l0[k].n);
#pragma unroll
        for (int h = 0; h < H; ++h)
            if (h == 0 || band.live) mine += final_count(q0[k][h], h * 64 + lane, n, eta);
        for (uint32_t c = band.live ? 64 * H : 64; c < (n + 1) / 2; c += 64) {
            const uint32_t i = c + lane;
            const int4 q = i < l0[k].cap2 ? l0[k].src4[i] : make_int4(0, 0, 0, 0);
            mine += final_count(q, i, n, eta);
        }
    }
    }
    if (lane == 0) sh_cnt[wib] = mine;
    __syncthreads();
    uint32_t off = 0, tot = 0;
#pragma unroll
    for (int i = 0; i < kWavesPerBlock; ++i) {
        if (i < wib) off += sh_cnt[i];
        tot += sh_cnt[i];
    }
    const unsigned long long cap = (unsigned long long)p.out_cap;
    if (threadIdx.x == 0) {
        const unsigned long long base = atomicAdd(&p.st->selected_ctr, (unsigned long long)tot);
        sh_base = base;
        const unsigned long long end = base + tot;
        atomicMax(p.out_count, (int32_t)(end < cap ? end : cap));
        if (end > cap) {
            p.st->overflow = 1u;  // every writer stores the same value
            if (p.status_out) atomicOr(p.status_out, kStOverflow);
        }
        if (b.records) final_results(p, eta);
    }
    // by other waves, beside the round trip of the reservation
    if (b.records && threadIdx.x == kBlock - 64) bands_record(p, eta);
    if (b.records && threadIdx.x == kBlock - 128) hint_record(p, eta);
    __syncthreads();
    unsigned long long pos = sh_base + off;

    // pass B: same traversal, now writing; the first group is still in registers
    if (!from_lists) {
        for (uint32_t sw = first; sw < last; sw += kWavesPerBlock) final_emit_dense(p, sw, lane, eta, cap, pos);
        return;
    }
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const uint32_t n = __builtin_amdgcn_readfirstlane(l0[k].n);
#pragma unroll
        for (int h = 0; h < H; ++h)
            if (h == 0 || band.live) final_emit(p, q0[k][h], h * 64 + lane, n, eta, cap, pos);
        for (uint32_t c = band.live ? 64 * H : 64; c < (n + 1) / 2; c += 64) {
            const uint32_t i = c + lane;
            const int4 q = i < l0[k].cap2 ? l0[k].src4[i] : make_int4(0, 0, 0, 0);
            final_emit(p, q, i, n, eta, cap, pos);
        }
    }
}

// ---------------------------------------------------------------------------------------------
// k_eta + k_select: last stage of a call that keeps so much of a long vector that lists would not pay (see
// select_dense in the host code).  k_eta, one block, evaluates eta_M; the blocks of k_select start in address order,
// each takes kSelectTiles tiles per wave into registers, reserves its output range with one atomic and writes the pairs
// and the tiles back with the selected entries zeroed.  Whole lines, where clearing the entries one by one leaves
// lines that are written in part, and the pairs come in nearly ascending order, which the scatter that follows
// profits from.  The set of pairs is deterministic, the order of the blocks' ranges is not.  Bound by HBM: at 138 M
// elements and a ratio of 0.1 204 us for 1.22 GB, the scatter 243; k_final_lists took 235, the dense stage that wrote its
// lists 30 more than one that only sums, and the scatter 270.  Loads that go past the caches want stores that do so as
// well (all but those of a vector that the caches hold): a training step of 138 M, 3 stages, with ordinary and with such
// stores 863 and 835 us, 90 M 576 and 547, 70 M, 2 stages 431 and 408.  XCDs have pieces of 256 KB (piece_order): 138 M 812 and
// 808, 66 M, 2 stages 385.2 and 383.5.
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(kBlock) void k_eta(Params p)
{
    const StageEta se = stage_prologue(p, whole_grid(), false);
    if (threadIdx.x == 0) {
        *p.out_eta = se.eta;
        const uint32_t status = p.st->status_after[p.M];  // written by this thread in the prologue
        p.st->diag.status = status;
        if (p.status_out && status) *p.status_out = status;
        bands_record(p, se.eta);
    }
}

// WHOLE: all tiles of the block are complete.  KEEP: ordinary loads (see keeps_much in the host code)
template <bool WHOLE, bool KEEP>
__device__ __forceinline__ void select_body(const Params& p, uint32_t first, uint32_t* sh_cnt, uint32_t* sh_base)
{
    constexpr int kWaves = kSelectBlock / 64;
    const int lane = threadIdx.x & 63, wib = threadIdx.x >> 6;
    const uint32_t t0 = first + wib * kSelectTiles;
    f4 a[kSelectTiles];
#pragma unroll
    for (int u = 0; u < kSelectTiles; ++u) {
        const int64_t i = (int64_t)(t0 + u) * kTile + lane * 4 - p.shift;
        if constexpr (WHOLE && KEEP) {
            a[u] = *reinterpret_cast<const f4*>(p.acc + i);
        } else if constexpr (WHOLE) {
            a[u] = __builtin_nontemporal_load(reinterpret_cast<const f4*>(p.acc + i));
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) a[u][j] = i + j >= 0 && i + j < p.d ? p.acc[i + j] : 0.0f;  // 0 is never above eta
        }
    }
    const float eta = p.st->diag.eta[p.M - 1];
    uint32_t mine = 0;
#pragma unroll
    for (int u = 0; u < kSelectTiles; ++u)
#pragma unroll
        for (int j = 0; j < 4; ++j) mine += (uint32_t)__popcll(__ballot(__builtin_fabsf(a[u][j]) > eta));
    if (lane == 0) sh_cnt[wib] = mine;
    __syncthreads();
    uint32_t pos = 0, total = 0;
#pragma unroll
    for (int i = 0; i < kWaves; ++i) {
        if (i < wib) pos += sh_cnt[i];
        total += sh_cnt[i];
    }
    const uint32_t cap = (uint32_t)p.out_cap;
    if (threadIdx.x == 0) {
        const unsigned long long base = atomicAdd(&p.st->selected_ctr, (unsigned long long)total);
        *sh_base = (uint32_t)base;
        const unsigned long long end = base + total;
        atomicMax(p.out_count, (int32_t)(end < cap ? end : cap));
        if (end > cap) {
            p.st->overflow = 1u;  // every writer stores the same value
            if (p.status_out) atomicOr(p.status_out, kStOverflow);
        }
    }
    __syncthreads();
    pos += *sh_base;  // at most d: 32 bits hold it
#pragma unroll
    for (int u = 0; u < kSelectTiles; ++u) {
        const int64_t i = (int64_t)(t0 + u) * kTile + lane * 4 - p.shift;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const float x = a[u][j];
            const bool sel = __builtin_fabsf(x) > eta;
            const unsigned long long mask = __ballot(sel);
            const uint32_t at = pos + lane_prefix(mask);
            if (sel && at < cap) {  // pairs beyond the capacity stay in the residual
                p.out_idx[at] = (int32_t)(i + j);
                p.out_val[at] = x;
                a[u][j] = 0.0f;
            }
            pos += (uint32_t)__popcll(mask);
        }
        if (p.residual) {
            if constexpr (WHOLE) {
                if constexpr (KEEP) *reinterpret_cast<f4*>(p.residual + i) = a[u];
                else __builtin_nontemporal_store(a[u], reinterpret_cast<f4*>(p.residual + i));
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (i + j >= 0 && i + j < p.d) p.residual[i + j] = a[u][j];
            }
        }
    }
}

template <bool KEEP>
__global__ __launch_bounds__(kSelectBlock) void k_select(Params p)
{
    __shared__ uint32_t sh_cnt[kSelectBlock / 64];
    __shared__ uint32_t sh_base;
    constexpr uint32_t kTiles = kSelectBlock / 64 * kSelectTiles;
    const uint32_t place = piece_order<32>(blockIdx.x, gridDim.x);
    const uint32_t first = (p.reverse ? gridDim.x - 1 - place : place) * kTiles;
    if (first + kTiles <= p.nfull && (first > 0 || p.shift == 0)) select_body<true, KEEP>(p, first, sh_cnt, &sh_base);
    else select_body<false, KEEP>(p, first, sh_cnt, &sh_base);
}

// ---------------------------------------------------------------------------------------------
// k_gather: survivor lists of the last stage -> contiguous (index, value) output; residual update.
// Used when the last stage read the dense vector (M = 1): no atomics, output order is fixed.
// ---------------------------------------------------------------------------------------------
__device__ __forceinline__ void gather_body(const Params& p, Blk b)
{
    __shared__ unsigned long long sh_u[kWavesPerBlock][2];
    const int lane = threadIdx.x & 63, wib = threadIdx.x >> 6;
    const uint32_t t = threadIdx.x;
    const uint32_t w = b.id * kWavesPerBlock + wib;
    const uint32_t w0 = b.id * kWavesPerBlock;
    const bool active = w < p.nwaves;
    // independent loads first: block counts, the block's wave counts, this wave's count and first entries
    const unsigned long long c = t < p.nblocks ? (unsigned long long)p.blk_in[t] : 0ull;
    uint32_t mine = (lane < wib && w0 + lane < p.nwaves) ? p.cnt_in[w0 + lane] : 0u;
    uint32_t n_in = active ? p.cnt_in[w] : 0u;
    const int2* __restrict__ src = p.seg_in + seg_begin(p, active ? w : 0);
    const int2 first = src[lane];

    // exclusive prefix of the per-block counts at this block, and their total
    unsigned long long below = wave_sum_u64(t < b.id ? c : 0ull);
    unsigned long long total = wave_sum_u64(c);
    if (lane == 0) {
        sh_u[wib][0] = below;
        sh_u[wib][1] = total;
    }
    __syncthreads();
    below = 0;
    total = 0;
#pragma unroll
    for (int i = 0; i < kWavesPerBlock; ++i) {
        below += sh_u[i][0];
        total += sh_u[i][1];
    }
    const unsigned long long cap = (unsigned long long)p.out_cap;
    if (b.id == 0 && t == 0) {
        *p.out_count = (int32_t)(total > cap ? cap : total);
        *p.out_eta = p.st->diag.eta[p.M - 1];
        p.st->selected_ctr = total;
        p.st->overflow = total > cap ? 1u : 0u;
        const uint32_t status = p.st->status_after[p.M];
        p.st->diag.status = status;
        if (p.status_out) *p.status_out = status | (total > cap ? kStOverflow : 0u);
    }
    if (!active) return;
    // offset of this wave inside the block: counts of the block's earlier waves
#pragma unroll
    for (int o = 4; o > 0; o >>= 1) mine += __shfl_down(mine, o, 64);  // lanes 0..7 only carry data
    const unsigned long long base = below + __builtin_amdgcn_readfirstlane(mine);
    n_in = __builtin_amdgcn_readfirstlane(n_in);
    for (uint32_t i = lane; i < n_in; i += 64) {
        const unsigned long long pos = base + i;
        if (pos < cap) {  // pairs beyond the capacity stay in the residual
            const int2 q = i < 64 ? first : src[i];
            p.out_idx[pos] = q.x;
            p.out_val[pos] = __int_as_float(q.y);
            if (p.residual) p.residual[q.x] = 0.0f;
        }
    }
}

// ---------------------------------------------------------------------------------------------
// k_small: a whole call in one block of 1024 threads, for a vector short enough for one CU.  A call
// of several kernels on such a vector is all launches, prologues and drains; here a stage is a sweep over registers or
// LDS, a sum over the block and the closed form.  All loads of a thread are in flight at once: one round trip to HBM.
// Fifteen waves hold the vector in registers.  Once the first threshold
// is known a wave lists what exceeds it in LDS, and everything after that reads the lists: their sums, the later stages,
// the selection.  (A wave whose exceedances are many or outgrow its list goes on with all of its elements.)  The sixteenth
// wave evaluates the closed forms; while the data are on their way it runs through the first stage's for nothing, and ahead
// of it, if there are several stages, through a later stage's, so that their code is in the instruction cache when the sums
// arrive (not for the gamma law, see small_evaluate).
// What bounds it is a serial chain on one CU, and instructions that are not in the cache: code that a call does not run
// through costs it nothing, but what it does run through costs more unrolled than as a loop, and so do rows of registers that
// a short vector does not fill.  In a graph, us, with the vector in LDS, every sweep and the selection over all of it and one wave
// of sixteen evaluating; with registers and lists; and so: 30011 elements, GPD, 3 stages, ratio 0.01 16.5, 13.4 and 13.2; 1000
// elements, exponential law, 1 stage 3.93, 4.18 and 3.40; 12000, gamma, 2 stages, 0.1 10.2, 11.0 and 10.5; 36000, exponential, 1
// stage, 0.5 12.1, 13.8 and 10.9.  With the residual stored as it was formed the last wave had its data 2700 cycles later;
// with a branch around every element's way to the list the lists took 6300 cycles, 5500 without.
// The sums, the thresholds and the order of the output are fixed.
// 24 kernels: the law; 16 bits or 32 (a kernel of its own for each 16-bit type and for calls without residual made 36, and a process's first
// call took 7.0 ms, now 4.4); N of 1, 4 and 10, and for the longest vectors WHOLE.
// ---------------------------------------------------------------------------------------------

// A data wave's share of the vector: N float4s per lane.
template <int DIST, int N>
struct SmallShare {
    f4 c[N];  // zeros past the end of the vector

    // f(valid, value, index), the wave together
    template <typename F>
    __device__ __forceinline__ void each(int32_t t, int32_t d, F f) const
    {
#pragma unroll
        for (int u = 0; u < N; ++u) {
            const int32_t i = 4 * (u * kSmallData + t);
            if (4 * u * kSmallData < d) {  // uniform
#pragma unroll
                for (int j = 0; j < 4; ++j) f(i + j < d, c[u][j], i + j);
            }
        }
    }
};

// Sums of y = |x| - eta and y^2 over what exceeds eta, and their number, of one wave.
template <int DIST>
struct SmallSums {
    double y = 0.0, yy = 0.0;
    uint32_t n = 0;  // wave-uniform
    __device__ __forceinline__ void add(bool valid, float x, float eta)
    {
        const float a = __builtin_fabsf(x);
        const bool sel = valid && a > eta;
        n += (uint32_t)__popcll(__ballot(sel));
        const double v = (double)(sel ? a : eta) - (double)eta;
        y += v;
        if constexpr (DIST != kDistExp) yy = __builtin_fma(v, v, yy);
    }
};

// The wave that evaluates the closed forms.  `sh`: the data waves' sums.
template <int DIST>
__device__ __forceinline__ void small_evaluate(Params& p, int lane, const double (*sh)[4], const uint32_t* sh_cnt, float* sh_eta)
{
    const double d = (double)p.d;
    PrologueLoads g = {};
    g.seen = __builtin_nanf("");
    __builtin_amdgcn_s_setprio(3);  // the others wait for it
    StageEta r = {};
    auto stage = [&](int m, bool dry) {
        StageSums sums = {d, DIST == kDistGamma ? -d : 3.0 * d, d};  // mean 1, variance 2
        g.eta_prev = dry ? 1.0f : r.eta;
        if (!dry) {
            __syncthreads();
            double v[3];
#pragma unroll
            for (int q = 0; q < 3; ++q) v[q] = lane < kSmallWaves - 1 ? sh[lane][q] : 0.0;
            wave_totals(v);
            sums = StageSums{v[0], v[1], v[2]};
        }
        p.stage = m;
        p.L_stage = stage_L(p, m - 1);
        StageRecord rec;
        r = stage_eval(p, false, g, sums, rec);
        if (dry) return;
        if (lane == 0) *sh_eta = r.eta;
        __syncthreads();
        if (m == 1 && lane == 0) fit_reset_state(p);
        g.status = rec.status;
        g.frozen = rec.frozen;
        if (lane == 0) stage_record(p, r, rec);
    };
    if constexpr (DIST == kDistGamma) {
        // lgamma's constants, hoisted out of a loop, would not fit the registers: the first stage on its own, no dry runs
        stage(1, false);
#pragma unroll 1
        for (int m = 2; m <= p.M; ++m) {
            __builtin_assume(m >= 2);
            stage(m, false);
        }
    } else {
#pragma unroll 1
        for (int it = p.M > 1 ? -1 : 0; it <= p.M; ++it) {
            int m = it > 0 ? it : (it < 0 ? 2 : 1);  // ahead of the stages the second one's form and the first one's
            asm volatile("" : "+s"(m));
            stage(m, it <= 0);
        }
    }
    __syncthreads();  // the data waves' counts
    uint32_t total = 0;
#pragma unroll
    for (int i = 0; i < kSmallWaves - 1; ++i) total += sh_cnt[i];
    const uint32_t cap = (uint32_t)p.out_cap;
    if (lane == 0) {
        *p.out_count = (int32_t)(total > cap ? cap : total);
        *p.out_eta = r.eta;
        p.st->selected_ctr = total;
        p.st->overflow = total > cap ? 1u : 0u;
        p.st->diag.status = g.status;
        if (p.status_out) *p.status_out = g.status | (total > cap ? kStOverflow : 0u);
    }
}

// A list pays for a selection of up to a quarter of the wave's share (36000 elements, exponential law, 2 stages, ratio 0.15 with
// an eighth 16.3 us, so 13.1, a third the same), and for the sums of a later stage while up to 96 of the
// first row's 256 elements exceed the first threshold (the gamma law keeps more than it is asked for: 20000 elements, 2 stages,
// ratio 0.1 with lists of whatever length 16.0 us, so 14.6; up to 144 of 256 the same).
constexpr uint32_t kSmallMuch = 4, kSmallMost = 96;
// A call of one stage with a ratio above 0.15 makes no lists at all and stores the residual once, when it has selected: 36000
// elements, exponential law, with lists and without, ratio 0.16 10.2 us and 10.9, 0.2 10.7 and 10.9, 0.25 13.7 and 10.9; 0.5, with
// lists that are given up, 12.6 and 10.9.
constexpr double kSmallWhole = 1.9;  // log(1 / 0.15)

// A data wave.  `list`: room for kSmallList<N> pairs.  HALF: the gradient is of 16 bits.  WHOLE: a call without lists; where N
// <= 4 one kernel does both.
template <int DIST, bool HALF, int N, bool WHOLE>
__device__ __forceinline__ void small_data(const Params& p, int lane, int wib, int2* list, double (*sh)[4], uint32_t* sh_cnt,
                                           const float* sh_eta)
{
    const int32_t t = wib * 64 + lane, d = (int32_t)p.d;
    const bool ec = p.residual != nullptr;
    typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));
    SmallShare<DIST, N> x;
    // the last, incomplete float4 is its owner's, element by element; past the end the last element again
    const int32_t tail = d & ~3;
    const bool owner = tail < d && (tail >> 2) % kSmallData == t;
    const bool f16 = HALF && p.gt == kGradF16;
    float rest[3], rest_r[3] = {0.0f, 0.0f, 0.0f};
    if (owner) {
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            const int32_t i = tail + j < d ? tail + j : d - 1;
            if constexpr (HALF) rest[j] = f16 ? load_grad1<kGradF16>(p.grad, i) : load_grad1<kGradBf16>(p.grad, i);
            else rest[j] = load_grad1<kGradF32>(p.grad, i);
            if (ec) rest_r[j] = p.residual[i];
        }
    }
    if (d >= 4) {
        // whole float4s, wherever the buffers start; past the end the last one again: the loads stay unconditional
        typedef uint32_t u2 __attribute__((ext_vector_type(2), aligned(2)));
        typedef std::conditional_t<HALF, u2, f4u> Raw;
        Raw raw[N];
#pragma unroll
        for (int u = 0; u < N; ++u) {
            const int32_t i = 4 * (u * kSmallData + t);
            const size_t at = (size_t)(i + 4 <= d ? i : d - 4) * (HALF ? 2 : 4);
            raw[u] = __builtin_nontemporal_load(reinterpret_cast<const Raw*>(reinterpret_cast<const char*>(p.grad) + at));
        }
        auto widen = [&] {
            if constexpr (!HALF) {
#pragma unroll
                for (int u = 0; u < N; ++u) x.c[u] = raw[u];
            } else if (f16) {
#pragma unroll
                for (int u = 0; u < N; ++u) x.c[u] = widen4<kGradF16>(raw[u]);
            } else {
#pragma unroll
                for (int u = 0; u < N; ++u) x.c[u] = widen4<kGradBf16>(raw[u]);
            }
        };
        if (ec) {
            f4 r[N];
#pragma unroll
            for (int u = 0; u < N; ++u) {
                const int32_t i = 4 * (u * kSmallData + t);
                r[u] = *reinterpret_cast<const f4u*>(p.residual + (i + 4 <= d ? i : d - 4));
            }
            widen();
#pragma unroll
            for (int u = 0; u < N; ++u) x.c[u] = x.c[u] + r[u];
        } else {
            widen();
        }
    }
    f4 end = {0.0f, 0.0f, 0.0f, 0.0f};
    if (owner) {
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            if (tail + j >= d) continue;
            end[j] = rest[j];
            if (ec) {
                end[j] = rest[j] + rest_r[j];
                p.residual[tail + j] = end[j];
            }
        }
    }
#pragma unroll
    for (int u = 0; u < N; ++u) {
        const int32_t i = 4 * (u * kSmallData + t);
        if (i + 4 > d) x.c[u] = i < d ? end : f4{0.0f, 0.0f, 0.0f, 0.0f};
    }

    auto sums_out = [&](double a, double b, double n) {
        double v[2] = {a, b};
        wave_totals(v);
        if (lane == 0) {
            sh[wib][0] = v[0];
            sh[wib][1] = v[1];
            sh[wib][2] = n;
        }
        __syncthreads();
    };
    {
        double s1 = 0.0, s2 = 0.0, sl = 0.0;
        int se = 0;
        x.each(t, d, [&](bool valid, float v, int32_t) {
            if (DIST != kDistGamma || valid) fit_accum<DIST>(v, s1, s2, sl, se);  // zeros leave s1 and s2 alone
        });
        sums_out(s1, DIST == kDistGamma ? sl + (double)se : s2, 0.0);
    }
    const bool whole = N > 4 ? WHOLE : p.M == 1 && p.L_stage < kSmallWhole;
    if (ec && !whole) {  // while the closed form is evaluated: ahead of that the stores would hold other waves' loads back
#pragma unroll
        for (int u = 0; u < N; ++u) {
            const int32_t i = 4 * (u * kSmallData + t);
            if (i + 4 <= d) *reinterpret_cast<f4u*>(p.residual + i) = x.c[u];
        }
    }
    __syncthreads();
    float eta = *sh_eta;
    uint32_t pos = 0;  // the wave's next place in the output
    auto positions = [&](uint32_t mine) {
        if (lane == 0) sh_cnt[wib] = mine;
        __syncthreads();  // also between the residual's stores and the clearing
#pragma unroll
        for (int i = 0; i < kSmallWaves - 1; ++i) pos += i < wib ? sh_cnt[i] : 0u;
    };
    const uint32_t cap = (uint32_t)p.out_cap;
    // writes what is selected of 64 entries; whether the lane's was
    auto emit_pairs = [&](bool in, float v, int32_t i) {
        const bool sel = in && __builtin_fabsf(v) > eta;
        const unsigned long long mask = __ballot(sel);
        const uint32_t at = pos + lane_prefix(mask);
        const bool out = sel && at < cap;  // pairs beyond the capacity stay in the residual
        if (out) {
            p.out_idx[at] = i;
            p.out_val[at] = v;
        }
        pos += (uint32_t)__popcll(mask);
        return out;
    };
    // the float4 `c`, of whose entries those that are selected go to the output and become zero
    auto emit_row = [&](f4 c, int32_t i) {
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (emit_pairs(true, c[j], i + j)) c[j] = 0.0f;
        if (!ec) return;
        if (i + 4 <= d) {
            *reinterpret_cast<f4u*>(p.residual + i) = c;
        } else {
#pragma unroll
            for (int j = 0; j < 3; ++j)
                if (i + j < d) p.residual[i + j] = c[j];
        }
    };
    if (__builtin_expect(whole, 0)) {
        uint32_t n = 0;
        x.each(t, d, [&](bool, float v, int32_t) { n += (uint32_t)__popcll(__ballot(__builtin_fabsf(v) > eta)); });
        positions(n);
#pragma unroll
        for (int u = 0; u < N; ++u)
            if (4 * u * kSmallData < d) emit_row(x.c[u], 4 * (u * kSmallData + t));  // uniform
        return;
    }
    // what exceeds the first threshold
    constexpr uint32_t kRoom = kSmallList<N> - 64;
    // where all of a wave's share has room and the law keeps to its ratio no list is given up: 15360 elements 5.20 us, 5.28 with
    // the code for it
    constexpr bool kMayGiveUp = N > 4 || (N > 1 && DIST == kDistGamma);
    uint32_t len = 0;
#pragma unroll
    for (int u = 0; u < N; ++u) {
        const int32_t i = 4 * (u * kSmallData + t);
        if (4 * u * kSmallData >= d || (kMayGiveUp && len > kRoom)) continue;  // uniform; a list that is too short is none
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const bool sel = __builtin_fabsf(x.c[u][j]) > eta;
            const unsigned long long mask = __ballot(sel);
            // every lane writes, without a branch: what is not selected, or does not fit, to the places behind the list
            const uint32_t at = min(len, kRoom) + lane_prefix(mask);
            list[sel ? at : kSmallList<N> - 1] = make_int2(i + j, __float_as_int(x.c[u][j]));
            len += (uint32_t)__popcll(mask);
        }
        if (kMayGiveUp && u == 0 && len > kSmallMost) len = kRoom + 1;
    }
    const bool listed = !kMayGiveUp || len <= kRoom;
    // Where the list does not serve the elements take its room, the lane's own in rows: what goes through them is a loop then
    // (30011 elements, GPD, 3 stages, with that code unrolled over the registers 13.5 us, so 13.2)
    static_assert(kSmallList<N> * sizeof(int2) >= N * 64 * sizeof(f4), "room for the wave's share");
    f4* const rows = reinterpret_cast<f4*>(list) + lane;
    auto rows_store = [&] {
#pragma unroll
        for (int u = 0; u < N; ++u) rows[u * 64] = x.c[u];
    };
    if (!listed) rows_store();
    // the lane's entries among the first 64 * kHead of the list stay in registers; stale past the list's end
    constexpr int kHead = N > 1 ? 8 : 4;
    int2 head[kHead];
#pragma unroll
    for (int u = 0; u < kHead; ++u) head[u] = list[u * 64 + lane];
    // f(valid, value, index) for those, the wave together: from the list, or, if it is none, from all elements
    auto exceeding = [&](auto f) {
        if (listed) {
#pragma unroll
            for (uint32_t u = 0; u < kHead; ++u)
                if (u * 64 < len) f(u * 64 + lane < len, __int_as_float(head[u].y), head[u].x);
#pragma unroll 1
            for (uint32_t k = 64 * kHead; k < len; k += 128) {
                const int2 e = list[k + lane], g = list[k + 64 + lane];
                f(k + lane < len, __int_as_float(e.y), e.x);
                f(k + 64 + lane < len, __int_as_float(g.y), g.x);
            }
        } else {
#pragma unroll 1
            for (int u = 0; 4 * u * kSmallData < d; ++u) {
                const f4 c = rows[u * 64];
#pragma unroll
                for (int j = 0; j < 4; ++j) f(true, c[j], 4 * (u * kSmallData + t) + j);
            }
        }
    };
#pragma unroll 1
    for (int m = 2; m <= p.M; ++m) {
        SmallSums<DIST> q;
        exceeding([&](bool in, float v, int32_t) { q.add(in, v, eta); });
        sums_out(q.y, q.yy, (double)q.n);
        __syncthreads();
        eta = *sh_eta;
    }

    uint32_t mine = len;
    if (p.M > 1 || !listed) {
        mine = 0;
        exceeding([&](bool in, float v, int32_t) { mine += (uint32_t)__popcll(__ballot(in && __builtin_fabsf(v) > eta)); });
    }
    positions(mine);
    // A wave that selects much of its share, or has no list, goes through its elements once more and stores whole float4s: one
    // by one the cleared entries of 12000 elements, gamma law, of which it keeps 31 %, cost 3 us more (see kSmallMuch).
    if (listed && mine * kSmallMuch <= (uint32_t)(d / (kSmallWaves - 1))) {
        exceeding([&](bool in, float v, int32_t i) {
            if (emit_pairs(in, v, i) && ec) p.residual[i] = 0.0f;
        });
        return;
    }
    if (listed) rows_store();
#pragma unroll 1
    for (int u = 0; 4 * u * kSmallData < d; ++u) emit_row(rows[u * 64], 4 * (u * kSmallData + t));
}

// N: float4s per lane of a data wave, 4 * kSmallData * N >= d
template <int DIST, bool HALF, int N, bool WHOLE>
__global__ __launch_bounds__(kSmallBlock) void k_small(Params p)
{
    extern __shared__ __align__(16) int2 lists[];  // kSmallList<N> for each data wave
    __shared__ double sh[kSmallWaves - 1][4];
    __shared__ uint32_t sh_cnt[kSmallWaves - 1];
    __shared__ float sh_eta;
    const int lane = threadIdx.x & 63, wib = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    p.theta = 0.0f;  // no candidate lists
    p.dist = DIST;
    // Both sides pass the same barriers: two for every stage, one ahead of the output.
    if (wib == kSmallWaves - 1) small_evaluate<DIST>(p, lane, sh, sh_cnt, &sh_eta);
    else small_data<DIST, HALF, N, WHOLE>(p, lane, wib, lists + wib * kSmallList<N>, sh, sh_cnt, &sh_eta);
}

// ---------------------------------------------------------------------------------------------
// k_scatter_add: the step after the sparsifier in Algorithm 2 - a worker's (index, value) pairs are
// added into the dense aggregate, dense[idx[i]] += scale * val[i].  The indices of one list are
// distinct, so plain read-modify-write needs no atomics and the result is deterministic; lists of
// several workers are added by consecutive launches.  Product and sum are fused: one rounding per element.
// Bound by the lines that long lists touch.  Pairs that fill the L2 caches (half of their 32 MB) are read past them, as the dense lines
// need the room: 13.8 M pairs in 138 M elements, alone, 1024 blocks, ordinary and non-temporal loads 270 and 267 us, 8192
// blocks 257 and 254; 4 M 127 and 114, 3.5 M 98 and 90; but a list that the caches may still hold 1.4 M 46 and 50, 0.3 M 9.4 and
// 13.3.  Non-temporal loads or stores of the dense lines are slower (390, 268 at 8192 blocks), and four pairs per thread change
// nothing.
// ---------------------------------------------------------------------------------------------
constexpr int64_t kScatterStream = 1 << 21;  // pairs
__global__ __launch_bounds__(kBlock) void k_scatter_add(float* __restrict__ dense, int64_t d, const int32_t* __restrict__ idx,
                                                        const float* __restrict__ val, const int32_t* __restrict__ count,
                                                        int64_t capacity, float scale, uint32_t* __restrict__ bad)
{
    int64_t n = (int64_t)*count;
    if (n > capacity) n = capacity;
    const int64_t stride = (int64_t)gridDim.x * kBlock;
    auto add = [&](auto stream) {
        constexpr bool STREAM = decltype(stream)::value;
        for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n; i += stride) {
            const int64_t j = (int64_t)(STREAM ? __builtin_nontemporal_load(idx + i) : idx[i]);
            if (j < 0 || j >= d) {  // never written; reported
                atomicOr(bad, 1u);
                continue;
            }
            dense[j] = fmaf(scale, STREAM ? __builtin_nontemporal_load(val + i) : val[i], dense[j]);
        }
    };
    if (n >= kScatterStream) add(std::true_type());
    else add(std::false_type());
}

__global__ void k_clear_u32(uint32_t* p) { *p = 0; }

// a fill kernel rather than a memset: callers may record the stream into a HIP graph
void launch_clear_u32(uint32_t* p, hipStream_t s) { hipLaunchKernelGGL(k_clear_u32, dim3(1), dim3(1), 0, s, p); }

// Blocks: as many as run at once, or, where the buffers have room for a list that is long enough to gain by it, several times as
// many, so that blocks that fall behind do not end last.  With 1024, 4096 and 8192 blocks 13.8 M pairs take 267, 259 and 254 us, a
// training step of 138 M elements, ratio 0.1 859, 851 and 846; 4 M pairs 114, 113 and 113; but 100 pairs in long buffers
// 2.1, 3.3 and 5.0, and 138000 4.7, 4.7 and 6.3: such calls pay 3 us, of a step of 380 and more.
constexpr int64_t kScatterBlocks = 2 * kMaxBlocks, kScatterBlocksLong = 16 * kMaxBlocks, kScatterLong = 8000000;
void launch_scatter_add(float* dense, int64_t d, const int32_t* idx, const float* val, const int32_t* count,
                        int64_t capacity, float scale, uint32_t* bad, hipStream_t s)
{
    // the list length is only known on the device: a thread for every place of the capacity, capped; idle blocks exit at
    // once.  Top-k's capacity is its length, and with four places per thread that was 13 blocks for 25557 pairs, each
    // a chain of four updates: 7.1 us, against 4.0 for as many pairs in four times the capacity.
    int64_t blocks = (capacity + kBlock - 1) / kBlock;
    if (blocks < 1) blocks = 1;
    const int64_t most = capacity < kScatterLong ? kScatterBlocks : kScatterBlocksLong;
    if (blocks > most) blocks = most;
    hipLaunchKernelGGL(k_scatter_add, dim3((uint32_t)blocks), dim3(kBlock), 0, s, dense, d, idx, val, count, capacity,
                       scale, bad);
}

// ---------------------------------------------------------------------------------------------
// kernels: one call on one vector (the grid is the vector's), or a batch of vectors in one launch
// (every block belongs to one vector and finds that vector's arguments in a table on the device)
// ---------------------------------------------------------------------------------------------
// Arguments of this block's vector in a batched launch.  final_grid: the launch uses the last stage's
// (smaller) grid.
__device__ __forceinline__ Params batch_params(const BatchArgs& a, bool final_grid, Blk& b, uint32_t gb = blockIdx.x)
{
    const uint32_t t = __builtin_amdgcn_readfirstlane((uint32_t)(final_grid ? a.tb->fmap[gb] : a.tb->map[gb]));
    const TensorDesc& ds = a.tb->desc[t];
    Params p = {};
    p.grad = reinterpret_cast<const char*>(a.grad) + ds.offset * (a.gt == kGradF32 ? 4 : 2);
    p.gt = a.gt;
    p.residual = a.residual ? a.residual + ds.offset : nullptr;
    p.acc_w = p.residual ? p.residual : (a.acc_own ? a.acc_own + ds.offset : nullptr);
    p.acc = p.acc_w ? p.acc_w : reinterpret_cast<const float*>(p.grad);
    p.d = ds.d;
    p.shift = (uint32_t)((uintptr_t)p.acc >> 2) & (uint32_t)(kGrid - 1);
    p.nfull = (uint32_t)((ds.d + p.shift) / kTile);
    p.nwaves = ds.nwaves;
    p.tq = ds.tq;
    p.tr = ds.tr;
    p.nblocks = ds.nblocks;
    p.reverse = a.reverse;
    p.acc_reset = 1;
    p.dist = a.dist;
    p.M = a.M;
    p.stage = a.stage;
#pragma unroll
    for (int m = 0; m < SIDCO_MAX_STAGES; ++m) p.L[m] = a.L[m];
    p.L_stage = a.L_stage;
    p.L_next = a.L_next;
    p.theta = a.theta;
    p.theta_min = a.theta_min;
    p.use_hint = a.use_hint;
    p.cand_stage = a.cand_stage;
    p.st = &a.tb->st[t];
    p.part_in = a.part[a.in] + ds.first_block;
    p.part_out = a.part[a.out] + ds.first_block;
    p.cnt_in = a.cnt[a.in] + ds.first_block * kWavesPerBlock;
    p.cnt_out = a.cnt[a.out] + ds.first_block * kWavesPerBlock;
    p.blk_in = a.blk[a.in] + ds.first_block;
    p.blk_out = a.blk[a.out] + ds.first_block;
    p.seg_in = a.seg[a.in] + ds.seg_off;
    p.seg_out = a.seg[a.out] + ds.seg_off;
    p.out_idx = a.out_idx + ds.out_offset;
    p.out_val = a.out_val + ds.out_offset;
    p.out_count = a.out_counts + ds.index;
    p.out_eta = a.out_etas + ds.index;
    p.out_cap = ds.out_cap;
    p.bands = a.bands;
#pragma unroll
    for (int m = 0; m < kBandStages; ++m) p.band_w[m] = a.band_w[m];
    p.band_max = kBandMaxWidthBatch;
    b.id = gb - (final_grid ? ds.first_final : ds.first_block);
    b.n = final_grid ? ds.nfinal : ds.nblocks;
    b.none = 0;
    b.records = b.id == 0;
    return p;
}

// Tiles of block b of a vector's dense grid: those of its (at most) kWavesPerBlock waves.
__device__ __forceinline__ void block_tiles(const Params& p, Blk b, uint32_t& T0, uint32_t& T1)
{
    const uint32_t w0 = b.id * kWavesPerBlock;
    const uint32_t w1 = w0 + kWavesPerBlock < p.nwaves ? w0 + kWavesPerBlock : p.nwaves;
    T0 = w0 < p.nwaves ? tile_begin(p, w0) : 0;
    T1 = w0 < p.nwaves ? tile_begin(p, w1) : 0;
}

template <int DIST, bool EC, int GT>
__global__ __launch_bounds__(kBlock, 4) void k_fit(Params p) { fit_body<DIST, EC, GT>(p, whole_grid()); }
// PAST: the sweep goes past the caches without bands too (see launch_fit_bands)
template <int DIST, bool EC, int GT, int NB, bool PAST>
__global__ __launch_bounds__(kBlock, 4) void k_fit_bands(Params p)
{
    // the edges were written at the end of the call before: a round trip, and the first tile is requested ahead of it
    // (from kBandMinD elements on every wave has several)
    const AccTile first =
        acc_first<EC, fit_writes<EC, GT>(), GT, EC>(p, blockIdx.x * kWavesPerBlock + (threadIdx.x >> 6), threadIdx.x & 63);
    const Bands e = p.st->band_next;
    if (bands_usable(e, NB + 1)) fit_bands_body<DIST, EC, GT, NB>(p, whole_grid(), e, &first);
    else fit_body<DIST, EC, GT, PAST>(p, whole_grid(), &first);
}
template <bool STATS, bool WRITE, bool KEEP, bool BANDS>
__global__ __launch_bounds__(kBlock, 4) void k_compact(Params p)
{
    compact_body<STATS, WRITE, false, KEEP, BANDS>(p, stage_grid(p));
}
template <bool BANDS>
__global__ __launch_bounds__(kBlock, 4) void k_lists(Params p)
{
    lists_body<BANDS>(p, stage_grid(p));
}
template <bool BANDS>
__global__ __launch_bounds__(kBlock) void k_final_lists(Params p)
{
    Blk b = stage_grid(p);
    b.records = blockIdx.x == 0;
    if (b.records) {
        final_record<BANDS>(p, b);
        return;
    }
    --b.id;
    --b.n;
    final_body<BANDS>(p, b);
}
__global__ __launch_bounds__(kBlock) void k_gather(Params p) { gather_body(p, whole_grid()); }

template <int DIST, bool EC, int GT>
__global__ __launch_bounds__(kBlock) void k_fit_batched(BatchArgs a)
{
    Blk b;
    const Params p = batch_params(a, false, b);
    fit_body<DIST, EC, GT>(p, b);
}
// The first pass of a batch in the flat shape (see k_fit_flat): blockIdx.y is a block of the batch's dense grid
// - it names the vector and, within it, the tiles that block's waves own - and blockIdx.x a chunk of
// kFlatChunk = 8 of those tiles, two per wave (a block's look into the batch's table is a chain of two round trips
// ahead of its data; 161 tensors, 25.6 M elements, with one, two and four tiles per wave: 86.1, 84.1 and 87.5 us).  Blocks run in the order x first, then y: address
// order.  Chunks past the end of a y's tiles leave zeros and exit (the host launches the flat shape only when few
// are).
// `pieces`: of every 256 blocks an XCD has 32 that follow each other (see piece_order).
// BANDS: behind a call of the same layout (see k_fit_bands).  Every chunk also leaves the sums above the first stage's band
// and a list of the band's entries and of all that the second stage may ask for; the first stage's kernel writes its lists
// from that, and the later stages are those of any batch.  The per-wave shape with bands was slower (66 M elements in 50
// tensors 185 us for the pass against 128, 161 tensors, 25.6 M 72 against 52).  With ordinary loads and stores of the
// residual: 66 M 167 us a call against 146, 40 M in 50 tensors 119 against 101, 25.6 M in 161 79 against 76.  A tensor that
// has no bands (yet, or while its thresholds jump) is read again by the first stage: its blocks take the plain pass, whose
// residual stays in the caches.

// What a lane of such a pass looks for with bands.
template <int DIST>
struct FlatBands {
    float lo, hi, cand;
    double y = 0.0, yy = 0.0;
    uint32_t n = 0, len = 0;
    int2* list;  // the wave's, in LDS: room for all of its elements
    // the wave together; idx is the element's
    __device__ __forceinline__ void look(float x, int32_t idx)
    {
        const float m = __builtin_fabsf(x);
        const bool above = m > hi, keep = (m > lo && !above) || m > cand;
        n += (uint32_t)__popcll(__ballot(above));
        const double v = (double)(above ? m : hi) - (double)hi;
        y += v;
        if (DIST != kDistExp) yy = __builtin_fma(v, v, yy);
        const unsigned long long mask = __ballot(keep);
        if (keep) list[len + lane_prefix(mask)] = make_int2(idx, __float_as_int(x));
        len += (uint32_t)__popcll(mask);
    }
};

// A wave's two tiles of the chunk that starts at tile `first`.
template <int DIST, bool EC, int GT, bool LOOK>
__device__ __forceinline__ void flat_chunk(const Params& p, uint32_t first, uint32_t T1, int wib, int lane, FitSums<DIST>& f,
                                           FlatBands<DIST>& fb)
{
    constexpr bool WRITE = fit_writes<EC, GT>(), PAST = EC && LOOK;
    if (first + kFlatChunk <= T1 && first + kFlatChunk <= p.nfull && (first > 0 || p.shift == 0)) {
        AccTile a[kFlatTiles];
        const size_t i = (size_t)(first + wib) * kTile + lane * 4 - p.shift;
        constexpr size_t step = (size_t)(kFlatBlock / 64) * kTile;
#pragma unroll
        for (int u = 0; u < kFlatTiles; ++u) a[u] = acc_load<EC, WRITE, GT, PAST>(p, i + u * step);
#pragma unroll
        for (int u = 0; u < kFlatTiles; ++u) {
            f4 c = a[u].g;
            if (EC) c = c + a[u].r;
            if (WRITE) acc_store<PAST>(p.acc_w, i + u * step, c);
            f.tile(c, 0);
            if constexpr (LOOK) {
#pragma unroll
                for (int j = 0; j < 4; ++j) fb.look(c[j], (int32_t)(i + u * step) + j);
            }
        }
        return;
    }
    const uint32_t end = first + kFlatChunk < T1 ? first + kFlatChunk : T1;
    for (uint32_t t = first + wib; t < end; t += kFlatBlock / 64) {
        if (t < p.nfull && (t > 0 || p.shift == 0)) {
            const size_t i = (size_t)t * kTile + lane * 4 - p.shift;
            const AccTile a = acc_load<EC, WRITE, GT, false>(p, i);
            f4 c = a.g;
            if (EC) c = c + a.r;
            if (WRITE) acc_store<false>(p.acc_w, i, c);
            f.tile(c, 0);
            if constexpr (LOOK) {
#pragma unroll
                for (int j = 0; j < 4; ++j) fb.look(c[j], (int32_t)i + j);
            }
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int64_t i = (int64_t)t * kTile + lane * 4 + j - p.shift;
                float x = 0.0f;  // above no edge
                if (i >= 0 && i < p.d) x = fit_one<DIST, EC, GT>(p, i, f.s1, f.s2, f.sl, f.se);
                if constexpr (LOOK) fb.look(x, (int32_t)i);
            }
        }
    }
}

template <int DIST, bool EC, int GT, bool BANDS>
__global__ __launch_bounds__(kFlatBlock) void k_fit_flat_batched(BatchArgs a)
{
    constexpr int Q = BANDS ? 6 : 3;  // sums
    __shared__ double sh[kFlatBlock / 64][Q];
    __shared__ int2 sh_list[BANDS ? kFlatBlock / 64 : 1][BANDS ? kFlatTiles * kTile : 1];
    __shared__ uint32_t sh_len[kFlatBlock / 64];
    Blk b;
    uint32_t x = blockIdx.x, y = blockIdx.y;
    if (a.pieces) {
        const uint32_t place = piece_order<256>(y * gridDim.x + x, gridDim.y * gridDim.x);
        y = place / gridDim.x;
        x = place - y * gridDim.x;
    }
    const Params p = batch_params(a, false, b, y);
    Bands e;
    if constexpr (BANDS) e = p.st->band_next;  // beside the descriptor, ahead of all stores: not a round trip of its own
    uint32_t T0, T1;
    block_tiles(p, b, T0, T1);
    const uint32_t first = T0 + x * kFlatChunk;
    const size_t stride = (size_t)gridDim.y * gridDim.x, slot = (size_t)y * gridDim.x + x;
    if (b.id == 0 && x == 0 && threadIdx.x == 0) fit_reset_state(p);
    if (first >= T1) {  // the whole block
        if (threadIdx.x < Q) a.flat[threadIdx.x * stride + slot] = 0.0;
        if (BANDS && threadIdx.x == 0) a.chunk_cnt[slot] = 0;
        return;
    }
    const int lane = threadIdx.x & 63, wib = threadIdx.x >> 6;
    FitSums<DIST> f;
    FlatBands<DIST> fb;
    if constexpr (BANDS) {
        if (bands_usable(e, p.M)) {
            fb.lo = uniform(e.lo[0]);
            fb.hi = uniform(e.hi[0]);
            fb.cand = uniform(e.lo[1]);
            fb.list = sh_list[wib];
            flat_chunk<DIST, EC, GT, true>(p, first, T1, wib, lane, f, fb);
        } else {
            flat_chunk<DIST, EC, GT, false>(p, first, T1, wib, lane, f, fb);
        }
    } else {
        flat_chunk<DIST, EC, GT, false>(p, first, T1, wib, lane, f, fb);
    }
    double v[Q];
    {
        double w_sum[BANDS ? 4 : 2] = {f.s1, DIST == kDistGamma ? f.sl + (double)f.se : f.s2};
        if constexpr (BANDS) {
            w_sum[2] = fb.y;
            w_sum[3] = fb.yy;
        }
        wave_totals(w_sum);
        v[0] = w_sum[0];
        v[1] = DIST == kDistGpd ? w_sum[1] : 0.0;
        v[2] = DIST == kDistGamma ? w_sum[1] : 0.0;
        if constexpr (BANDS) {
            v[3] = w_sum[2];
            v[4] = w_sum[3];
            v[5] = (double)fb.n;
        }
    }
    if (lane == 0) {
#pragma unroll
        for (int q = 0; q < Q; ++q) sh[wib][q] = v[q];
        sh_len[wib] = fb.len;
    }
    __syncthreads();
    if (threadIdx.x < Q) {
        double tot = 0.0;
#pragma unroll
        for (int w = 0; w < kFlatBlock / 64; ++w) tot += sh[w][threadIdx.x];
        a.flat[threadIdx.x * stride + slot] = tot;
    }
    if constexpr (BANDS) {
        uint32_t at = 0, all = 0;
#pragma unroll
        for (int w = 0; w < kFlatBlock / 64; ++w) {
            at += w < wib ? sh_len[w] : 0u;
            all += sh_len[w];
        }
        int2* list = a.chunk_list + slot * kChunkList;
        for (uint32_t q = lane; q < fb.len && at + q < kChunkList; q += 64) list[at + q] = sh_list[wib][q];
        if (threadIdx.x == 0) {
            a.chunk_cnt[slot] = all < kChunkList ? all : kChunkList;
            if (all > kChunkList) p.st->band_over = 1;
        }
    }
}

// Folds the chunks' partial sums of every block y of the batch's dense grid into that block's slot, in a
// fixed order: one wave per y.
__global__ __launch_bounds__(kBlock) void k_fit_reduce_batched(BatchArgs a)
{
    const int lane = threadIdx.x & 63;
    const uint32_t y = blockIdx.x * kWavesPerBlock + (threadIdx.x >> 6);
    if (y >= a.flat_blocks) return;  // the whole wave; no block-wide synchronisation below
    Blk b;
    const Params p = batch_params(a, false, b, y);
    const size_t stride = (size_t)a.flat_gx * a.flat_blocks;
    const double* part = a.flat + (size_t)y * a.flat_gx;
    double v[3] = {0.0, 0.0, 0.0};
    for (uint32_t c = lane; c < a.flat_gx; c += 64) {
        v[0] += part[c];
        if (p.dist == kDistGpd) v[1] += part[stride + c];
        if (p.dist == kDistGamma) v[2] += part[2 * stride + c];
    }
    wave_totals(v);
    if (lane == 0) {
        p.part_out[0 * kBatchBlocks + b.id] = v[0];
        p.part_out[1 * kBatchBlocks + b.id] = v[1];
        p.part_out[2 * kBatchBlocks + b.id] = v[2];
    }
}

// CHUNKS: three blocks per CU, as without.  A batch's grid is up to 1024 blocks; with the 104 registers of eight lists asked
// for at once 512 of them ran first and the rest after them.  With that, and the heads requested in any case, 25.6 M
// elements in 161 tensors took 40.5 us and now 26.6 where the thresholds jump (15.0 and 12.7 where they keep still), 66 M in
// 50 87.7 and 63.1 (20.0 and 16.4); without bands 26.5 and 63.5.  Where the partial sums are folded they are staged in
// LDS: loaded by the first wave they are 40 registers, which went to scratch here (46 spilled, now none), and a call of 25.6 M
// elements in 3 tensors took 84.9 us and now 80.2, 66 M in 8 193.7 and 174.2, in 15 198.6 and 180.9.
template <bool STATS, bool WRITE, bool FLAT, bool KEEP, bool CHUNKS = false>
__global__ __launch_bounds__(kBlock, CHUNKS ? 6 : 4) void k_compact_batched(BatchArgs a)
{
    Blk b;
    const Params p = batch_params(a, false, b);
    FlatPart fp = {};
    if (FLAT) {
        fp.part = a.flat + (size_t)(blockIdx.x - b.id) * a.flat_gx;  // from the vector's first block on
        fp.n = p.nblocks * a.flat_gx;
        fp.stride = a.flat_blocks * a.flat_gx;
    }
    ChunkPart cp = {};
    if (CHUNKS) {
        const size_t first = (size_t)blockIdx.x * a.flat_gx;
        cp.n = a.flat_gx;
        cp.stride = a.flat_blocks * a.flat_gx;
        cp.above = a.flat + 3 * (size_t)cp.stride + first;
        cp.cnt = a.chunk_cnt + first;
        cp.list = a.chunk_list + first * kChunkList;
    }
    compact_body<STATS, WRITE, FLAT, KEEP, false, CHUNKS>(p, b, fp, cp);
}
__global__ __launch_bounds__(kBlock, 4) void k_lists_batched(BatchArgs a)
{
    Blk b;
    const Params p = batch_params(a, false, b);
    lists_body(p, b);
}
__global__ __launch_bounds__(kBlock) void k_final_lists_batched(BatchArgs a)
{
    Blk b;
    const Params p = batch_params(a, true, b);
    final_body(p, b);
}
__global__ __launch_bounds__(kBlock) void k_gather_batched(BatchArgs a)
{
    Blk b;
    const Params p = batch_params(a, false, b);
    gather_body(p, b);
}

// ---------------------------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------------------------
template <bool EC, int GT>
static void launch_fit_as(const Params& p, hipStream_t s)
{
    const dim3 grid(p.nblocks), block(kBlock);
    switch (p.dist) {
        case kDistExp: hipLaunchKernelGGL((k_fit<kDistExp, EC, GT>), grid, block, 0, s, p); break;
        case kDistGamma: hipLaunchKernelGGL((k_fit<kDistGamma, EC, GT>), grid, block, 0, s, p); break;
        default: hipLaunchKernelGGL((k_fit<kDistGpd, EC, GT>), grid, block, 0, s, p); break;
    }
}

template <bool EC, int GT>
static void launch_fit_flat_as(const Params& p, double* flat_part, uint32_t nflat, hipStream_t s)
{
    const dim3 grid(nflat), block(kFlatBlock);
    switch (p.dist) {
        case kDistExp:
            hipLaunchKernelGGL((k_fit_flat<kDistExp, EC, GT>), grid, block, 0, s, p, flat_part, nflat);
            break;
        case kDistGamma:
            hipLaunchKernelGGL((k_fit_flat<kDistGamma, EC, GT>), grid, block, 0, s, p, flat_part, nflat);
            break;
        default: hipLaunchKernelGGL((k_fit_flat<kDistGpd, EC, GT>), grid, block, 0, s, p, flat_part, nflat); break;
    }
}

template <bool EC, int GT>
static void launch_fit_shape(const Params& p, bool flat, double* scratch, hipStream_t s)
{
    if (flat) {
        const uint32_t nflat = fit_flat_blocks(p.d, p.shift);
        launch_fit_flat_as<EC, GT>(p, scratch, nflat, s);
        const uint32_t per = (nflat + kMaxBlocks - 1) / kMaxBlocks;
        hipLaunchKernelGGL(k_fit_reduce, dim3(kMaxBlocks / kWavesPerBlock), dim3(kBlock), 0, s, p, scratch, nflat, per);
        return;
    }
    launch_fit_as<EC, GT>(p, s);
}

template <int GT>
static void launch_fit_type(const Params& p, bool flat, double* scratch, hipStream_t s)
{
    if (p.residual) launch_fit_shape<true, GT>(p, flat, scratch, s);
    else launch_fit_shape<false, GT>(p, flat, scratch, s);
}

template <bool EC, int GT, int NB, bool PAST>
static void launch_fit_bands_as(const Params& p, hipStream_t s)
{
    const dim3 grid(p.nblocks), block(kBlock);
    switch (p.dist) {
        case kDistExp: hipLaunchKernelGGL((k_fit_bands<kDistExp, EC, GT, NB, PAST>), grid, block, 0, s, p); break;
        case kDistGamma: hipLaunchKernelGGL((k_fit_bands<kDistGamma, EC, GT, NB, PAST>), grid, block, 0, s, p); break;
        default: hipLaunchKernelGGL((k_fit_bands<kDistGpd, EC, GT, NB, PAST>), grid, block, 0, s, p); break;
    }
}

template <bool EC, int GT, bool PAST>
static void launch_fit_bands_stages(const Params& p, hipStream_t s)
{
    if (p.M == 2) launch_fit_bands_as<EC, GT, 1, PAST>(p, s);
    else launch_fit_bands_as<EC, GT, 2, PAST>(p, s);
}

template <int GT>
static void launch_fit_bands_type(const Params& p, hipStream_t s)
{
    if (!p.residual) launch_fit_bands_stages<false, GT, false>(p, s);
    else if (p.d >= kBandPastMinD) launch_fit_bands_stages<true, GT, true>(p, s);
    else launch_fit_bands_stages<true, GT, false>(p, s);
}

// p.M = 2 or 3
void launch_fit_bands(const Params& p, hipStream_t s)
{
    switch (p.gt) {
        case kGradF16: launch_fit_bands_type<kGradF16>(p, s); break;
        case kGradBf16: launch_fit_bands_type<kGradBf16>(p, s); break;
        default: launch_fit_bands_type<kGradF32>(p, s); break;
    }
}

template <bool HALF, int N, bool WHOLE = false>
static void launch_small_as(const Params& p, hipStream_t s)
{
    constexpr size_t lds = (kSmallWaves - 1) * kSmallList<N> * sizeof(int2);
    const dim3 grid(1), block(kSmallBlock);
    switch (p.dist) {
        case kDistExp: hipLaunchKernelGGL((k_small<kDistExp, HALF, N, WHOLE>), grid, block, lds, s, p); break;
        case kDistGamma: hipLaunchKernelGGL((k_small<kDistGamma, HALF, N, WHOLE>), grid, block, lds, s, p); break;
        default: hipLaunchKernelGGL((k_small<kDistGpd, HALF, N, WHOLE>), grid, block, lds, s, p); break;
    }
}

template <bool HALF>
static void launch_small_size(const Params& p, hipStream_t s)
{
    constexpr int kShort = 4, kLong = (kSmallMaxD + 4 * kSmallData - 1) / (4 * kSmallData);
    if (p.d <= 4 * kSmallData) launch_small_as<HALF, 1>(p, s);
    else if (p.d <= 4 * kSmallData * kShort) launch_small_as<HALF, kShort>(p, s);
    else if (p.M > 1 || p.L_stage >= kSmallWhole) launch_small_as<HALF, kLong>(p, s);
    else launch_small_as<HALF, kLong, true>(p, s);
}

// needs p.d <= kSmallMaxD
void launch_small(const Params& p, hipStream_t s)
{
    if (p.gt == kGradF32) launch_small_size<false>(p, s);
    else launch_small_size<true>(p, s);
}

// `flat`: the launch shape (see fit_uses_flat).  `scratch`: device memory for 3 * fit_flat_blocks(d, shift) doubles in
// the flat shape (else unused)
void launch_fit(const Params& p, bool flat, double* scratch, hipStream_t s)
{
    switch (p.gt) {
        case kGradF16: launch_fit_type<kGradF16>(p, flat, scratch, s); break;
        case kGradBf16: launch_fit_type<kGradBf16>(p, flat, scratch, s); break;
        default: launch_fit_type<kGradF32>(p, flat, scratch, s); break;
    }
}

void launch_compact(const Params& p, bool stats, bool write, bool keep, hipStream_t s)
{
    const dim3 grid(p.nblocks), block(kBlock);
    if (p.bands == kBandsUse) {  // statistics always: a last stage on the dense vector is another kernel
        if (write) hipLaunchKernelGGL((k_compact<true, true, false, true>), grid, block, 0, s, p);
        else hipLaunchKernelGGL((k_compact<true, false, false, true>), grid, block, 0, s, p);
        return;
    }
    if (stats && write && keep) hipLaunchKernelGGL((k_compact<true, true, true, false>), grid, block, 0, s, p);
    else if (stats && write) hipLaunchKernelGGL((k_compact<true, true, false, false>), grid, block, 0, s, p);
    else if (stats && keep) hipLaunchKernelGGL((k_compact<true, false, true, false>), grid, block, 0, s, p);
    else if (stats) hipLaunchKernelGGL((k_compact<true, false, false, false>), grid, block, 0, s, p);
    else if (keep) hipLaunchKernelGGL((k_compact<false, true, true, false>), grid, block, 0, s, p);
    else hipLaunchKernelGGL((k_compact<false, true, false, false>), grid, block, 0, s, p);
}

void launch_lists(const Params& p, hipStream_t s)
{
    if (p.bands == kBandsUse) hipLaunchKernelGGL(k_lists<true>, dim3(p.nblocks), dim3(kBlock), 0, s, p);
    else hipLaunchKernelGGL(k_lists<false>, dim3(p.nblocks), dim3(kBlock), 0, s, p);
}

void launch_final_lists(const Params& p, uint32_t grid_blocks, hipStream_t s)
{
    // a block reads at most kFinalGroup lists per wave (see final_body)
    const uint32_t least = (p.nwaves + kFinalGroup * kWavesPerBlock - 1) / (kFinalGroup * kWavesPerBlock);
    if (grid_blocks < least) grid_blocks = least;
    if (p.bands == kBandsUse) hipLaunchKernelGGL(k_final_lists<true>, dim3(grid_blocks + 1), dim3(kBlock), 0, s, p);
    else hipLaunchKernelGGL(k_final_lists<false>, dim3(grid_blocks + 1), dim3(kBlock), 0, s, p);
}

void launch_select(const Params& p, bool keep, hipStream_t s)
{
    constexpr uint32_t kTiles = kSelectBlock / 64 * kSelectTiles;
    const uint32_t tiles = p.nwaves * p.tq + p.tr;
    hipLaunchKernelGGL(k_eta, dim3(1), dim3(kBlock), 0, s, p);
    const dim3 grid((tiles + kTiles - 1) / kTiles), block(kSelectBlock);
    if (keep) hipLaunchKernelGGL(k_select<true>, grid, block, 0, s, p);
    else hipLaunchKernelGGL(k_select<false>, grid, block, 0, s, p);
}

void launch_gather(const Params& p, hipStream_t s)
{
    hipLaunchKernelGGL(k_gather, dim3(p.nblocks), dim3(kBlock), 0, s, p);
}

// batched: `blocks` is the sum of the vectors' grids (the last stage's own, smaller sum for launch_final).
// `flat_gx` > 0: the first pass in the flat shape, `flat_gx` chunks of 8 tiles per block of the dense grid, with
// a.flat holding 3 * flat_gx * blocks doubles (6 with bands); `fold`: a second kernel folds them.
template <bool EC, int GT, bool BANDS>
static void launch_fit_batched_as(const BatchArgs& a, uint32_t blocks, uint32_t flat_gx, bool fold, hipStream_t s)
{
    if (flat_gx > 0) {
        const dim3 grid(flat_gx, blocks), block(kFlatBlock);
        switch (a.dist) {
            case kDistExp: hipLaunchKernelGGL((k_fit_flat_batched<kDistExp, EC, GT, BANDS>), grid, block, 0, s, a); break;
            case kDistGamma: hipLaunchKernelGGL((k_fit_flat_batched<kDistGamma, EC, GT, BANDS>), grid, block, 0, s, a); break;
            default: hipLaunchKernelGGL((k_fit_flat_batched<kDistGpd, EC, GT, BANDS>), grid, block, 0, s, a); break;
        }
        if (fold)
            hipLaunchKernelGGL(k_fit_reduce_batched, dim3((blocks + kWavesPerBlock - 1) / kWavesPerBlock), dim3(kBlock), 0, s,
                               a);
        return;
    }
    const dim3 grid(blocks), block(kBlock);
    switch (a.dist) {
        case kDistExp: hipLaunchKernelGGL((k_fit_batched<kDistExp, EC, GT>), grid, block, 0, s, a); break;
        case kDistGamma: hipLaunchKernelGGL((k_fit_batched<kDistGamma, EC, GT>), grid, block, 0, s, a); break;
        default: hipLaunchKernelGGL((k_fit_batched<kDistGpd, EC, GT>), grid, block, 0, s, a); break;
    }
}

template <int GT>
static void launch_fit_batched_type(const BatchArgs& a, bool ec, uint32_t blocks, uint32_t flat_gx, bool fold, hipStream_t s)
{
    const bool bands = a.bands == kBandsUse;
    if (ec && bands) launch_fit_batched_as<true, GT, true>(a, blocks, flat_gx, fold, s);
    else if (ec) launch_fit_batched_as<true, GT, false>(a, blocks, flat_gx, fold, s);
    else if (bands) launch_fit_batched_as<false, GT, true>(a, blocks, flat_gx, fold, s);
    else launch_fit_batched_as<false, GT, false>(a, blocks, flat_gx, fold, s);
}

void launch_fit_batched(const BatchArgs& a, bool ec, uint32_t blocks, uint32_t flat_gx, bool fold, hipStream_t s)
{
    switch (a.gt) {
        case kGradF16: launch_fit_batched_type<kGradF16>(a, ec, blocks, flat_gx, fold, s); break;
        case kGradBf16: launch_fit_batched_type<kGradBf16>(a, ec, blocks, flat_gx, fold, s); break;
        default: launch_fit_batched_type<kGradF32>(a, ec, blocks, flat_gx, fold, s); break;
    }
}

template <bool FLAT, bool KEEP>
static void launch_compact_batched_as(const BatchArgs& a, bool stats, bool write, uint32_t blocks, hipStream_t s)
{
    const dim3 grid(blocks), block(kBlock);
    if (stats && write) hipLaunchKernelGGL((k_compact_batched<true, true, FLAT, KEEP>), grid, block, 0, s, a);
    else if (stats) hipLaunchKernelGGL((k_compact_batched<true, false, FLAT, KEEP>), grid, block, 0, s, a);
    else hipLaunchKernelGGL((k_compact_batched<false, true, FLAT, KEEP>), grid, block, 0, s, a);
}

// `flat`: the first stage, behind a flat first pass whose partial sums have not been folded.  `keep`: ordinary loads
void launch_compact_batched(const BatchArgs& a, bool stats, bool write, bool flat, bool keep, uint32_t blocks, hipStream_t s)
{
    if (a.bands == kBandsUse && a.stage == 1) {  // such a stage writes lists, and no call that keeps the vector has bands
        const dim3 grid(blocks), block(kBlock);
        if (flat) hipLaunchKernelGGL((k_compact_batched<true, true, true, false, true>), grid, block, 0, s, a);
        else hipLaunchKernelGGL((k_compact_batched<true, true, false, false, true>), grid, block, 0, s, a);
        return;
    }
    if (flat && keep) launch_compact_batched_as<true, true>(a, stats, write, blocks, s);
    else if (flat) launch_compact_batched_as<true, false>(a, stats, write, blocks, s);
    else if (keep) launch_compact_batched_as<false, true>(a, stats, write, blocks, s);
    else launch_compact_batched_as<false, false>(a, stats, write, blocks, s);
}

void launch_lists_batched(const BatchArgs& a, uint32_t blocks, hipStream_t s)
{
    hipLaunchKernelGGL(k_lists_batched, dim3(blocks), dim3(kBlock), 0, s, a);
}

void launch_final_lists_batched(const BatchArgs& a, uint32_t final_blocks, hipStream_t s)
{
    hipLaunchKernelGGL(k_final_lists_batched, dim3(final_blocks), dim3(kBlock), 0, s, a);
}

void launch_gather_batched(const BatchArgs& a, uint32_t blocks, hipStream_t s)
{
    hipLaunchKernelGGL(k_gather_batched, dim3(blocks), dim3(kBlock), 0, s, a);
}

}  // namespace sidco
