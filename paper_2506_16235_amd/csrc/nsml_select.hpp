/*
 * libnsml device code, part 2: the head of the selection: sample, what to stage, the streaming
 * pass, the plan, and the radix steps over the dense accumulator that the fallback uses.
 * Included by nsml_kernels.hip (one translation unit); not a public header.
 */
#ifndef NSML_SELECT_HPP
#define NSML_SELECT_HPP

namespace {

/* ------------------------------------------------------------------ sample / predict */

/* Level-0 histogram of a sample of acc = grad + residual: runs of 16 consecutive elements,
 * every run of a small bucket, evenly spaced ones of a large one.  skip (weights): buckets whose word is not NONE need no sample
 * (see k_wpredict; 109 M weights 9.4 us, so 4.6). */
template <bool SUM>   /* SUM: keys of g + r; else keys of g alone (the weight stage) */
__global__ __launch_bounds__(WG) void k_sample(const float *__restrict__ g, const float *__restrict__ r,
                                               Tables t, uint32_t *__restrict__ hist_s, const uint32_t *__restrict__ skip)
{
    __shared__ uint32_t h[NB0];
    const uint32_t tid = threadIdx.x;
    for (int i = tid; i < NB0; i += WG) h[i] = 0;
    const uint32_t b = find_bucket<uint32_t>(t.samp0, t.B, blockIdx.x);
    if (!SUM && skip && skip[b] != NONE) return;     /* same for the whole workgroup */
    const uint32_t wi = blockIdx.x - t.samp0[b];
    const uint64_t lo = t.off[b], hi = t.off[b + 1];
    const uint64_t a0 = lo & ~3ull;
    const uint64_t run_elems = SAMPLE_RUN * sample_stride(hi - lo);
    const uint64_t n_runs = (hi - a0 + run_elems - 1) / run_elems;
    wg_sync();
#pragma unroll 4
    for (uint32_t i = 0; i < RUNS_PER_WG * SAMPLE_RUN / (4 * WG); ++i) {
        const uint64_t run = (uint64_t)wi * RUNS_PER_WG + i * (4 * WG / SAMPLE_RUN) + tid / (SAMPLE_RUN / 4);
        if (run < n_runs) {
            const uint64_t gi = a0 + run * run_elems + (tid % (SAMPLE_RUN / 4)) * 4;
            float x[4], y[4];
            uint32_t m = load_quad(g, gi, lo, hi, x);
            if (SUM) load_quad(r, gi, lo, hi, y);
            if (SUM && t.pmask) {
                const uint64_t rel = gi - a0;
                m &= ~pruned_bits(t.pmask, t.tile0[b] + (uint32_t)(rel / TILE), (uint32_t)(rel % TILE) / 4);
            }
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if ((m >> j) & 1u) atomicAdd(&h[keyof(SUM ? __fadd_rn(x[j], y[j]) : x[j]) >> SH0], 1u);
        }
    }
    wg_sync();
    hist_flush(h, hist_s + (uint64_t)b * NB0, NB0);
}

/* The finest bin shift with which [L, W) takes at most NHB bins (never below SH1: the steps that follow
 * take at least the last 7 bits from the keys themselves; at most SH0, a wider window ends in the
 * open last bin). */
__device__ __forceinline__ uint32_t window_shift(uint32_t L, uint32_t W)
{
    uint32_t s = SH1;
    while (s < (uint32_t)SH0 && ((W - 1u) >> s) - (L >> s) >= (uint32_t)NHB) ++s;
    return s;
}

/* Per bucket: what the streaming pass stages and counts, from the sample histogram.  The sample
 * count above the true k-th key is binomial with mean ks = k * m / n.
 *   candidates  k at most an eighth of the bucket: L_b = lower edge of the digit that has
 *               ks + 4 sqrt(ks) + 4 sampled keys above it; everything from L_b up is staged and
 *               contains the k largest unless the sample was very unlucky
 *   band        larger k (ratios towards 1): staging everything above a bound would be most of
 *               the bucket, so only the level-0 digits between the ranks ks +- (4 sqrt(ks) + 4)
 *               are staged, [L_b, H_b); the elements above H_b are survivors for certain and are
 *               only counted
 *   zero        even the optimistic rank lies among keys below 2^19 (in practice: exact zeros,
 *               as in an embedding whose rows were not touched), or k is the whole bucket: the
 *               threshold key is 0, nothing is staged, non-zero and zero keys are counted
 * The window of keys that the streaming pass counts in NHB bins is the band itself, or for candidates
 * reaches from L_b to the digit of rank ks - 2 (4 sqrt(ks) + 4): the k-th key lies in it with a wide
 * margin, and one bin is all that stays undecided.  (Counting the keys above the window one by one
 * in the same bins was no gain in safety and cost an atomic each.)
 * A bucket for which none of this fits (or whose guess turns out wrong once the exact counts are
 * known) takes the dense passes and still gets the exact result. */
template <typename WALK>      /* the sample's histogram: find(rank, digit, above, at), total; -> whether there is anything to stage or count */
__device__ __forceinline__ bool predict_bucket(const Tables &t, uint32_t b, uint64_t nb, uint32_t k, double pop, bool exact, uint32_t wide, const WALK &w, uint32_t *res)
{
    const uint32_t tid = threadIdx.x;
    const KeyPar nothing = make_uint4(NONE, NONE, NONE, SH1);
    const uint32_t m = w.total;
    if (m == 0) {
        if (tid == 0) t.par[b] = nothing;
        return false;
    }
    const double ks = (double)k * (double)m / pop;
    const double cap_b = (double)(t.tile0[b + 1] - t.tile0[b]) * (double)SEG_CAP;
    auto clip = [&](double x) { return x < 1.0 ? 1.0 : (x > (double)m ? (double)m : x); };
    /* the margin: four standard deviations of a binomial sample, times what the bucket has
     * learned (a sample of runs of a gradient whose large values come in runs has far
     * fewer independent draws than entries; a bucket whose guess missed widens its margin).  Where so wide a margin
     * leaves nothing that can be staged, half of it is tried, down to the plain one (a bucket that had once missed
     * was on the dense passes for 64 calls: 25 M elements at 0.8 500 us a call, so 285). */
    uint32_t widen = (t.margin[b] & 0xFFu ? t.margin[b] & 0xFFu : 1u) * wide;
    while (true) {
        const double dev = exact ? 0.0 : (4.0 * sqrt(ks) + 4.0) * (double)widen;
        const double want_d = exact ? (double)k : ceil(ks + dev);
        const double r_up = clip(floor(ks - dev)), r_dn = clip(ceil(ks + dev)), r_top = clip(floor(ks - 2.0 * dev));
        const double r_c = clip(want_d);
        uint32_t digit, above, at;
        if (w.find((uint32_t)r_c, digit, above, at)) { res[0] = digit; res[1] = above; res[2] = at; }
        if (w.find((uint32_t)r_up, digit, above, at)) { res[3] = digit; res[4] = above; res[5] = at; }
        if (w.find((uint32_t)r_dn, digit, above, at)) { res[6] = digit; res[7] = above; res[8] = at; }
        if (w.find((uint32_t)r_top, digit, above, at)) res[9] = digit;
        wg_sync();
        /* every thread comes to the same p */
        KeyPar p = nothing;
        bool done = false;
        if (want_d <= (double)m && candidates_fit(k, t.tile0[b + 1] - t.tile0[b])) {
            const double est = (double)(res[1] + res[2]) * pop / (double)m;
            if (est <= 0.8 * cap_b) {
                p.x = res[0] << SH0;
                p.z = (max(res[9], res[0]) + 1u) << SH0;
                p.w = window_shift(p.x, p.z);
                done = true;
            }
        }
        if (!done) {
            const uint32_t dig_up = res[3], dig_dn = res[6];
            if (dig_up == 0u) {
                p = make_uint4(1u, 1u, 1u, SH1);
            } else {
                /* a pessimistic rank among the zeros (digit 0) while the optimistic one is not: the band
                 * starts at key 1, zeros are only counted, and the plan decides between a zero
                 * threshold and one inside the band */
                const double in_band = (double)res[7] + (dig_dn != 0u ? (double)res[8] : 0.0) - (double)res[4];
                const double est = in_band * pop / (double)m;
                if (est <= 0.8 * cap_b) {
                    p.x = dig_dn != 0u ? dig_dn << SH0 : 1u;
                    p.y = p.z = (dig_up + 1u) << SH0;
                    p.w = window_shift(p.x, p.z);
                } else if (exact) {
                    /* too many keys in one digit to stage them, but all of the bucket was sampled: the dense passes
                     * need not look for that digit again */
                    p.w = SH0;
                    if (tid == 0) { t.T[b] = res[0]; t.need[b] = k - res[1]; }
                }
            }
        }
        if (p.x != NONE || exact || widen == 1u) {
            if (tid == 0) t.par[b] = p;
            return p.x != NONE;
        }
        widen >>= 1;
        wg_sync();                                       /* res is written again */
    }
}

/* The sample was taken by k_sample: more than four buckets for every compute unit, one of PRE_BIG elements and more among them, or every bucket
 * is sent to the dense passes (then there is none). */
__global__ __launch_bounds__(WG) void k_predict(Tables t, uint32_t *__restrict__ hist_s, int force_dense)
{
    __shared__ uint32_t tmp[WG];
    __shared__ uint32_t res[10];         /* digit, above, at for three ranks; digit of the window's top */
    const uint32_t b = blockIdx.x, tid = threadIdx.x;
    const uint64_t nb = t.off[b + 1] - t.off[b];
    const uint32_t k = t.k[b];
    if (b == 0 && tid < 4) t.nhard[tid] = 0u;      /* counted anew by this call's plan ([1]: the barrier of k_hard) */
    if (nb == 0 || force_dense) {
        if (tid == 0) t.par[b] = make_uint4(NONE, NONE, NONE, SH1);
        return;
    }
    if ((uint64_t)k == nb) {             /* everything is sent: all keys >= 1, and the zeros as ties of key 0 */
        if (tid == 0) t.par[b] = make_uint4(1u, 1u, 1u, SH1);
        for (int i = tid; i < NB0; i += WG) hist_s[(uint64_t)b * NB0 + i] = 0u;     /* left clean for the next call */
        return;
    }
    DigitWalk<NB0> w;
    w.load(hist_s + (uint64_t)b * NB0, tmp);
    w.clear(hist_s + (uint64_t)b * NB0);
    /* the sample was drawn from the parameters that can be selected: all of them, or the
     * ones the pruning step kept */
    predict_bucket(t, b, nb, k, t.pmask ? (double)t.kw[b] : (double)nb, nb < SAMPLE_ALL_BELOW, 1u, w, res);
}

/* Sample and prediction of a bucket by one workgroup, and the tables of a new (ratio, bits) beside them: three launches
 * that wait for each other in one.  What a compute unit can fetch alone (25 - 50 GB/s) bounds it, so the sample is
 * PRE_ELEMS elements (in the same runs of 16), and in buckets of which k_sample takes every element the margin of the
 * candidates is twice as wide (a wider band would overflow the segments of clustered values).  ResNet-50's 161 buckets: 9.6 us, by k_sample and k_predict 12 + 8 (and 5 for the tables); 1 Mi
 * elements 7.5, 6.2 + 5.5.  With 32768 elements 22 us.
 * A bucket in which so few leave nothing to stage (a large group of equal values near the threshold) is sampled once more, for
 * a narrower band may fit: 32768 elements at most (compress at 0.4 as 32-bit values, us, without / with: 400 buckets of 40003 clipped values
 * 245 / 178, 12 of 3 M 277 / 242).  All of it where no bucket of the layout is too large for that: then the dense passes need not look
 * for the first digit, a read and two barriers less for all of them (100000 elements of two magnitudes 194 / 169, by k_sample 160;
 * 250000 220 / 214, 189; with a larger bucket beside it nothing is gained: 4 M elements in 100 buckets 290 / 328). */
constexpr uint32_t PRE_T = 1024, PRE_U = 2, PRE_AGAIN_U = 4;       /* 16-byte accesses a thread has in flight, per operand */
constexpr uint32_t PRE_ELEMS = 8192, PRE_AGAIN_ELEMS = 32768;
constexpr uint32_t PRE_COPIES = 8, PRE_ROW = NB0 + 4;       /* copies of the histogram, and words of one: the copies of a digit in different banks */
constexpr uint64_t PRE_BIG = 1ull << 22;           /* larger buckets need a larger sample (16 of 4 M, rows of zeros: already 4 % slower) */
__device__ __forceinline__ uint64_t pre_stride(uint64_t nb) { return nb < 2u * PRE_ELEMS ? 1u : nb / PRE_ELEMS; }
/* of the second sample; whole: every bucket of the layout has less than SAMPLE_ALL_BELOW elements */
__device__ __forceinline__ uint64_t again_stride(uint64_t nb, bool whole)
{
    return whole ? 1u : max(sample_stride(nb), nb / PRE_AGAIN_ELEMS);
}
/* the histogram's digits from the top, four per thread */
struct DigitWalk1024 {
    uint32_t c[NB0 / PRE_T], sum, incl, total;
    int top;
    __device__ __forceinline__ void load(const uint32_t *h, uint32_t *tmp)
    {
        const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
        top = NB0 - 1 - (int)threadIdx.x * (NB0 / (int)PRE_T);
        sum = 0;
#pragma unroll
        for (uint32_t i = 0; i < NB0 / PRE_T; ++i) { c[i] = h[top - (int)i]; sum += c[i]; }
        incl = sum;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) { const uint32_t y = __shfl_up(incl, d, 64); if (lane >= (uint32_t)d) incl += y; }
        if (lane == 63) tmp[wave] = incl;
        wg_sync();
        total = 0;
#pragma unroll
        for (uint32_t v = 0; v < PRE_T / 64; ++v) { incl += v < wave ? tmp[v] : 0u; total += tmp[v]; }
    }
    __device__ __forceinline__ bool find(uint32_t want, uint32_t &digit, uint32_t &above, uint32_t &at) const
    {
        uint32_t acc = incl - sum;
        if (!(acc < want && want <= incl)) return false;
#pragma unroll
        for (uint32_t i = 0; i < NB0 / PRE_T; ++i) {
            if (acc + c[i] >= want) { digit = (uint32_t)(top - (int)i); above = acc; at = c[i]; return true; }
            acc += c[i];
        }
        return false;
    }
};
/* The histogram h of a bucket's runs, one in `stride`, by a workgroup of PRE_T threads with U accesses each in flight per operand.
 * COPIES: of the histogram, which the lanes take in turn and which are added up at the end (a few values that nearly all
 * elements have are one word's additions after the other otherwise: those 100000 elements 188 us with one copy). */
template <uint32_t U, uint32_t COPIES>
__device__ __forceinline__ void sample_bucket(const float *__restrict__ g, const float *__restrict__ r, const Tables &t, uint32_t b,
                                              uint64_t lo, uint64_t hi, uint64_t stride, uint32_t *h)
{
    const uint32_t tid = threadIdx.x;
    const uint64_t a0 = lo & ~3ull, run_elems = SAMPLE_RUN * stride, n_runs = (hi - a0 + run_elems - 1) / run_elems;
    const uint32_t tile0b = t.pmask ? t.tile0[b] : 0u;
    for (uint32_t i = tid * 4u; i < COPIES * PRE_ROW; i += PRE_T * 4u) *reinterpret_cast<uint4 *>(h + i) = make_uint4(0u, 0u, 0u, 0u);
    wg_sync();
    uint32_t *hc = h + (COPIES > 1 ? (tid % COPIES) * PRE_ROW : 0u);
    constexpr uint32_t RUNS = PRE_T / (SAMPLE_RUN / 4);         /* per access of all threads */
    /* a wavefront goes on as long as its first lane has a run: the addition for all of it below counts 64 lanes */
#pragma unroll 1
    for (uint64_t first = tid / 64 * (64 / (SAMPLE_RUN / 4)); first < n_runs; first += RUNS * U) {
        const uint64_t run0 = first + (tid & 63u) / (SAMPLE_RUN / 4);
        f4 x[U], y[U];
        uint32_t m[U];
#pragma unroll
        for (uint32_t u = 0; u < U; ++u) {
            const uint64_t gi = a0 + (run0 + u * RUNS) * run_elems + (tid % (SAMPLE_RUN / 4)) * 4;
            x[u] = y[u] = f4{0.f, 0.f, 0.f, 0.f};
            m[u] = 0u;
            if (run0 + u * RUNS < n_runs && gi >= lo && gi + 4 <= hi) {
                x[u] = *reinterpret_cast<const f4 *>(g + gi);
                y[u] = *reinterpret_cast<const f4 *>(r + gi);
                m[u] = 0xFu;
                if (t.pmask) m[u] = ~pruned_bits(t.pmask, tile0b + (uint32_t)((gi - a0) / TILE), (uint32_t)((gi - a0) % TILE) / 4) & 0xFu;
            }
        }
#pragma unroll
        for (uint32_t u = 0; u < U; ++u) {
            const uint64_t gi = a0 + (run0 + u * RUNS) * run_elems + (tid % (SAMPLE_RUN / 4)) * 4;
            if (run0 + u * RUNS < n_runs && gi < hi && (gi < lo || gi + 4 > hi)) {
                /* the bucket's first and last quad may be partly another's */
                float xa[4], ya[4];
                m[u] = load_quad(g, gi, lo, hi, xa);
                load_quad(r, gi, lo, hi, ya);
                if (t.pmask) m[u] &= ~pruned_bits(t.pmask, tile0b + (uint32_t)((gi - a0) / TILE), (uint32_t)((gi - a0) % TILE) / 4);
                x[u] = f4{xa[0], xa[1], xa[2], xa[3]};
                y[u] = f4{ya[0], ya[1], ya[2], ya[3]};
            }
            uint32_t d[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) d[j] = keyof(__fadd_rn(x[u][j], y[u][j])) >> SH0;
            /* runs of equal keys (zeros): one addition for the wavefront */
            const uint32_t fd = __builtin_amdgcn_readfirstlane(d[0]);
            if (__all(m[u] == 0xFu && d[0] == fd && d[1] == fd && d[2] == fd && d[3] == fd)) {
                if ((tid & 63u) == 0u) atomicAdd(&h[fd], 256u);
                continue;
            }
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if ((m[u] >> j) & 1u) atomicAdd(&hc[d[j]], 1u);
        }
    }
    wg_sync();
    if constexpr (COPIES > 1) {
        static_assert(NB0 == 4u * PRE_T, "four digits per thread");
        uint4 sum = make_uint4(0u, 0u, 0u, 0u);
#pragma unroll
        for (uint32_t q = 0; q < COPIES; ++q) {
            const uint4 v = *reinterpret_cast<const uint4 *>(h + q * PRE_ROW + tid * 4u);
            sum.x += v.x; sum.y += v.y; sum.z += v.z; sum.w += v.w;
        }
        *reinterpret_cast<uint4 *>(h + tid * 4u) = sum;      /* (read by this thread alone) */
        wg_sync();
    }
}
__global__ __launch_bounds__(PRE_T) void k_presample(const float *__restrict__ g, const float *__restrict__ r, Tables t, double ratio,
                                                     int bits, bool whole, uint64_t n_chunks, uint32_t *__restrict__ chunk_b)
{
    __shared__ __align__(16) uint32_t h[PRE_COPIES * PRE_ROW];
    static_assert(sizeof h >= (SETUP_MAX_B + 1) * sizeof(uint64_t), "the set-up's chunk prefixes take its place");
    __shared__ uint32_t tmp[PRE_T / 64], res[10];
    const uint32_t b = blockIdx.x, tid = threadIdx.x;
    if (b >= t.B) {                                  /* workgroups beyond the buckets: set-up */
        setup_all<PRE_T>(t, ratio, bits, n_chunks, chunk_b, reinterpret_cast<uint64_t *>(h), b - t.B, gridDim.x - t.B);
        return;
    }
    if (b == 0 && tid < 4) t.nhard[tid] = 0u;      /* counted anew by this call's plan ([1]: the barrier of k_hard) */
    const uint64_t lo = t.off[b], hi = t.off[b + 1], nb = hi - lo, stride = pre_stride(nb);
    const uint32_t k = (uint32_t)survivors_dev(ratio, nb);
    if (nb == 0 || (uint64_t)k == nb) {              /* everything is sent: all keys >= 1, and the zeros as ties of key 0 */
        if (tid == 0) t.par[b] = nb == 0 ? make_uint4(NONE, NONE, NONE, SH1) : make_uint4(1u, 1u, 1u, SH1);
        return;
    }
    DigitWalk1024 w;
    auto predict = [&](uint64_t step) __attribute__((always_inline)) {
        w.load(h, tmp);
        return predict_bucket(t, b, nb, k, t.pmask ? (double)kept_dev(ratio, nb) : (double)nb, step == 1u,
                              nb < SAMPLE_ALL_BELOW && (uint64_t)k * 8u <= nb ? 2u : 1u, w, res);
    };
    sample_bucket<PRE_U, 1>(g, r, t, b, lo, hi, stride, h);
    if (predict(stride)) return;
    const uint64_t again = again_stride(nb, whole);
    if (stride <= again || (!whole && w.total != 0u && res[3] == res[6])) return;      /* (a band of one digit cannot get narrower) */
    sample_bucket<PRE_AGAIN_U, PRE_COPIES>(g, r, t, b, lo, hi, again, h);
    (void)predict(again);
}

/* ------------------------------------------------------------------ the streaming pass */

/* What the two streaming passes (gradient, weights) share: the flagged elements of the workgroup's
 * tile, staged in index order, and the window's bins.  NTH threads hold a tile of TILE / (4 NTH) rows, row
 * u's quads at u * NTH + thread.  The positions come from ballots inside a wavefront and one exchange of
 * wavefront totals; the staged elements go through LDS so that a tile's few dozen leave in one or two
 * full-width stores (stored by the lanes that hold them, every wavefront sends partly filled lines of
 * its own: at 2.4 % staged that pass took 3.7 instead of 3.2 ms on 1.7 G elements).
 * HIST: the bins are counted here, in LDS first: with error feedback the accumulators pile up just under
 * the threshold, and single addresses in memory take 3 ns per update.  Flushing a tile's few dozen
 * different bins still costs (419 M elements at ratio 0.5: 930 us against 780 without; 25 M at
 * 0.05: 66 against 57), so from HIST_MAX_TILES up k_bins counts them from the staged elements instead. */
constexpr uint32_t HIST_MAX_TILES = 16384;
template <bool HIST> struct StageBins { uint32_t h[NHB]; };
template <> struct StageBins<false> { };
template <bool HIST>
struct StageShared {
    StageBins<HIST> bins;
    float sv[SEG_CAP];
    uint32_t si[SEG_CAP];
    uint32_t wtot[TILE / 256], whi[TILE / 256], wlo[TILE / 256];
};

template <int NTH, bool HIST>
__device__ __forceinline__ void stage_tile(const float (&a)[TILE / (4 * NTH)][4], const uint32_t (&cm)[TILE / (4 * NTH)], const KeyPar &p,
                                           uint32_t b, uint32_t tile, uint32_t li0, const Cand &c, uint32_t *__restrict__ hist,
                                           uint32_t *__restrict__ ovf, StageShared<HIST> &sm)
{
    constexpr int Q = TILE / (4 * NTH);
    constexpr uint32_t W = NTH / 64;
    const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    uint32_t pos[Q], wtot[Q];
    uint32_t fl[Q];                                    /* flagged elements of the quad */
#pragma unroll
    for (int u = 0; u < Q; ++u) {
        uint32_t hi = 0, lo = 0;
        fl[u] = 0; pos[u] = wtot[u] = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const bool in = (cm[u] >> j) & 1u;
            const uint32_t key = keyof(a[u][j]);
            fl[u] |= (in && key >= p.x && key < p.y ? 1u : 0u) << j;
            hi += __popcll(__ballot(in && key >= p.z));
        }
        if (p.y != NONE) {
            /* a band (or nothing) is staged: the elements below it are counted as well */
#pragma unroll
            for (int j = 0; j < 4; ++j) lo += __popcll(__ballot(((cm[u] >> j) & 1u) && keyof(a[u][j]) < p.x));
        }
        if (__ballot(fl[u] != 0u)) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint64_t bal = __ballot((fl[u] >> j) & 1u);
                pos[u] = __builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bal, pos[u]));   /* flagged ones in lower lanes */
                wtot[u] += __popcll(bal);
            }
        }
        if (lane == 0) { sm.wtot[u * W + wave] = wtot[u]; sm.whi[u * W + wave] = hi; sm.wlo[u * W + wave] = lo; }
    }
    if constexpr (HIST)
        for (uint32_t i = tid; i < (uint32_t)NHB; i += NTH) sm.bins.h[i] = 0u;
    wg_sync();
    uint32_t all = 0, before[Q];
#pragma unroll
    for (uint32_t w = 0; w < Q * W; ++w) {
#pragma unroll
        for (int u = 0; u < Q; ++u) if (w == (uint32_t)u * W) before[u] = all;
        all += sm.wtot[w];
    }
    if (W > 1) {
#pragma unroll
        for (int u = 0; u < Q; ++u)
#pragma unroll
            for (uint32_t w = 0; w < W; ++w) before[u] += w < wave ? sm.wtot[u * W + w] : 0u;
    }
    if (tid == 0) {
        uint32_t thi = 0, tlo = 0;
#pragma unroll
        for (uint32_t w = 0; w < Q * W; ++w) { thi += sm.whi[w]; tlo += sm.wlo[w]; }
        /* the true count: more than the segment holds means "read this tile from the dense
         * source" to the kernels that follow */
        c.cnt[tile] = all;
        c.G[tile] = thi;
        c.E[tile] = tlo;
        if (all > SEG_CAP) *ovf = 1u;
        if constexpr (HIST)
            if (thi) atomicAdd(hist + ((uint64_t)b * NHC + blockIdx.x % NHC) * HROW + NHB, thi);
    }
    if (all == 0u) return;                             /* same for the whole workgroup */
    const uint32_t top = (p.z - 1u) >> p.w;
#pragma unroll
    for (int u = 0; u < Q; ++u) {
        if (wtot[u] == 0u) continue;
        uint32_t at = pos[u] + before[u];
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if ((fl[u] >> j) & 1u) {
                if (at < SEG_CAP) { sm.sv[at] = a[u][j]; sm.si[at] = li0 + (u * NTH + tid) * 4u + j; }
                ++at;
                if constexpr (HIST) {
                    const uint32_t key = keyof(a[u][j]);
                    if (key < p.z) atomicAdd(&sm.bins.h[min(top - (key >> p.w), (uint32_t)NHB - 1u)], 1u);
                }
            }
    }
    wg_sync();
    const uint64_t cbase = (uint64_t)tile * SEG_CAP;
    for (uint32_t i = tid; i < min(all, SEG_CAP); i += NTH) { c.idx[cbase + i] = sm.si[i]; c.val[cbase + i] = sm.sv[i]; }
    if constexpr (HIST) hist_flush(sm.bins.h, hist + ((uint64_t)b * NHC + blockIdx.x % NHC) * HROW, NHB, NTH);
}

/* acc = grad + residual over a tile, written over residual (Sec. 4.2 Step 3: what top-k filters out
 * is accumulated locally; the add is that), the counts and bins of the keys, and the staged
 * elements.  Bound by HBM: 12 bytes per element plus 8 per staged one.  One tile per workgroup, four
 * workgroups per compute unit: 1.68 G elements in 3.1 ms (6.5 TB/s; workgroups that walked 8 tiles with
 * a contiguous 16 KiB per wavefront and a 4096-bin histogram took 3.46 ms), 25.6 M in 64 us (75). */
template <bool EMIT, bool PRUNE, bool NT, bool HIST>
__global__ __launch_bounds__(STH, 8) void k_ef_emit(const float *__restrict__ g, float *__restrict__ r,
                                                    Tables t, uint32_t *__restrict__ hist, Cand c,
                                                    double *__restrict__ tile_sq)
{
    __shared__ StageShared<HIST> sm;
    __shared__ double sq_w[STH / 64];
    const uint32_t tile = grid_tile();
    if (tile >= t.n_tiles) return;
    const uint4 d = t.desc[tile];
    const uint32_t tid = threadIdx.x, e = tid * 4u, first = d.w & 0xFFFFu, last = d.w >> 16;
    const uint64_t gi = (((uint64_t)d.y << 32) | d.x) + e;
    float av[1][4];
    float (&a)[4] = av[0];
    double sq;
    uint32_t mv[1] = {0xFu};
    uint32_t &m = mv[0];
    if (e >= first && e + 4u <= last) {
        const f4 x = __builtin_nontemporal_load(reinterpret_cast<const f4 *>(g + gi));
        const f4 y = __builtin_nontemporal_load(reinterpret_cast<const f4 *>(r + gi));
        f4 v;
        v.x = __fadd_rn(x.x, y.x); v.y = __fadd_rn(x.y, y.y); v.z = __fadd_rn(x.z, y.z); v.w = __fadd_rn(x.w, y.w);
        st_out<NT>(reinterpret_cast<f4 *>(r + gi), v);
        a[0] = v.x; a[1] = v.y; a[2] = v.z; a[3] = v.w;
        sq = (double)(__fmaf_rn(x.x, x.x, __fmul_rn(x.y, x.y)) + __fmaf_rn(x.z, x.z, __fmul_rn(x.w, x.w)));
    } else {
        m = 0; sq = 0.0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            a[j] = 0.0f;
            if (e + j >= first && e + j < last) {
                const float x = g[gi + j];
                a[j] = __fadd_rn(x, r[gi + j]);
                r[gi + j] = a[j];
                sq += (double)__fmul_rn(x, x);
                m |= 1u << j;
            }
        }
    }
    /* the tile's share of |grad|^2 (by-product for the density test of Algorithm 2 Step 1): a fixed
     * reduction tree, so the sum does not depend on scheduling */
    sq = wave_sum_last(sq);
    if ((tid & 63u) == 63u) sq_w[tid >> 6] = sq;
    if (EMIT) {
        if (PRUNE) m &= ~pruned_bits(t.pmask, tile, tid);
        const uint32_t b = d.z;
        stage_tile<STH, HIST>(av, mv, t.par[b], b, tile, (uint32_t)(gi - e - t.off[b]), c, hist, t.ovf + b, sm);
    } else {
        wg_sync();
    }
    if (tid == 0) {
        double tot = 0.0;
#pragma unroll
        for (uint32_t w = 0; w < STH / 64; w += 4) tot += (sq_w[w] + sq_w[w + 1]) + (sq_w[w + 2] + sq_w[w + 3]);
        tile_sq[tile] = tot;
    }
}

/* How a bucket is decided (PATH_*), from its exact counts: n_hi elements at or above the window's top; found: the k-th key lies
 * in the window, in its bin `bin`, with `above` elements above that bin and `at` in it; total: all of the window's.  The staged elements can decide
 * it when they are known to hold every element of that bin: in candidate mode they are exactly the elements with
 * key >= L_b, so they do iff there are at least k of them and the key lies below the window's top; in band mode iff it
 * lies inside the band; in both only if the undecided keys of the bin fit the bucket's list of them (k_select_count).  In
 * zero mode the counts settle everything: fewer non-zero elements than k means threshold key 0. */
struct Plan { uint32_t path, T, need, sh, why; };
__device__ __forceinline__ Plan plan_bucket(const Tables &t, uint32_t b, const KeyPar &p, uint32_t want, uint32_t n_hi, uint32_t total, bool found,
                                            uint32_t bin, uint32_t above, uint32_t at, uint32_t ovf, uint32_t segs)
{
    Plan q = {PATH_DENSE, 0u, want, SH_NONE, 0u};
    if (p.x == NONE) {
        q.why = WHY_NO_GUESS;
        if (p.w == (uint32_t)SH0) { q.T = t.T[b]; q.need = t.need[b]; q.sh = SH0; }       /* (left there by the prediction) */
    }
    else if (p.x == p.y) {
        /* n_hi = non-zero keys among the selectable elements: if they are no more than k,
         * all of them survive and zeros (lowest indices first) fill the rest */
        if (n_hi <= want) { q.path = PATH_ZERO; q.need = want - n_hi; q.sh = SH0; }
        else q.why = WHY_NONZEROS;
    } else if (p.x == 1u && p.y != NONE && (uint64_t)n_hi + total <= want) {
        /* the band starts at key 1 and everything non-zero is still not enough: zero threshold */
        q.path = PATH_ZERO; q.need = want - (n_hi + total); q.sh = SH0;
    } else if (found) {
        /* a tile whose segment overflowed is read from the dense accumulator by the kernels
         * that find the threshold; the survivors of such a bucket are then taken from the dense
         * accumulator as well (PATH_BAND), since the staged entries cannot supply them all */
        const uint32_t top = (p.z - 1u) >> p.w;
        if (bin == (uint32_t)NHB - 1u && (p.x >> p.w) != top - bin) q.why = WHY_OUTSIDE_BAND;    /* the open last bin */
        else {
            q.T = top - bin; q.need = want - above; q.sh = p.w;
            if (!list_pays(at, segs, t.n_tiles)) q.why = WHY_NO_ROOM;       /* (the dense passes go on from that bin) */
            else q.path = p.y == NONE && !ovf ? PATH_CAND : PATH_BAND;
        }
    } else q.why = n_hi < want ? WHY_TOO_FEW : WHY_OUTSIDE_BAND;
    return q;
}
/* The plan's record (one thread per bucket). */
__device__ __forceinline__ void plan_store(const Tables &t, uint32_t b, const Plan &q)
{
    t.why[b] = q.why;
    {
        /* low byte: factor on the margin of the prediction (1, 2, 4, 8, 16); above it: calls since it last grew.
         * A guess that missed doubles it, 64 calls without a miss halve it. */
        const uint32_t mg = t.margin[b];
        uint32_t f = mg & 0xFFu ? mg & 0xFFu : 1u, age = mg >> 8;
        if (q.why == WHY_TOO_FEW || q.why == WHY_OUTSIDE_BAND) { f = f < 16u ? f * 2u : 16u; age = 0u; }
        else if (++age >= 64u) { f = f > 1u ? f / 2u : 1u; age = 0u; }
        t.margin[b] = (age << 8) | f;
    }
    t.T[b] = q.T;
    t.need[b] = q.need;
    t.sh[b] = q.sh;
    t.fast[b] = q.path;
    if (q.path != PATH_CAND) atomicAdd(t.nhard, 1u);
    if (q.path == PATH_DENSE) atomicAdd(t.nhard + 2, 1u);
    if (q.path == PATH_DENSE && q.sh == SH_NONE) atomicAdd(t.nhard + 3, 1u);
}
/* An empty bucket: nothing can match. */
__device__ __forceinline__ void plan_empty(const Tables &t, uint32_t b)
{
    t.T[b] = NONE; t.need[b] = 0; t.fast[b] = PATH_CAND; t.sh[b] = SH0; t.why[b] = 0u;
}

/* |grad|^2 of a bucket by a workgroup of NT threads: strided partial sums, then a fixed tree.  red: NT / 64 words. */
template <uint32_t NT>
__device__ __forceinline__ void bucket_sq(const Tables &t, uint32_t b, const double *__restrict__ tile_sq, double *red, double *__restrict__ out)
{
    double acc = 0.0;
    const uint32_t t1 = t.tile0[b + 1];
#pragma unroll 4
    for (uint32_t s = t.tile0[b] + threadIdx.x; s < t1; s += NT) acc += tile_sq[s];
    acc = wave_sum_last(acc);
    if ((threadIdx.x & 63u) == 63u) red[threadIdx.x >> 6] = acc;
    wg_sync();
    if (threadIdx.x != 0) return;
    double tot = 0.0;
    for (uint32_t w = 0; w < NT / 64; w += 4) tot += (red[w] + red[w + 1]) + (red[w + 2] + red[w + 3]);
    *out = tot;
}

/* The plan when every bucket is sent to the dense passes (force_dense). */
__global__ __launch_bounds__(1024) void k_plan_dense(Tables t, const double *__restrict__ tile_sq, double *__restrict__ l2sq)
{
    __shared__ double red[16];
    const uint32_t b = blockIdx.x;
    bucket_sq<1024>(t, b, tile_sq, red, l2sq + b);
    if (threadIdx.x != 0) return;
    if (t.k[b] == 0u) { plan_empty(t, b); return; }
    plan_store(t, b, Plan{PATH_DENSE, 0u, t.k[b], SH_NONE, WHY_NO_GUESS});
}

/* One workgroup: the list of tiles that belong to buckets on the dense passes.  (The team's first step: done by the last
 * workgroup of the launch that makes the plans, it needs a device-scope fence in every workgroup there, which on this multi-die
 * GPU writes back each L2 and costs more than a launch.) */
__device__ __forceinline__ void fb_plan_body(const Tables &t)
{
    __shared__ uint32_t tmp[WG];
    const uint32_t tid = threadIdx.x;
    uint32_t carry = 0;
    for (uint32_t base = 0; base < t.B; base += WG) {
        const uint32_t bb = base + tid;
        const bool fb = bb < t.B && !t.fast[bb];
        const uint32_t x = fb ? t.tile0[bb + 1] - t.tile0[bb] : 0u;
        const uint32_t incl = block_incl_scan(x, tmp);
        const uint32_t tot = tmp[WG - 1];
        wg_sync();
        if (bb < t.B) t.ftile0[bb] = carry + incl - x;
        carry += tot;
    }
    if (tid == 0) t.ftile0[t.B] = carry;
}

/* The next digit of a dense bucket's k-th key from its histogram over the accumulator: level 0 the 12 bits
 * from position 19 up, of the buckets of which nothing is known yet; level 1 the bits below what is known down to
 * position 7; level 2 the last 7.  The histogram is left clean for the next call. */
template <int LEVEL>
__device__ __forceinline__ void pick_body(const Tables &t, uint32_t *__restrict__ hist, uint32_t *__restrict__ err, uint32_t b)
{
    constexpr int NB = LEVEL == 0 ? NB0 : LEVEL == 1 ? NB1 : NB2;
    __shared__ uint32_t tmp[WG];
    const uint32_t tid = threadIdx.x;
    if (t.k[b] == 0u) return;                  /* an empty bucket: other workgroups may be writing its words (plan_empty) */
    if (t.fast[b]) return;                     /* decided from its staged elements */
    const uint32_t want = t.need[b], sh = t.sh[b];
    if (want == 0) return;
    if (LEVEL == 0 && sh != SH_NONE) return;
    DigitWalk<NB> w;
    w.load(hist + (uint64_t)b * NB, tmp);
    w.clear(hist + (uint64_t)b * NB);
    if (w.total < want) {                  /* cannot happen: the level above counted them */
        if (tid == 0) err[0] = 1u;
        return;
    }
    uint32_t digit, above, at;
    if (w.find(want, digit, above, at)) {
        t.T[b] = LEVEL == 0 ? digit : (t.T[b] << (LEVEL == 1 ? sh - (uint32_t)SH1 : 7u)) | digit;
        t.need[b] = want - above;
        if (LEVEL == 0) t.sh[b] = SH0;
    }
}

/* Exclusive scan, in place, of a dense bucket's counts per tile.  Both counts of a tile travel as
 * one 64-bit word (neither total can reach 2^32: a bucket has fewer elements), and every thread
 * takes four consecutive tiles, so a round covers 1024 tiles with one scan.
 * Totals that do not give k survivors (cannot happen: the steps before counted them) raise the flag.  coded: the
 * survivors are written and coded next, through the places written, so such a bucket is left alone from here on, like
 * one that is coded already.  (A pruning bitmap is written whole, whatever the totals say.) */
__device__ __forceinline__ void scan_body(const Tables &t, uint32_t *__restrict__ G, uint32_t *__restrict__ E, uint32_t *__restrict__ err, bool coded, uint32_t b)
{
    __shared__ uint64_t tmp[WG / 64];
    const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (t.k[b] == 0u || t.fast[b] != PATH_DENSE) return;      /* (empty: see pick_body) */
    const uint32_t t0 = t.tile0[b], t1 = t.tile0[b + 1];
    uint64_t carry = 0;
    for (uint32_t base = t0; base < t1; base += WG * 4) {
        const uint32_t i0 = base + tid * 4;
        uint64_t v[4], x = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            v[j] = i0 + j < t1 ? ((uint64_t)G[i0 + j] << 32) | (uint64_t)E[i0 + j] : 0ull;
            x += v[j];
        }
        const uint64_t own = x;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const uint32_t hi = __shfl_up((uint32_t)(x >> 32), d, 64), lo = __shfl_up((uint32_t)x, d, 64);
            if (lane >= (uint32_t)d) x += ((uint64_t)hi << 32) | (uint64_t)lo;
        }
        if (lane == 63) tmp[wave] = x;
        wg_sync();
        uint64_t before = carry, total = 0;
#pragma unroll
        for (uint32_t w = 0; w < WG / 64; ++w) { before += w < wave ? tmp[w] : 0ull; total += tmp[w]; }
        wg_sync();
        uint64_t run = before + x - own;         /* exclusive prefix of this thread's first tile */
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (i0 + j < t1) { G[i0 + j] = (uint32_t)(run >> 32); E[i0 + j] = (uint32_t)run; }
            run += v[j];
        }
        carry += total;
    }
    if (tid == 0) {
        const uint32_t above = (uint32_t)(carry >> 32), ties = (uint32_t)carry, e_b = t.need[b];
        if (above + e_b != t.k[b] || e_b > ties) {
            err[0] = 1u;
            if (coded) t.fast[b] = PATH_LEFT;
        }
    }
}

/* ------------------------------------------------------------------ dense passes */

/* Histogram of a level's digit over the dense source of the buckets on the dense passes.  A work
 * unit is FB_TILES consecutive tiles of that list, of one bucket or several; the LDS histogram is
 * flushed when the bucket changes.  The team is a workgroup per compute unit, so what bounds it is how much each
 * has in flight: FB_AHEAD tiles at a time (two 16-byte accesses per thread and tile; one tile at a time took 1.5
 * times as long as the four accesses that a tile had when it was twice as large). */
constexpr uint32_t FB_TILES = 16, FB_AHEAD = 4;
template <int LEVEL>
__device__ __forceinline__ void fb_refine_body(const float *__restrict__ r, const Tables &t,
                                               uint32_t *__restrict__ hist, uint32_t *h,
                                               uint32_t bid, uint32_t nblk)
{
    constexpr int NB = LEVEL == 0 ? NB0 : LEVEL == 1 ? NB1 : NB2;
    constexpr int Q = TILE / (4 * WG);
    constexpr uint32_t DSH = LEVEL == 0 ? SH0 : LEVEL == 1 ? SH1 : 0;
    const uint32_t tid = threadIdx.x;
    const uint32_t total = t.ftile0[t.B];
    for (uint32_t f0 = bid * FB_TILES; f0 < total; f0 += nblk * FB_TILES) {
        const uint32_t f1 = min(total, f0 + FB_TILES);
        uint32_t f = f0;
        while (f < f1) {                               /* bucket by bucket (the same in every thread) */
            const uint32_t b = find_bucket<uint32_t>(t.ftile0, t.B, f), fend = min(f1, t.ftile0[b + 1]);
            const uint32_t sh = t.sh[b];
            if (LEVEL == 0 && sh != SH_NONE) { f = fend; continue; }
            const uint32_t psh = LEVEL == 0 ? 31u : LEVEL == 1 ? sh : (uint32_t)SH1;       /* key >> psh is what is known */
            const uint32_t dmask = LEVEL == 1 ? (1u << (sh - SH1)) - 1u : NB - 1u;
            const uint32_t prefix = LEVEL == 0 ? 0u : t.T[b];
            for (int i = tid; i < NB; i += WG) h[i] = 0;
            wg_sync();
            for (; f < fend; f += FB_AHEAD) {
                float x[FB_AHEAD][Q][4];
                uint32_t m[FB_AHEAD][Q];
                const uint32_t tile = t.tile0[b] + (f - t.ftile0[b]);
                const TileGeo s = tile_geo(t, b, tile);
#pragma unroll
                for (uint32_t v = 0; v < FB_AHEAD; ++v)
#pragma unroll
                    for (int u = 0; u < Q; ++u) {
                        m[v][u] = 0u;
                        if (f + v < fend) {
                            m[v][u] = load_quad(r, s.base + (uint64_t)v * TILE + (uint64_t)(u * WG + tid) * 4, s.lo, s.hi, x[v][u]);
                            if (t.pmask) m[v][u] &= ~pruned_bits(t.pmask, tile + v, u * WG + tid);
                        }
                    }
#pragma unroll
                for (uint32_t v = 0; v < FB_AHEAD; ++v)
#pragma unroll
                    for (int u = 0; u < Q; ++u) {
                        if (f + v >= fend) continue;
                        uint32_t d[4], hit = 0;
#pragma unroll
                        for (int j = 0; j < 4; ++j) {
                            const uint32_t key = keyof(x[v][u][j]);
                            d[j] = (key >> DSH) & dmask;
                            if (((m[v][u] >> j) & 1u) && (key >> psh) == prefix) hit |= 1u << j;
                        }
                        /* runs of equal keys: one addition for the wavefront */
                        const uint32_t fd = __builtin_amdgcn_readfirstlane(d[0]);
                        if (__all(hit == 0xFu && d[0] == fd && d[1] == fd && d[2] == fd && d[3] == fd)) {
                            if ((tid & 63) == 0) atomicAdd(&h[fd], 256u);
                            continue;
                        }
#pragma unroll
                        for (int j = 0; j < 4; ++j)
                            if ((hit >> j) & 1u) atomicAdd(&h[d[j]], 1u);
                    }
            }
            f = fend;
            wg_sync();
            hist_flush(h, hist + (uint64_t)b * NB, NB);
            wg_sync();
        }
    }
}

}  // namespace

#endif
