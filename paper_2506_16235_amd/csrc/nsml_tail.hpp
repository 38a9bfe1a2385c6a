/*
 * libnsml device code, part 5: the tail of the selection.
 * Included by nsml_kernels.hip (one translation unit); not a public header.
 *
 * What the tail knows when it starts (left by the streaming pass): the bins of the window of keys, from which
 * k_select_count makes the plan: for every bucket the leading bits b0 of its k-th largest key (down to the shift of the bins that the streaming pass
 * counted) and how many of the keys that share them are still wanted; for
 * every staging segment its entries (index, value) in index order.  Entries above b0 are
 * survivors, entries below it are not, the ones that share it are the only undecided ones, and
 * they are few.
 *
 *   k_select_count   per segment: entries above b0; the keys of the undecided entries go to the bucket's list
 *   k_select_finish  per bucket, one workgroup of 1024 threads: threshold key T and tie allowance
 *                    e from those few keys (the remaining bits, histograms in LDS); per segment
 *                    the number of survivors and of threshold ties that precede it in the bucket;
 *                    per chunk of the payload the segment that holds its first survivor
 *   k_encode         PATH_CAND, per chunk of `chunk` consecutive survivors: gathers them in index
 *                    order from the staged entries into LDS, then scale, codes, packing, indices
 *                    and the residual update, all from LDS; with 16- and 32-bit values also
 *                    PATH_DENSE
 *   k_band           16- and 32-bit values: the survivors of PATH_BAND and PATH_ZERO from the dense
 *                    accumulator, tile by tile
 *   k_hard           codes, PATH_BAND / PATH_ZERO (survivors too many to stage: a band of keys around
 *                    the threshold was staged instead, or the threshold is key 0): survivors
 *                    taken from the dense accumulator and coded in one streaming pass;
 *                    PATH_DENSE: every radix step over the dense accumulator, barriers between
 *   k_quant          codes the chunks k_hard wrote uncoded
 *   k_wrest, k_whard the same machinery for the pruning bitmap of the weight stage
 * Every small kernel here is a handful of dependent memory round trips long, which is what a
 * small kernel costs on this GPU; tables that a kernel would otherwise search for (workgroup ->
 * segments, chunk -> bucket, chunk -> first segment) are therefore prepared by the kernel before.
 */
#ifndef NSML_TAIL_HPP
#define NSML_TAIL_HPP

namespace {

constexpr uint32_t SEL_THREADS = 1024;     /* k_select_finish workgroup: 16 wavefronts */
constexpr uint32_t SEL_WAVES = SEL_THREADS / 64;
constexpr uint32_t ENC_BLK = 2048;         /* survivors gathered in LDS at a time */

/* Inclusive scan over a workgroup of 16 wavefronts, total the sum of all; tmp: 16 words of LDS.  A wavefront's total comes
 * from its scan, the wavefronts before it from a scan of the 16 totals that every row of 16 lanes does for itself.
 * (With shuffles and 64-bit words a search of the digit below took 1.7 us, so 0.6.) */
__device__ __forceinline__ uint32_t scan_totals(const uint32_t *tmp, uint32_t &total)
{
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    uint32_t v = tmp[threadIdx.x & 15u];
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xF, 0xF, true);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xF, 0xF, true);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xF, 0xF, true);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xF, 0xF, true);
    total = (uint32_t)__builtin_amdgcn_readlane((int)v, 15);
    return wave ? (uint32_t)__builtin_amdgcn_readlane((int)v, (int)wave - 1) : 0u;
}
__device__ __forceinline__ uint32_t block16_incl_scan(uint32_t x, uint32_t *tmp, uint32_t &total)
{
    x = wave_incl_scan(x);
    if ((threadIdx.x & 63u) == 63u) tmp[threadIdx.x >> 6] = x;
    wg_sync();
    x += scan_totals(tmp, total);
    wg_sync();
    return x;
}

/* The digit of an LDS histogram of NB bins that holds the want-th entry counted from the top
 * digit down (1 <= want <= number of entries).  Every thread of the workgroup of 16 wavefronts must
 * call it; res (3 words of LDS) receives digit, entries in higher digits, entries in the digit.
 * Returns false (in every thread) when the histogram holds fewer than `want` entries. */
template <int NB>
__device__ __forceinline__ bool find_digit_lds(const uint32_t *h, uint32_t want, uint32_t *tmp, uint32_t *res)
{
    /* four digits per thread from the top */
    const int top = NB - 1 - (int)threadIdx.x * 4;
    uint32_t cnt[4] = {0u, 0u, 0u, 0u}, sum = 0;
    if (top >= 3) {
        const uint4 v = *reinterpret_cast<const uint4 *>(h + top - 3);
        cnt[0] = v.w; cnt[1] = v.z; cnt[2] = v.y; cnt[3] = v.x;
        sum = (cnt[0] + cnt[1]) + (cnt[2] + cnt[3]);
    }
    uint32_t total;
    uint32_t incl = wave_incl_scan(sum);
    if ((threadIdx.x & 63u) == 63u) tmp[threadIdx.x >> 6] = incl;
    wg_sync();
    incl += scan_totals(tmp, total);
    uint32_t acc = incl - sum;
    if (acc < want && want <= incl) {
        uint32_t q = 0;
#pragma unroll
        for (uint32_t i = 0; i < 3; ++i) if (q == i && acc + cnt[i] < want) { acc += cnt[i]; ++q; }
        res[0] = (uint32_t)top - q; res[1] = acc; res[2] = q == 0 ? cnt[0] : q == 1 ? cnt[1] : q == 2 ? cnt[2] : cnt[3];
    }
    wg_sync();
    return total >= want;
}

/* Largest i in [lo, hi) with f(i) <= x, for a non-decreasing f with f(lo) <= x; the whole
 * workgroup of NT threads searches, NT probes a round.  sh: one word of LDS. */
template <uint32_t NT, typename F>
__device__ __forceinline__ uint32_t wg_search_le(uint32_t lo, uint32_t hi, uint64_t x, F f, uint32_t *sh)
{
    while (hi - lo > 1) {
        const uint32_t step = (hi - lo + NT - 1u) / NT;
        const uint32_t p = lo + threadIdx.x * step, q = p + step;
        if (p < hi && f(p) <= x && (q >= hi || x < f(q))) *sh = p;
        wg_sync();
        const uint32_t np = *sh;
        wg_sync();
        lo = np;
        hi = np + step < hi ? np + step : hi;
    }
    return lo;
}

/* ------------------------------------------------------------------ k_select_count */

constexpr uint32_t SELC_ROWS = 8;          /* rows of 64 entries a wavefront has in flight */

/* Work list of k_select_count, fixed by the bucket layout: workgroup w takes segments
 * [x.y, x.z) of bucket x.x. */
__global__ __launch_bounds__(WG) void k_selmap(const uint32_t *__restrict__ sel0, const uint32_t *__restrict__ tile0,
                                               uint32_t B, uint32_t n_sel, uint32_t selSh, uint4 *__restrict__ selw)
{
    const uint32_t w = blockIdx.x * WG + threadIdx.x;
    if (w >= n_sel) return;
    const uint32_t b = find_bucket<uint32_t>(sel0, B, w);
    const uint32_t seg_lo = tile0[b], seg_hi = tile0[b + 1];
    const uint32_t s0 = seg_lo + ((w - sel0[b]) << selSh);
    selw[w] = make_uint4(b, s0, min(seg_hi, s0 + (1u << selSh)), 0u);
}

/* chunk -> bucket, fixed by the layout and (ratio, bits) */
__global__ __launch_bounds__(WG) void k_chunkmap(const uint64_t *__restrict__ C, uint32_t B, uint64_t NC,
                                                 uint32_t *__restrict__ chunk_b)
{
    const uint64_t c = (uint64_t)blockIdx.x * WG + threadIdx.x;
    if (c < NC) chunk_b[c] = find_bucket<uint64_t>(C, B, c);
}

/* a list entry: the 19 key bits below the level-0 digit, and above them the segment's number inside the workgroup */
__device__ __forceinline__ uint32_t list_entry(uint32_t key, uint32_t segl) { return (segl << SH0) | (key & ((1u << SH0) - 1u)); }

/* A staging segment that overflowed (more staged elements than a quarter of what it covers: its
 * count says so) is read from the dense accumulator instead: the elements its wavefront of the
 * streaming pass covered, in index order, minus the pruned ones.  This is their range. */
struct DenseSeg {
    uint64_t e0;         /* first element (global index) */
    uint32_t len;
};
__device__ __forceinline__ DenseSeg dense_seg(const Tables &t, uint32_t b, uint32_t ss)
{
    const TileGeo s = tile_geo(t, b, ss);
    const uint64_t z = min(s.hi, s.base + (uint64_t)TILE);
    DenseSeg d;
    d.e0 = max(s.lo, s.base);
    d.len = (uint32_t)(z - d.e0);
    return d;
}
/* whether element e (global index) of a bucket whose first tile is tile0b and starts at lo_al
 * (its offset rounded down to a multiple of 4) is pruned */
__device__ __forceinline__ bool pruned_elem(const uint32_t *__restrict__ pmask, uint32_t tile0b, uint64_t lo_al, uint64_t e)
{
    const uint64_t pos = e - lo_al;
    return (pmask[(uint64_t)(tile0b + (uint32_t)(pos / TILE)) * (TILE / 32) + (uint32_t)((pos % TILE) >> 5)] >> (pos & 31u)) & 1u;
}

/* The window's bins of large gradients, from the staged elements (and from the dense source `r` where a
 * segment overflowed): a workgroup takes the segments of one workgroup of k_select_count, 16 or 4
 * lanes each, counts in LDS and adds what it has to one of the bucket's copies.  Bound by reading the
 * staged values (419 M elements at ratio 0.5, 3 % staged: 30 us; 109 M at 0.01: 17); an overflowed segment is
 * fetched whole, and the next one while it is counted (BERT-shaped gradient at 0.1: 35 us; without the next one on its
 * way 65, one load after the other 71). */
constexpr uint32_t BINS_U = 8;             /* entries a lane has in flight */
__global__ __launch_bounds__(WG) void k_bins(Tables t, Cand c, const uint4 *__restrict__ selw, uint32_t selSh,
                                             uint32_t *__restrict__ hist, const float *__restrict__ r)
{
    __shared__ uint32_t h[NHB], hi_all;
    const uint4 wk = selw[blockIdx.x];
    const uint32_t b = wk.x, s0 = wk.y, s1 = wk.z, tid = threadIdx.x;
    const uint32_t lanes = WG >> selSh, seg = s0 + (tid >> (8u - selSh)), gl = tid & (lanes - 1u);
    const uint32_t cnt = seg < s1 ? c.cnt[seg] : 0u;
    uint32_t hi = gl == 0u && seg < s1 ? c.G[seg] : 0u;     /* elements at or above the window's top */
    const KeyPar p = t.par[b];
    uint32_t *row = hist + ((uint64_t)b * NHC + blockIdx.x % NHC) * HROW;
    if (p.x == NONE) return;                         /* no guess; the same for the whole workgroup */
    if (tid == 0) hi_all = 0u;
    wg_sync();
    hi = wave_incl_scan(hi);
    if ((tid & 63u) == 63u && hi) atomicAdd(&hi_all, hi);
    wg_sync();
    if (tid == 0 && hi_all) atomicAdd(row + NHB, hi_all);
    if (p.x == p.y) return;                          /* nothing was staged */
    if (!__syncthreads_or(cnt != 0u)) return;
    for (uint32_t i = tid; i < (uint32_t)NHB; i += WG) h[i] = 0u;
    const uint32_t top = (p.z - 1u) >> p.w;
    auto count = [&](uint32_t key) { if (key < p.z) atomicAdd(&h[min(top - (key >> p.w), (uint32_t)NHB - 1u)], 1u); };
    wg_sync();
    const uint32_t len = cnt > SEG_CAP ? 0u : cnt;
    const float *v = c.val + (uint64_t)seg * SEG_CAP;
    for (uint32_t i0 = gl; i0 < len; i0 += lanes * BINS_U) {
        float x[BINS_U];
#pragma unroll
        for (uint32_t u = 0; u < BINS_U; ++u) x[u] = i0 + u * lanes < len ? v[i0 + u * lanes] : 0.0f;
#pragma unroll
        for (uint32_t u = 0; u < BINS_U; ++u) if (i0 + u * lanes < len) count(keyof(x[u]));
    }
    if (t.ovf[b]) {                                  /* same for the whole workgroup */
        const uint32_t lane = tid & 63u;
        const uint32_t tile0b = t.tile0[b];
        const uint64_t lo_al = t.off[b] & ~3ull;
        /* which of them: a lane per segment, the same in every wavefront */
        uint64_t todo = __ballot(lane < s1 - s0 && c.cnt[s0 + min(lane, s1 - s0 - 1u)] > SEG_CAP);
        DenseSeg dn = {};
        float xn[TILE / WG];
        auto fetch = [&]() {
            dn = dense_seg(t, b, s0 + (uint32_t)__builtin_ctzll(todo));
#pragma unroll
            for (uint32_t u = 0; u < TILE / WG; ++u) { const uint32_t e = u * WG + tid; xn[u] = e < dn.len ? r[dn.e0 + e] : 0.0f; }
        };
        if (todo) fetch();
        while (todo) {
            const DenseSeg d = dn;
            float x[TILE / WG];
#pragma unroll
            for (uint32_t u = 0; u < TILE / WG; ++u) x[u] = xn[u];
            todo &= todo - 1ull;
            if (todo) fetch();                       /* the next one is on its way while this is counted */
#pragma unroll
            for (uint32_t u = 0; u < TILE / WG; ++u) {
                const uint32_t e = u * WG + tid, key = keyof(x[u]);
                if (e < d.len && key >= p.x && key < p.z && !(t.pmask && pruned_elem(t.pmask, tile0b, lo_al, d.e0 + e))) count(key);
            }
        }
    }
    wg_sync();
    hist_flush(h, row, NHB);
}

/* Every workgroup first makes its bucket's plan for itself from the window's bins, 33 KB that the L2
 * holds; a kernel of its own for it was one more that the next had to wait for (ResNet-50's 161 buckets: 9.0 + 9.9 us, so
 * 12.8; BERT's 199: 9.2 + 10.2, so 15.3; one bucket of 1 Mi elements: 6.0 + 5.4, so 7.0).
 * Then, per staging segment of the buckets decided from staged elements (PATH_CAND, PATH_BAND), with
 * b0 the leading bits of the bucket's k-th key: G = entries above b0 (plus, in band mode, the elements
 * above the band the streaming pass counted).  The keys of the entries that share b0, the only undecided
 * ones, go to the bucket's list (the undecided key bits and the segment's number inside the workgroup in one
 * word, in no particular order); a workgroup's part of it is one range, whose place and length are left in `part`:
 * its own share, or when that is too small a range of the room that the bucket's workgroups have in common (the
 * plan has counted the keys: they fit).  (With shares alone, a cluster of survivors sent the bucket to a search by
 * one thread per segment: 12 - 50 ms on 110 M elements, now 0.1; with the common room alone every workgroup waits
 * for its place in it: 3200 of them 62 us, so 36.)
 * A workgroup takes 16 or 64 consecutive segments (1 << selSh) as one list of entries, dealt to its four wavefronts row
 * by row (64 entries), so its work follows the number of entries and not the longest segment; lane l
 * of every wavefront keeps the count of segment l, from the ballots of the rows and the part of each row
 * that belongs to it.  Overflowed segments are read from the accumulator, the next one on its way while one is counted:
 * up to 16 of them are a workgroup's longest work (BERT-shaped gradient at 0.1: 42 us one after the other, so 28). */
template <bool GRAD>      /* GRAD: the gradient; else weights (nband: how many the bucket's band holds) */
__global__ __launch_bounds__(WG, 8) void k_select_count(Tables t, Cand c, const uint4 *__restrict__ selw,
                                                     const uint32_t *__restrict__ hist,
                                                     uint32_t *__restrict__ cursor, uint2 *__restrict__ part,
                                                     uint32_t *__restrict__ lkey, uint32_t *__restrict__ err, const float *__restrict__ r,
                                                     uint32_t *__restrict__ nband)
{
    __shared__ uint32_t lk[LCAP];
    __shared__ uint32_t pre[SELC_SEGS], cg[SELC_SEGS];
    __shared__ uint32_t lcur, lbase;
    const uint4 wk = selw[blockIdx.x];
    const uint32_t b = wk.x, s0 = wk.y, s1 = wk.z;
    const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    /* issued before the bucket's state is known */
    const uint32_t ms = s0 + lane;
    const bool mine = ms < s1;
    const uint32_t mcnt = mine ? c.cnt[ms] : 0u;
    uint32_t mg0 = mine ? c.G[ms] : 0u;              /* band mode: elements above the band, counted by the streaming pass */
    const KeyPar p = t.par[b];
    uint32_t path, b0, sh;                           /* b0: the key bits from position sh up */
    {
        /* the bucket's plan, made by each of its workgroups for itself, four bins of the window per thread from the top */
        const uint32_t seg0 = t.tile0[b], segs_b = t.tile0[b + 1] - seg0, want = t.k[b], ovf = t.ovf[b];
        const uint32_t *row = hist + (uint64_t)b * NHC * HROW;
        uint32_t h[4] = {0u, 0u, 0u, 0u}, n_hi = 0;
#pragma unroll
        for (uint32_t q = 0; q < NHC; ++q) {
            const uint4 v = reinterpret_cast<const uint4 *>(row + q * HROW)[tid];
            h[0] += v.x; h[1] += v.y; h[2] += v.z; h[3] += v.w;
            n_hi += row[q * HROW + NHB];
        }
        const uint32_t sum = (h[0] + h[1]) + (h[2] + h[3]);
        uint32_t incl = wave_incl_scan(sum), tot = 0;
        if (lane == 63) pre[wave] = incl;
        wg_sync();
#pragma unroll
        for (uint32_t v = 0; v < WG / 64; ++v) { incl += v < wave ? pre[v] : 0u; tot += pre[v]; }
        uint64_t acc = (uint64_t)n_hi + incl - sum;
        if (acc < want && want <= acc + sum) {       /* at most one thread */
            uint32_t i = 0;
#pragma unroll
            for (uint32_t u = 0; u < 3; ++u) if (i == u && acc + h[u] < want) { acc += h[u]; ++i; }
            cg[0] = 4u * tid + i; cg[1] = (uint32_t)acc; cg[2] = i == 0 ? h[0] : i == 1 ? h[1] : i == 2 ? h[2] : h[3];
        }
        wg_sync();
        const bool found = n_hi < want && (uint64_t)n_hi + tot >= want;
        const Plan q = GRAD ? plan_bucket(t, b, p, want, n_hi, tot, found, cg[0], cg[1], cg[2], ovf, segs_b) : plan_weights(t, p, want, found, cg[0], cg[1], cg[2], ovf, segs_b);
        if (s0 == seg0 && tid == 0) {
            if (GRAD) plan_store(t, b, q);
            else { plan_weights_store(t, b, q); nband[b] = tot; }
        }
        path = q.path; b0 = q.T; sh = q.sh;
        if (path != PATH_CAND && path != PATH_BAND) return;      /* same for the whole workgroup */
        wg_sync();                                   /* pre and cg are written again */
    }
    if (p.y == NONE) mg0 = 0u;                       /* no band was staged: the staged entries hold everything above */
    const bool dense = mcnt > SEG_CAP;               /* an overflowed segment is read from the dense accumulator, where nothing is missing */
    const uint32_t len = dense ? 0u : mcnt;
    const uint32_t seg_end = wave_incl_scan(len), seg_start = seg_end - len;
    const uint32_t total = __builtin_amdgcn_readlane(seg_end, 63);
    if (wave == 0) { pre[lane] = seg_start; cg[lane] = 0u; }
    if (tid == 0) lcur = 0u;
    wg_sync();
    uint32_t my_g = 0;
    /* an undecided key of segment s (of this workgroup) */
    auto undecided = [&](uint32_t key, uint32_t s) {
        const uint32_t at = atomicAdd(&lcur, 1u);
        if (at < LCAP) lk[at] = list_entry(key, s);
    };
    const bool crowded = total >= 32u * (s1 - s0);   /* half a row per segment and more: a wavefront takes a whole segment */
    if (crowded) {
        for (uint32_t q = wave; q < s1 - s0; q += WG / 64) {
            const uint32_t cnt = __builtin_amdgcn_readlane(len, q);
            const float *v = c.val + (uint64_t)(s0 + q) * SEG_CAP;
            float x[SEG_CAP / 64];
#pragma unroll
            for (uint32_t u = 0; u < SEG_CAP / 64; ++u) { const uint32_t i = u * 64 + lane; x[u] = i < cnt ? v[i] : 0.0f; }
            uint32_t g = 0;
#pragma unroll
            for (uint32_t u = 0; u < SEG_CAP / 64; ++u) {
                if (u * 64 >= cnt) break;            /* same for the whole wavefront */
                const uint32_t key = keyof(x[u]);
                const bool in = u * 64 + lane < cnt;
                g += __popcll(__ballot(in && (key >> sh) > b0));
                if (in && (key >> sh) == b0) undecided(key, q);
            }
            if (lane == q) my_g = g;
        }
    }
    for (uint32_t i0 = wave * 64; !crowded && i0 < total; i0 += SELC_ROWS * WG) {
        float x[SELC_ROWS];
        uint32_t sg[SELC_ROWS];
#pragma unroll
        for (uint32_t u = 0; u < SELC_ROWS; ++u) {
            const uint32_t i = i0 + u * WG + lane;
            uint32_t q = 0;                          /* the last segment that starts at or before i */
#pragma unroll
            for (uint32_t st = SELC_SEGS / 2; st >= 1; st >>= 1) q += pre[q + st] <= i ? st : 0u;
            sg[u] = q;
            x[u] = i < total ? c.val[(uint64_t)(s0 + q) * SEG_CAP + (i - pre[q])] : 0.0f;
        }
#pragma unroll
        for (uint32_t u = 0; u < SELC_ROWS; ++u) {
            const uint32_t r0 = i0 + u * WG;
            if (r0 >= total) break;                  /* same for the whole wavefront */
            const uint32_t key = keyof(x[u]);
            const bool in = r0 + lane < total;
            const uint64_t bg = __ballot(in && (key >> sh) > b0);
            /* the part of this row that belongs to segment `lane` */
            const uint32_t pa = seg_start > r0 ? min(seg_start - r0, 64u) : 0u, pz = seg_end > r0 ? min(seg_end - r0, 64u) : 0u;
            const uint64_t ma = pa >= 64u ? ~0ull : (1ull << pa) - 1ull, mz = pz >= 64u ? ~0ull : (1ull << pz) - 1ull;
            my_g += __popcll(bg & mz & ~ma);
            if (in && (key >> sh) == b0) undecided(key, sg[u]);
        }
    }
    if (my_g) atomicAdd(&cg[lane], my_g);
    /* element e of a segment that is read from the dense source, if it counts */
    auto dense_in = [&](const DenseSeg &d, uint32_t e, uint32_t key) {
        return e < d.len && key >= p.x               /* (zeros lie below a band that starts at key 1) */
               && !(t.pmask && pruned_elem(t.pmask, t.tile0[b], t.off[b] & ~3ull, d.e0 + e));
    };
    const uint64_t over = __ballot(dense);           /* the same in every wavefront */
    uint64_t todo = over;
    DenseSeg dn = {};
    float xn[TILE / WG];
    auto fetch = [&]() {
        dn = dense_seg(t, b, s0 + (uint32_t)__builtin_ctzll(todo));
#pragma unroll
        for (uint32_t u = 0; u < TILE / WG; ++u) { const uint32_t e = u * WG + tid; xn[u] = e < dn.len ? r[dn.e0 + e] : 0.0f; }
    };
    if (todo) fetch();
    while (todo) {
        const uint32_t q = (uint32_t)__builtin_ctzll(todo);
        const DenseSeg d = dn;
        float x[TILE / WG];
#pragma unroll
        for (uint32_t u = 0; u < TILE / WG; ++u) x[u] = xn[u];
        todo &= todo - 1ull;
        if (todo) fetch();                           /* the next one is on its way while this is counted */
        uint32_t g = 0;
#pragma unroll
        for (uint32_t u = 0; u < TILE / WG; ++u) {
            const uint32_t key = keyof(x[u]);
            const bool in = dense_in(d, u * WG + tid, key);
            g += __popcll(__ballot(in && (key >> sh) > b0));
            if (in && (key >> sh) == b0) undecided(key, q);
        }
        if (lane == 0) atomicAdd(&cg[q], g);
    }
    wg_sync();
    if (wave == 0 && mine) c.G[ms] = (dense ? 0u : mg0) + cg[lane];     /* of a dense one the elements above the band were counted here as well */
    const uint32_t nl = lcur, tile0b = t.tile0[b], segs = t.tile0[b + 1] - tile0b;
    uint32_t *list = lkey + list_base(tile0b, b);
    const bool alone = s1 - s0 == segs;              /* the bucket's only workgroup: all of the list is its own */
    if (nl <= (s1 - s0) * OWN_PER_SEG || (alone && nl <= LCAP)) {
        const uint32_t at = (s0 - tile0b) * OWN_PER_SEG;
        if (tid == 0) part[blockIdx.x] = make_uint2(at, nl);
        for (uint32_t i = tid; i < nl; i += WG) list[at + i] = lk[i];
        return;
    }
    wg_sync();
    if (tid == 0) {
        const uint32_t at = atomicAdd(&cursor[b], nl);
        const bool fits = (uint64_t)at + nl <= list_room(segs);
        if (!fits) err[0] = 1u;                      /* cannot happen: the plan has counted them */
        part[blockIdx.x] = make_uint2(segs * OWN_PER_SEG + at, fits ? nl : 0u);
        lbase = fits ? at : NONE;
        lcur = 0u;
    }
    wg_sync();
    if (lbase == NONE) return;
    list += segs * OWN_PER_SEG + lbase;
    if (nl <= LCAP) {
        for (uint32_t i = tid; i < nl; i += WG) list[i] = lk[i];
        return;
    }
    /* rare: more of them than LDS holds; gone through once more, to their places in memory at once */
    auto store = [&](bool is, uint32_t key, uint32_t s) {
        const uint64_t bal = __ballot(is);
        if (!bal) return;                            /* same for the whole wavefront */
        uint32_t at = 0;
        if (lane == 0) at = atomicAdd(&lcur, (uint32_t)__popcll(bal));
        at = __builtin_amdgcn_readfirstlane(at);
        at = __builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bal, at));
        if (is) list[at] = list_entry(key, s);
    };
#pragma unroll 1
    for (uint32_t q = wave; q < s1 - s0; q += WG / 64) {
        if ((over >> q) & 1ull) {
            const DenseSeg d = dense_seg(t, b, s0 + q);
#pragma unroll 1
            for (uint32_t e0 = 0; e0 < d.len; e0 += 64) {
                const uint32_t e = e0 + lane, key = e < d.len ? keyof(r[d.e0 + e]) : 0u;
                store(dense_in(d, e, key) && (key >> sh) == b0, key, q);
            }
        } else {
            const uint32_t cnt = __builtin_amdgcn_readlane(len, q);
#pragma unroll 1
            for (uint32_t e0 = 0; e0 < cnt; e0 += 64) {
                const uint32_t e = e0 + lane, key = e < cnt ? keyof(c.val[(uint64_t)(s0 + q) * SEG_CAP + e]) : 0u;
                store(e < cnt && (key >> sh) == b0, key, q);
            }
        }
    }
}

/* ------------------------------------------------------------------ k_select_finish */

/* LDS of k_select_finish, one pool (u32 words):
 *   [0, 4096)        level-1 histogram; later the counts of up to FIN_MAX_SEGS segments
 *   FIN_AT_KEYS      undecided keys, when all of the bucket's fit
 *   FIN_AT_SEGS      their segment numbers as u16
 *   FIN_AT_UPRE      exclusive prefix of the lengths of the list's parts
 *   FIN_AT_UPOS      where each part begins in the list */
constexpr uint32_t FIN_KEYS_LDS = 3072;    /* undecided keys kept in LDS */
constexpr uint32_t FIN_MAX_SEGS = 16384;   /* segments whose counts fit the pool: larger buckets go in windows of so many */
constexpr uint32_t FIN_AT_KEYS = FIN_MAX_SEGS, FIN_AT_SEGS = FIN_AT_KEYS + FIN_KEYS_LDS, FIN_AT_UPRE = FIN_AT_SEGS + FIN_KEYS_LDS / 2;
constexpr uint32_t FIN_AT_UPOS = FIN_AT_UPRE + SEL_THREADS + 1;
constexpr uint32_t FIN_POOL = FIN_AT_UPOS + SEL_THREADS;
static_assert(NB1 <= FIN_MAX_SEGS, "the level-1 histogram overlaps the keys");

/* Exclusive prefixes of (elements above T, elements equal to T) over the segments [seg_lo, seg_hi) of a
 * bucket, in place over the per-segment counts, and for every chunk of the payload the segment that holds
 * its first survivor.  A round takes PER consecutive segments per thread.  run: the two totals of the
 * segments before, brought up to date.  count(s, g, q) adds to g and q what segment s holds above / equal
 * to T among its undecided keys. */
template <uint32_t PER, typename F>
__device__ __forceinline__ void finish_prefixes(const Tables &t, const Cand &c, uint32_t b, uint32_t seg_lo,
                                                uint32_t seg_hi, uint32_t e_b, uint32_t &run_g, uint32_t &run_e,
                                                uint32_t *__restrict__ chunk_seg, uint32_t *tmp, F count)
{
    const uint32_t tid = threadIdx.x, wave = tid >> 6;
    const uint32_t rounds = (seg_hi - seg_lo + SEL_THREADS * PER - 1) / (SEL_THREADS * PER);
    uint32_t *first = chunk_seg ? chunk_seg + t.C[b] : nullptr;
    const uint32_t chunk = t.chunk, chunkSh = t.chunkSh;
    uint32_t g_next[PER];
#pragma unroll
    for (uint32_t j = 0; j < PER; ++j) { const uint32_t s = seg_lo + tid * PER + j; g_next[j] = s < seg_hi ? c.G[s] : 0u; }
    for (uint32_t r = 0; r < rounds; ++r) {
        const uint32_t s0 = seg_lo + (r * SEL_THREADS + tid) * PER;
        uint32_t vg[PER], ve[PER], sum_g = 0, sum_e = 0;
#pragma unroll
        for (uint32_t j = 0; j < PER; ++j) {
            uint32_t g = g_next[j], q = 0;
            if (r + 1 < rounds) { const uint32_t sn = s0 + SEL_THREADS * PER + j; g_next[j] = sn < seg_hi ? c.G[sn] : 0u; }   /* fetched under this round's work */
            count(s0 + j, g, q);
            vg[j] = g; ve[j] = q;
            sum_g += g; sum_e += q;
        }
        uint32_t Gp = wave_incl_scan(sum_g), Ep = wave_incl_scan(sum_e), tot_g, tot_e;
        if ((tid & 63u) == 63u) { tmp[wave] = Gp; tmp[SEL_WAVES + wave] = Ep; }
        wg_sync();
        Gp += run_g + scan_totals(tmp, tot_g) - sum_g;
        Ep += run_e + scan_totals(tmp + SEL_WAVES, tot_e) - sum_e;
#pragma unroll
        for (uint32_t j = 0; j < PER; ++j) {
            const uint32_t s = s0 + j;
            if (s < seg_hi) {
                c.G[s] = Gp;
                c.E[s] = Ep;
                /* survivors of this segment have ranks [r0, r1): the chunks that start among them */
                const uint32_t r0 = Gp + min(e_b, Ep), r1 = Gp + vg[j] + min(e_b, Ep + ve[j]);
                if (first && r1 > r0)                    /* not for the weight stage: its ranks are no payload positions */
                    for (uint64_t cb = chunkSh < 32u ? ((uint64_t)r0 + chunk - 1u) >> chunkSh : ((uint64_t)r0 + chunk - 1u) / chunk; cb * chunk < r1; ++cb) first[cb] = s;
            }
            Gp += vg[j];
            Ep += ve[j];
        }
        run_g += tot_g;
        run_e += tot_e;
        wg_sync();                                       /* tmp is written again */
    }
}
/* The bucket's threshold and tie allowance, once its prefixes are done. */
__device__ __forceinline__ void finish_state(const Tables &t, uint32_t b, uint32_t T, uint32_t e_b, uint32_t kb, uint32_t above, uint32_t ties,
                                             uint32_t *__restrict__ err)
{
    if (threadIdx.x != 0) return;
    t.T[b] = T;
    t.need[b] = e_b;
    /* above + admitted ties must be exactly k */
    if (above + e_b != kb || e_b > ties) err[0] = 1u;
}

/* add to a word of LDS that many active lanes of the wavefront may share (equal keys): one addition then */
__device__ __forceinline__ void add_shared(uint32_t *h, uint32_t at, uint32_t add)
{
    const uint32_t fa = __builtin_amdgcn_readfirstlane(at), fv = __builtin_amdgcn_readfirstlane(add);
    const uint64_t here = __ballot(true);
    if (__ballot(at == fa && add == fv) == here) {
        if ((threadIdx.x & 63u) == (uint32_t)__builtin_ctzll(here)) atomicAdd(&h[fa], fv * (uint32_t)__popcll(here));
    } else {
        atomicAdd(&h[at], add);
    }
}

/* One workgroup of 1024 threads per bucket decided from staged elements: the threshold key T and
 * the tie allowance e from the bucket's undecided keys (12 + 7 remaining bits, histograms in LDS),
 * then every segment's place in the survivor order.  The keys are read once per step, four per thread in
 * flight, and kept in LDS when they fit.  A bucket of more than FIN_MAX_SEGS segments goes through every step
 * in windows of so many, a range of the list's parts each (110 M elements in one bucket, 0.1 %: 93 us; by one
 * thread per segment 264).  Bound by the latency of its steps: with scans by data-parallel moves, 32-bit prefixes and shifts for
 * the chunk numbers 8.1 us for ResNet-50's 161 buckets, 16 for BERT's 199, 7.4 for one of 1 Mi elements; with
 * shuffles, 64-bit words and 64-bit divisions 12.7, 22, 11.3.  PATH_ZERO buckets arrive with T = 0 and e known and only get the
 * prefixes.  in_windows: diagnostic, windows of two parts and nothing kept in LDS. */
__global__ __launch_bounds__(SEL_THREADS) void k_select_finish(Tables t, Cand c, const uint32_t *__restrict__ sel0, uint32_t selSh,
                                                               uint32_t *__restrict__ cursor, const uint2 *__restrict__ part,
                                                               const uint32_t *__restrict__ lkey,
                                                               uint32_t *__restrict__ chunk_seg,
                                                               uint32_t *__restrict__ err, int in_windows)
{
    __shared__ __align__(16) uint32_t pool[FIN_POOL];
    __shared__ __align__(16) uint32_t h2[NB2];
    __shared__ uint32_t tmp[2 * SEL_WAVES];
    __shared__ uint32_t res[4];
    const uint32_t b = blockIdx.x, tid = threadIdx.x;
    const uint32_t path = t.fast[b], kb = t.k[b];
    const uint32_t u0 = sel0[b], nun = sel0[b + 1] - u0;
    const uint32_t in_room = cursor[b];
    const uint32_t wun = in_windows ? 2u : min(SEL_THREADS, FIN_MAX_SEGS >> selSh);      /* parts per window */
    /* the first window's part of this thread, fetched before the bucket's state is known */
    uint2 mine = tid < min(nun, wun) ? part[u0 + tid] : make_uint2(0u, 0u);
    if (path == PATH_DENSE || kb == 0u) return;
    const uint32_t seg_lo = t.tile0[b], seg_hi = t.tile0[b + 1];
    const uint32_t b0 = t.T[b];                      /* the key bits from position sh up; PATH_ZERO: the full key (0) */
    const uint32_t need0 = t.need[b], sh = t.sh[b];
    uint32_t run_g = 0, run_e = 0;
    if (path == PATH_ZERO) {
        /* the streaming pass counted non-zero (G) and zero (E) keys per segment; when a band from
         * key 1 up was staged as well, G holds the keys above the band and the staged ones add to it */
        const bool mixed = t.par[b].x != t.par[b].y;
        finish_prefixes<4>(t, c, b, seg_lo, seg_hi, need0, run_g, run_e, chunk_seg, tmp,
                        [&](uint32_t s, uint32_t &g, uint32_t &q) {
                            if (s < seg_hi) { q += c.E[s]; if (mixed) g += c.cnt[s]; }
                        });
        finish_state(t, b, 0u, need0, kb, run_g, run_e, err);
        return;
    }
    uint32_t *h1 = pool, *cnts = pool, *keys = pool + FIN_AT_KEYS, *upre = pool + FIN_AT_UPRE, *upos = pool + FIN_AT_UPOS;
    uint16_t *segs = reinterpret_cast<uint16_t *>(pool + FIN_AT_SEGS);
    const uint32_t *list = lkey + list_base(seg_lo, b);
    for (uint32_t i = tid; i < NB1; i += SEL_THREADS) h1[i] = 0u;
    if (tid < NB2) h2[tid] = 0u;
    wg_sync();
    if (tid == 0 && in_room) cursor[b] = 0u;         /* every thread has read it: left clean for the next call */
    const bool one = nun <= wun;
    const uint32_t m1 = (1u << (sh - SH1)) - 1u;     /* level-1 digit: key bits sh-1 .. 7 (at most 12) */
    /* the parts [w0, w0 + wn) of the list: their prefixes and places to LDS; returns how many keys they hold */
    auto window = [&](uint32_t w0) {
        const uint32_t wn = min(wun, nun - w0);
        if (!one) mine = tid < wn ? part[u0 + w0 + tid] : make_uint2(0u, 0u);
        uint32_t tot;
        const uint32_t incl = block16_incl_scan(mine.y, tmp, tot);      /* (the window before has been consumed, too) */
        if (tid < wn) { upre[tid] = incl - mine.y; upos[tid] = mine.x; }
        if (tid == 0) upre[wn] = tot;
        wg_sync();
        return tot;
    };
    /* f(i, entry, segment number inside the window) for the n keys of the window */
    auto for_keys = [&](uint32_t w0, uint32_t n, auto f) {
        const uint32_t wn = min(wun, nun - w0);
        if (n >= 128u * wn) {
            /* long parts (many ties): a wavefront each, no search for a key's part */
#pragma unroll 1
            for (uint32_t q = tid >> 6; q < wn; q += SEL_WAVES) {
                const uint32_t i1 = upre[q + 1], shift = upos[q] - upre[q];
#pragma unroll 1
                for (uint32_t i0 = upre[q] + (tid & 63u); i0 < i1; i0 += 4 * 64) {
                    uint32_t e[4];
#pragma unroll
                    for (uint32_t u = 0; u < 4; ++u) { const uint32_t i = i0 + u * 64; e[u] = i < i1 ? list[shift + i] : 0u; }
#pragma unroll
                    for (uint32_t u = 0; u < 4; ++u) { const uint32_t i = i0 + u * 64; if (i < i1) f(i, e[u], (q << selSh) + (e[u] >> SH0)); }
                }
            }
            return;
        }
#pragma unroll 1
        for (uint32_t i0 = tid; i0 < n; i0 += 4 * SEL_THREADS) {
            uint32_t e[4], un[4];
#pragma unroll
            for (uint32_t u = 0; u < 4; ++u) {
                const uint32_t i = i0 + u * SEL_THREADS;
                e[u] = un[u] = 0u;
                if (i < n) {
                    uint32_t lo = 0, hi = wn;            /* upre[lo] <= i < upre[hi] */
                    while (hi - lo > 1) { const uint32_t mid = (lo + hi) >> 1; if (upre[mid] <= i) lo = mid; else hi = mid; }
                    un[u] = lo;
                    e[u] = list[upos[lo] + (i - upre[lo])];
                }
            }
#pragma unroll
            for (uint32_t u = 0; u < 4; ++u)
                if (i0 + u * SEL_THREADS < n) f(i0 + u * SEL_THREADS, e[u], (un[u] << selSh) + (e[u] >> SH0));
        }
    };
    bool resident = false;
    uint32_t n0 = 0;
    for (uint32_t w0 = 0; w0 < nun; w0 += wun) {
        const uint32_t n = n0 = window(w0);
        resident = one && n <= FIN_KEYS_LDS && !in_windows;
        for_keys(w0, n, [&](uint32_t i, uint32_t e, uint32_t seg) {
            add_shared(h1, (e >> SH1) & m1, 1u);
            if (resident) { keys[i] = e; segs[i] = (uint16_t)seg; }
        });
    }
    wg_sync();
    if (!find_digit_lds<NB1>(h1, need0, tmp, res)) { if (tid == 0) err[0] = 1u; return; }
    const uint32_t d1 = res[0];
    const uint32_t need1 = need0 - res[1];
    auto last_digit = [&](uint32_t e) { if (((e >> SH1) & m1) == d1) add_shared(h2, e & (NB2 - 1), 1u); };
    if (resident) {
        for (uint32_t i = tid; i < n0; i += SEL_THREADS) last_digit(keys[i]);
    } else {
        for (uint32_t w0 = 0; w0 < nun; w0 += wun) for_keys(w0, one ? n0 : window(w0), [&](uint32_t, uint32_t e, uint32_t) { last_digit(e); });
    }
    wg_sync();
    if (!find_digit_lds<NB2>(h2, need1, tmp, res)) { if (tid == 0) err[0] = 1u; return; }
    const uint32_t d2 = res[0];
    const uint32_t T = (b0 << sh) | (d1 << SH1) | d2;
    const uint32_t e_b = need1 - res[1];             /* ties admitted: 1 <= e_b <= keys equal to T */
    const uint32_t low = (1u << sh) - 1u, Tlow = T & low;      /* the undecided bits */
    for (uint32_t w0 = 0; w0 < nun; w0 += wun) {
        const uint32_t wn = min(wun, nun - w0);
        const uint32_t s_lo = seg_lo + (w0 << selSh), s_hi = min(seg_hi, s_lo + (wn << selSh));
        const uint32_t n = one ? n0 : window(w0);
        for (uint32_t i = tid; i < s_hi - s_lo; i += SEL_THREADS) cnts[i] = 0u;       /* takes the place of the level-1 histogram */
        wg_sync();
        /* per segment: keys above T (high half of its count) and equal to it */
        auto tally = [&](uint32_t e, uint32_t seg) {
            const uint32_t v = e & low;
            if (v >= Tlow) add_shared(cnts, seg, v > Tlow ? 1u << 16 : 1u);
        };
        if (resident) {
            for (uint32_t i = tid; i < n; i += SEL_THREADS) tally(keys[i], segs[i]);
        } else {
            for_keys(w0, n, [&](uint32_t, uint32_t e, uint32_t seg) { tally(e, seg); });
        }
        wg_sync();
        finish_prefixes<4>(t, c, b, s_lo, s_hi, e_b, run_g, run_e, chunk_seg, tmp,
                        [&](uint32_t s, uint32_t &g, uint32_t &q) {
                            if (s < s_hi) { const uint32_t v = cnts[s - s_lo]; g += v >> 16; q += v & 0xFFFFu; }
                        });
    }
    finish_state(t, b, T, e_b, kb, run_g, run_e, err);
}

/* ------------------------------------------------------------------ gather from the staged entries */

constexpr uint32_t CU = 4;                 /* entries of a segment a lane fetches at a time */

/* The survivors with ranks in [j0, j0 + n) out of segments [sA, sEnd) of a PATH_CAND bucket go to
 * sv / si.  GROUP lanes share a segment and SB segments per group are in flight: their counts and
 * prefixes, then the first batch of entries of each.  An entry above T, or an admitted tie, has
 * rank G + min(e, E), with G / E the numbers of entries above / equal to T before it: the prefixes
 * k_select_finish left per segment, then ballots, so nothing crosses wavefronts.  Returns how many
 * survivors this thread placed. */
template <uint32_t ENC_T, uint32_t GROUP, uint32_t SB>
__device__ __forceinline__ uint32_t gather_segments(const Cand &c, uint32_t sA, uint32_t sEnd, uint32_t T, uint32_t e_b,
                                                    uint32_t j0, uint32_t n, const uint32_t *meta, float *sv, uint32_t *si)
{
    constexpr uint32_t GROUPS = ENC_T / GROUP;       /* segments the workgroup works on side by side */
    const uint32_t tid = threadIdx.x, lane = tid & 63, gl = lane % GROUP, shift = lane - gl;
    const uint64_t below = (1ull << gl) - 1ull;
    const uint64_t gmask = GROUP == 64 ? ~0ull : ((1ull << (GROUP % 64)) - 1ull);
    uint32_t got = 0;
    for (uint32_t q0 = sA; q0 < sEnd; q0 += GROUPS * SB) {
        uint32_t cnt[SB], rg[SB], re[SB];
#pragma unroll
        for (uint32_t v = 0; v < SB; ++v) {
            const uint32_t s = q0 + v * GROUPS + tid / GROUP, at = s - sA;
            cnt[v] = rg[v] = re[v] = 0;
            if (s < sEnd) { cnt[v] = meta[at]; rg[v] = meta[ENC_T + at]; re[v] = meta[2u * ENC_T + at]; }
        }
        float x[SB][CU];
        uint32_t li[SB][CU];
        auto fetch = [&](uint32_t v, uint32_t i0) {
            const uint64_t base = (uint64_t)(q0 + v * GROUPS + tid / GROUP) * SEG_CAP + (i0 + gl);
            const float *pv = c.val + base;
            const uint32_t *pi = c.idx + base;
#pragma unroll
            for (uint32_t u = 0; u < CU; ++u) {
                const bool in = i0 + gl + u * GROUP < cnt[v];
                x[v][u] = in ? pv[u * GROUP] : 0.0f;
                li[v][u] = in ? pi[u * GROUP] : 0u;
            }
        };
#pragma unroll
        for (uint32_t v = 0; v < SB; ++v) fetch(v, 0);
#pragma unroll
        for (uint32_t v = 0; v < SB; ++v) {
            for (uint32_t i0 = 0;;) {
#pragma unroll
                for (uint32_t u = 0; u < CU; ++u) {
                    const uint32_t key = keyof(x[v][u]);
                    const bool in = i0 + u * GROUP + gl < cnt[v];
                    const bool isg = in && key > T, ise = in && key == T;
                    const uint64_t bg = (__ballot(isg) >> shift) & gmask;
                    const uint64_t be = (__ballot(ise) >> shift) & gmask;
                    const uint32_t pg = rg[v] + __popcll(bg & below), pe = re[v] + __popcll(be & below);
                    if (isg || (ise && pe < e_b)) {
                        const uint64_t slot = (uint64_t)pg + (uint64_t)min(e_b, pe) - (uint64_t)j0;   /* wraps below j0 */
                        if (slot < (uint64_t)n) { sv[slot] = x[v][u]; si[slot] = li[v][u]; ++got; }
                    }
                    rg[v] += __popcll(bg);
                    re[v] += __popcll(be);
                }
                i0 += CU * GROUP;
                if (!__any(i0 < cnt[v])) break;
                fetch(v, i0);
            }
        }
    }
    return got;
}

/* Gather survivors number [j0, j0 + n) of a PATH_CAND bucket (n <= ENC_BLK), in index order,
 * into LDS: sv their accumulator values, si their bucket-local indices.  sA = the segment that holds
 * survivor j0, sEnd = one past the last that can hold any of them.  How many lanes share a segment
 * follows how many survivors a segment holds on average: two at ratio 0.001, two hundred at 0.1.
 * (One list of entries over all segments, dealt evenly to the lanes by a search of the segment in
 * LDS, follows the work more closely and was slower: 178 us against 142 at ratio 0.1 on 109 M
 * elements, the searches alone keep the LDS busy.)  filled (LDS) counts what was placed. */
template <uint32_t ENC_T>
__device__ __forceinline__ void gather_survivors(const Cand &c, uint32_t sA, uint32_t sEnd, uint32_t T, uint32_t e_b, uint32_t j0,
                                                 uint32_t n, uint32_t *meta, float *sv, uint32_t *si, uint32_t *filled)
{
    const uint32_t m = sEnd - sA;
    uint32_t got = 0;
    for (uint32_t s0 = sA; s0 < sEnd; s0 += ENC_T) {
        /* counts and prefixes of up to ENC_T segments at once, not a memory round trip for every few of them (one bucket of 1 Mi elements: 12.3 us, so 11.5) */
        const uint32_t s = s0 + threadIdx.x, s1 = min(sEnd, s0 + ENC_T);
        if (s0 != sA) wg_sync();                     /* meta is written again */
        if (s < s1) { meta[threadIdx.x] = c.cnt[s]; meta[ENC_T + threadIdx.x] = c.G[s]; meta[2u * ENC_T + threadIdx.x] = c.E[s]; }
        wg_sync();
        if (n >= 24u * m) got += gather_segments<ENC_T, 64, 2>(c, s0, s1, T, e_b, j0, n, meta, sv, si);
        else if (n >= 6u * m) got += gather_segments<ENC_T, 16, 2>(c, s0, s1, T, e_b, j0, n, meta, sv, si);
        else got += gather_segments<ENC_T, 4, 4>(c, s0, s1, T, e_b, j0, n, meta, sv, si);
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) got += __shfl_xor(got, d, 64);
    if ((threadIdx.x & 63u) == 0u && got) atomicAdd(filled, got);
}

/* Codes of four values: rint(x / scale) of the correctly rounded quotient, clamped; 0 where the scale is.
 * The product with the reciprocal differs from that quotient by less than 4e-5 (v_rcp_f32 is
 * good to 2^-23, the two roundings add 2^-23, and the quotient is below 128.5), so away from the middle between two codes it gives the same code; the few
 * values near one, and what is not a finite number, are divided. */
template <int BITS>
__device__ __forceinline__ void quantize_four(const float (&x)[4], float scale, int (&q)[4])
{
    constexpr float QMAX = BITS == 8 ? 127.0f : 7.0f;
    const float inv = __builtin_amdgcn_rcpf(scale);
    bool sure = true;
    float w[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const float y = __fmul_rn(x[j], inv);
        w[j] = rintf(y);
        sure = sure && fabsf(__fsub_rn(y, w[j])) < 0.4999f;      /* (false for NaN) */
    }
    if (!sure) {
#pragma unroll
        for (int j = 0; j < 4; ++j) w[j] = scale != 0.0f ? rintf(__fdiv_rn(x[j], scale)) : 0.0f;
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) q[j] = (int)fminf(fmaxf(w[j], -QMAX), QMAX);
}

/* Largest over the wavefront, the same in all lanes. */
template <int CTRL, int ROWS>
__device__ __forceinline__ float dpp_max(float v)
{
    const int i = __float_as_int(v);
    return fmaxf(v, __int_as_float(__builtin_amdgcn_update_dpp(i, i, CTRL, ROWS, 0xF, false)));
}
__device__ __forceinline__ float wave_max(float v)
{
    v = dpp_max<0x111, 0xF>(v);
    v = dpp_max<0x112, 0xF>(v);
    v = dpp_max<0x114, 0xF>(v);
    v = dpp_max<0x118, 0xF>(v);
    v = dpp_max<0x142, 0xA>(v);
    v = dpp_max<0x143, 0xC>(v);
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}

/* ------------------------------------------------------------------ the dense accumulator */

/* Ordered write for the buckets whose survivors are taken from the dense accumulator (PATH_BAND,
 * PATH_ZERO, and PATH_DENSE once its own passes have left T, e and the per-segment prefixes):
 * one wavefront per staging segment walks the elements the segment covers, in index order, and writes the
 * survivors' indices and values to their final slots.  Ranks inside a row of 64 lanes x 4
 * elements come from ballots; nothing crosses wavefronts.  which: bit p set = serve PATH p. */
__device__ __forceinline__ void write_dense_body(const float *__restrict__ r, const Tables &t, const Cand &c,
                                                 uint32_t *__restrict__ idx_out, float *__restrict__ v_out,
                                                 uint32_t which, uint32_t bid, uint32_t nblk)
{
    const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (uint32_t ss = bid * (WG / 64) + wave; ss < t.n_tiles; ss += nblk * (WG / 64)) {
    const uint32_t b = t.tile_b[ss];
    const uint32_t path = t.fast[b];
    if (!((which >> path) & 1u) || t.k[b] == 0u) continue;
    const TileGeo s = tile_geo(t, b, ss);
    const uint32_t T = t.T[b], e_b = t.need[b];
    const uint64_t Pb = t.P[b];
    uint32_t run_g = c.G[ss], run_e = c.E[ss];
    const uint64_t lt = (1ull << lane) - 1ull;
    constexpr uint32_t wt0 = 0, wt1 = TILE / WTILE;
    /* the next wave-tile (64 lanes x 4 rows x 4 elements) is fetched while this one is written */
    float xn[4][4];
    uint32_t mn[4];
    auto fetch = [&](uint32_t wt) {
        const uint64_t wb = s.base + (uint64_t)wt * WTILE;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const uint64_t gi = wb + (uint64_t)(u * 64 + lane) * 4;
            mn[u] = load_quad(r, gi, s.lo, s.hi, xn[u]);
            if (t.pmask) mn[u] &= ~pruned_bits(t.pmask, ss, wt * WG + u * 64 + lane);
        }
    };
    fetch(wt0);
    for (uint32_t wt = wt0; wt < wt1; ++wt) {
        const uint64_t wb = s.base + (uint64_t)wt * WTILE;
        float x[4][4];
        uint32_t m[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            m[u] = mn[u];
#pragma unroll
            for (int j = 0; j < 4; ++j) x[u][j] = xn[u][j];
        }
        if (wt + 1 < wt1) fetch(wt + 1);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const uint64_t gi = wb + (uint64_t)(u * 64 + lane) * 4;
            uint32_t fg = 0, fe = 0;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint32_t key = keyof(x[u][j]);
                if ((m[u] >> j) & 1u) { fg |= (key > T ? 1u : 0u) << j; fe |= (key == T ? 1u : 0u) << j; }
            }
            /* entries of lower lanes come first, then this lane's own four in order */
            uint32_t pg = run_g, pe = run_e, tg = 0, te = 0;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint64_t bg = __ballot((fg >> j) & 1u), be = __ballot((fe >> j) & 1u);
                pg += __popcll(bg & lt); pe += __popcll(be & lt);
                tg += __popcll(bg); te += __popcll(be);
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const bool isg = (fg >> j) & 1u, ise = (fe >> j) & 1u;
                if (isg || (ise && pe < e_b)) {
                    const uint64_t pos = Pb + pg + min(e_b, pe);
                    idx_out[pos] = (uint32_t)(gi + j - s.lo);
                    v_out[pos] = x[u][j];
                }
                pg += isg ? 1u : 0u;
                pe += ise ? 1u : 0u;
            }
            run_g += tg;
            run_e += te;
        }
    }
    }
}

/* PATH_DENSE buckets, after their own passes have found T and e: elements above and equal to T
 * per staging segment (one wavefront per segment), the counts the scan turns into prefixes. */
__device__ __forceinline__ void segcount_dense_body(const float *__restrict__ r, const Tables &t, const Cand &c,
                                                    uint32_t bid, uint32_t nblk)
{
    const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (uint32_t ss = bid * (WG / 64) + wave; ss < t.n_tiles; ss += nblk * (WG / 64)) {
    const uint32_t b = t.tile_b[ss];
    if (t.fast[b] != PATH_DENSE || t.k[b] == 0u) continue;
    const TileGeo s = tile_geo(t, b, ss);
    const uint32_t T = t.T[b];
    uint32_t ng = 0, ne = 0;
    float x[TILE / 256][4];
    uint32_t m[TILE / 256];
#pragma unroll
    for (int u = 0; u < TILE / 256; ++u) {             /* all of the tile in flight */
        m[u] = load_quad(r, s.base + (uint64_t)(u * 64 + lane) * 4, s.lo, s.hi, x[u]);
        if (t.pmask) m[u] &= ~pruned_bits(t.pmask, ss, u * 64 + lane);
    }
#pragma unroll
    for (int u = 0; u < TILE / 256; ++u)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint32_t key = keyof(x[u][j]);
            const bool ok = (m[u] >> j) & 1u;
            ng += (ok && key > T) ? 1u : 0u;
            ne += (ok && key == T) ? 1u : 0u;
        }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) { ng += __shfl_xor(ng, d, 64); ne += __shfl_xor(ne, d, 64); }
    if (lane == 0) { c.G[ss] = ng; c.E[ss] = ne; }
    }
}

/* The buckets whose staged elements could not decide them (PATH_DENSE: an unlucky sample, a
 * staging segment that overflowed, a huge group of equal keys), in ONE launch of a fixed, small
 * grid whose workgroups meet at barriers between the steps: threshold, counts and prefixes
 * (dense_threshold), ordered write.  In the usual case there is no such bucket: each workgroup reads one
 * word and leaves, so the whole chain costs a single empty launch per call.
 * A barrier is an arrival counter in memory: every wavefront waits for its own stores, one thread
 * per workgroup then makes them visible device wide, counts the workgroup in and waits until all
 * have arrived, and drops what the caches hold afterwards.  The grid is small enough to be
 * resident at once; the wait is bounded by a clock all the same, and running out raises the
 * consistency flag. */
constexpr unsigned long long HARD_SPIN_TICKS = 500000000ull;      /* 5 s of the 100 MHz wall clock */

__device__ __forceinline__ void grid_barrier(uint32_t *bar, uint32_t target, uint32_t *__restrict__ err)
{
    __builtin_amdgcn_s_waitcnt(0);                   /* this wavefront's stores have reached the L2 */
    wg_sync();
    if (threadIdx.x == 0) {
        __threadfence();                             /* write the L2 back: visible to the other dies */
        __builtin_amdgcn_s_waitcnt(0);               /* ... before the arrival is: the compiler, which sees no access in flight here, leaves the fence's own wait out */
        __hip_atomic_fetch_add(bar, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const unsigned long long t0 = wall_clock64();
        while (__hip_atomic_load(bar, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < target) {
            __builtin_amdgcn_s_sleep(32);
            if (wall_clock64() - t0 > HARD_SPIN_TICKS) { err[0] = 1u; break; }
        }
        __threadfence();                             /* and nothing stale is read afterwards, by the other wavefronts either */
        __builtin_amdgcn_s_waitcnt(0);
    }
    wg_sync();
}

/* Threshold key, tie allowance and prefixes per tile of the buckets on the dense passes, by a team of
 * nblk resident workgroups: list of their tiles, then per level a histogram over the source and its
 * digit (the first one only where a bucket's leading bits are not known from the counts), then counts per tile and
 * their prefixes, with a barrier after each step.  h: NB0 words of LDS.  coded: see scan_body. */
__device__ __forceinline__ void dense_threshold(const float *__restrict__ r, const Tables &t, const Cand &c, uint32_t *__restrict__ f0,
                                                uint32_t *__restrict__ f1, uint32_t *__restrict__ f2, uint32_t *h, uint32_t *bar,
                                                uint32_t bid, uint32_t nblk, bool coded, uint32_t *__restrict__ err)
{
    uint32_t arrivals = 0;
    if (bid == 0) fb_plan_body(t);
    grid_barrier(bar, arrivals += nblk, err);
    if (t.nhard[3] != 0u) {                          /* (not written any more in this launch: the same in the whole team) */
        fb_refine_body<0>(r, t, f0, h, bid, nblk);
        grid_barrier(bar, arrivals += nblk, err);
        for (uint32_t b = bid; b < t.B; b += nblk) { wg_sync(); pick_body<0>(t, f0, err, b); }
        grid_barrier(bar, arrivals += nblk, err);
    }
    fb_refine_body<1>(r, t, f1, h, bid, nblk);
    grid_barrier(bar, arrivals += nblk, err);
    for (uint32_t b = bid; b < t.B; b += nblk) { wg_sync(); pick_body<1>(t, f1, err, b); }
    grid_barrier(bar, arrivals += nblk, err);
    fb_refine_body<2>(r, t, f2, h, bid, nblk);
    grid_barrier(bar, arrivals += nblk, err);
    for (uint32_t b = bid; b < t.B; b += nblk) { wg_sync(); pick_body<2>(t, f2, err, b); }
    grid_barrier(bar, arrivals += nblk, err);
    segcount_dense_body(r, t, c, bid, nblk);
    grid_barrier(bar, arrivals += nblk, err);
    for (uint32_t b = bid; b < t.B; b += nblk) { wg_sync(); scan_body(t, c.G, c.E, err, coded, b); }
    grid_barrier(bar, arrivals += nblk, err);
}

/* ------------------------------------------------------------------ whole values from the dense accumulator */

/* 16- and 32-bit values wait for no scale, so the survivors of a tile of a bucket whose threshold, tie allowance and
 * prefixes are known need nothing from any other tile: elements read once, ranks from ballots, values and indices through LDS to
 * where they go, and the elements written back as whole lines with what the survivors leave behind: the memory behind the caches reads a
 * 64-byte line before it writes a part of it (half the words of 268 M elements written 400 us, read and then written 402, read and
 * written whole 340; one in ten: 390 and 339).  A tile
 * per workgroup of NT threads.  pool: 2 * TILE words. */
/* Survivors of 256 elements from which their lines are written whole.  Compress, us, 30 buckets of 1 M elements as 32-bit values, from 6 / 16 / 40 up:
 * 33 of 256 on average 168.7 / 168.1 / 175.0, 15 in half of the rows 177.6 / 177.7 / 179.7, 8 in half of them 178.0 / 178.4 / 180.7.  Anything from 6 to
 * 16 does. */
constexpr uint32_t BAND_ROW = 16;
template <int BITS, uint32_t NT, bool PAST>       /* PAST: whole lines go past the caches, see st_out */
__device__ __forceinline__ void band_tile(float *__restrict__ r, const Tables &t, const Cand &c, uint32_t *__restrict__ idx_out, void *__restrict__ val,
                                          uint32_t *__restrict__ err, uint32_t tile, const uint4 &d, uint32_t *pool)
{
    static_assert(BITS >= 16, "no chunks");
    constexpr uint32_t Q = TILE / (4u * NT), W = NT / 64;
    __shared__ uint32_t wt[8];
    float *sv = reinterpret_cast<float *>(pool);
    uint32_t *si = pool + TILE;
    const uint32_t tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t b = d.z, first = d.w & 0xFFFFu, last = d.w >> 16;
    float *rt = r + (((uint64_t)d.y << 32) | d.x);
    const bool whole = first == 0u && last == (uint32_t)TILE, full = whole && t.pmask == nullptr;
    float x[Q][4];
    uint32_t m[Q];
#pragma unroll
    for (uint32_t u = 0; u < Q; ++u) {
        const uint32_t e = (u * NT + tid) * 4u;
        m[u] = 0;
        if (whole) {
            const f4 v = *reinterpret_cast<const f4 *>(rt + e);
            x[u][0] = v.x; x[u][1] = v.y; x[u][2] = v.z; x[u][3] = v.w;
            m[u] = 0xFu;
        } else {
#pragma unroll
            for (uint32_t j = 0; j < 4; ++j) {
                x[u][j] = 0.0f;
                if (e + j >= first && e + j < last) { x[u][j] = rt[e + j]; m[u] |= 1u << j; }
            }
        }
        if (t.pmask) m[u] &= ~pruned_bits(t.pmask, tile, u * NT + tid);
    }
    const uint32_t T = t.T[b], e_b = t.need[b], kb = t.k[b], Gs = c.G[tile], Es = c.E[tile];
    const uint64_t Pb = t.P[b];
    uint8_t *vb = reinterpret_cast<uint8_t *>(val) + t.V[b];
    const uint32_t li0 = (tile - t.tile0[b]) * (uint32_t)TILE - (uint32_t)(t.off[b] & 3ull);      /* (mod 2^32) */
    const uint32_t lim = e_b > Es ? e_b - Es : 0u, R0 = Gs + min(e_b, Es);                         /* ties still admitted, rank of the tile's first survivor */
    uint32_t row_g[Q], row_e[Q], bef[Q];
    /* keys as signed numbers, what does not count the lowest of them */
    auto keys = [&](uint32_t u, int32_t (&key)[4]) {
#pragma unroll
        for (int j = 0; j < 4; ++j) key[j] = (int32_t)keyof(x[u][j]);
        if (!full) {
#pragma unroll
            for (int j = 0; j < 4; ++j) key[j] = (m[u] >> j) & 1u ? key[j] : (int32_t)0x80000000u;
        }
    };
#pragma unroll
    for (uint32_t u = 0; u < Q; ++u) {
        row_g[u] = row_e[u] = bef[u] = 0;
        int32_t key[4];
        keys(u, key);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint64_t bg = __ballot(key[j] > (int32_t)T);
            row_g[u] += (uint32_t)__popcll(bg);
            row_e[u] += (uint32_t)__popcll(__ballot(key[j] == (int32_t)T));
            bef[u] = __builtin_amdgcn_mbcnt_hi((uint32_t)(bg >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bg, bef[u]));
        }
        if (lane == 0) wt[u * W + wave] = row_g[u] | (row_e[u] << 16);
    }
    wg_sync();
    uint32_t all = 0, before[Q];
    {
        const uint32_t mine = wt[lane & 7u];
#pragma unroll
        for (uint32_t w = 0; w < 8u; ++w) {
#pragma unroll
            for (uint32_t u = 0; u < Q; ++u) if (u * W + wave == w) before[u] = all;
            all += (uint32_t)__builtin_amdgcn_readlane((int)mine, (int)w);
        }
    }
    const uint32_t nsurv = (all & 0xFFFFu) + min(all >> 16, lim);
    if (R0 > kb || nsurv > kb - R0) {                /* the prefixes and the elements disagree: nothing is written (same for the whole workgroup) */
        if (tid == 0) err[0] = 1u;
        return;
    }
    auto left_of = [&](float v) { return BITS == 32 ? __fsub_rn(v, v) : __fsub_rn(v, __half2float(__float2half_rn(v))); };      /* (32 bits: NaN where no value was) */
#pragma unroll
    for (uint32_t u = 0; u < Q; ++u) {
        if (row_g[u] + row_e[u] == 0u) continue;     /* same for the whole wavefront */
        const uint32_t fg = before[u] & 0xFFFFu, fe = before[u] >> 16, e = (u * NT + tid) * 4u;
        int32_t key[4];
        keys(u, key);
        uint32_t bits = 0, s;
        if (row_e[u] == 0u || fe >= lim) {
#pragma unroll
            for (int j = 0; j < 4; ++j) bits |= (key[j] > (int32_t)T ? 1u : 0u) << j;
            s = fg + min(fe, lim) + bef[u];
        } else {
            uint32_t pe = fe;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint64_t be = __ballot(key[j] == (int32_t)T);
                pe = __builtin_amdgcn_mbcnt_hi((uint32_t)(be >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)be, pe));
            }
            s = fg + bef[u] + min(pe, lim);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const bool tie = key[j] == (int32_t)T;
                bits |= (key[j] > (int32_t)T || (tie && pe < lim) ? 1u : 0u) << j;
                pe += tie ? 1u : 0u;
            }
        }
        float y[4];
#pragma unroll
        for (uint32_t j = 0; j < 4; ++j) {
            y[j] = x[u][j];
            if (!((bits >> j) & 1u)) continue;
            sv[s] = x[u][j];
            si[s] = li0 + e + j;
            y[j] = left_of(x[u][j]);
            ++s;
        }
        /* (zeros that survive leave what they were: an embedding's untouched rows are not written back) */
        uint32_t diff = 0;
#pragma unroll
        for (uint32_t j = 0; j < 4; ++j) diff |= __float_as_uint(y[j]) ^ __float_as_uint(x[u][j]);
        if (!__any(diff)) continue;
        if (whole && row_g[u] + row_e[u] >= BAND_ROW) {
            st_out<PAST>(reinterpret_cast<f4 *>(rt + e), f4{y[0], y[1], y[2], y[3]});
        } else {
#pragma unroll
            for (uint32_t j = 0; j < 4; ++j)
                if ((bits >> j) & 1u) rt[e + j] = y[j];
        }
    }
    wg_sync();
    for (uint32_t i = tid; i < nsurv; i += NT) {
        const float v = sv[i];
        idx_out[Pb + R0 + i] = si[i];
        if (BITS == 32) reinterpret_cast<float *>(vb)[R0 + i] = v;
        else reinterpret_cast<__half *>(vb)[R0 + i] = __float2half_rn(v);
    }
}
/* Tiles of buckets on the paths `which` (bit p: PATH p), by nblk workgroups of NT threads. */
template <int BITS, uint32_t NT>
__device__ __forceinline__ void band_tiles(float *__restrict__ r, const Tables &t, const Cand &c, uint32_t *__restrict__ idx, void *__restrict__ val,
                                           uint32_t *__restrict__ err, uint32_t which, uint32_t *pool, uint32_t bid, uint32_t nblk)
{
    const uint32_t lane = threadIdx.x & 63;
    for (uint64_t t0 = bid; t0 < t.n_tiles; t0 += 64ull * nblk) {
        const uint64_t tl = t0 + (uint64_t)lane * nblk;
        const uint32_t path = t.fast[t.tile_b[min(tl, (uint64_t)t.n_tiles - 1u)]];
        for (uint64_t todo = __ballot(tl < t.n_tiles && ((which >> path) & 1u)); todo; todo &= todo - 1ull) {
            const uint32_t tile = (uint32_t)(t0 + (uint64_t)__builtin_ctzll(todo) * nblk);
            wg_sync();                               /* LDS is written again */
            band_tile<BITS, NT, false>(r, t, c, idx, val, err, tile, t.desc[tile], pool);
        }
    }
}
/* The buckets on the dense passes where values are whole, by the nblk workgroups of a resident team (WG threads of each): threshold,
 * counts and prefixes, then their survivors tile by tile. */
template <int BITS>
__device__ __forceinline__ void band_dense_buckets(float *__restrict__ r, const Tables &t, const Cand &c, uint32_t *__restrict__ f0,
                                                   uint32_t *__restrict__ f1, uint32_t *__restrict__ f2, uint32_t *__restrict__ idx,
                                                   void *__restrict__ val, uint32_t *__restrict__ err, uint32_t *pool, uint32_t bid, uint32_t nblk)
{
    static_assert(2 * TILE >= NB1, "the pool must hold the level-1 histogram");
    dense_threshold(r, t, c, f0, f1, f2, pool, t.nhard + 1, bid, nblk, true, err);
    band_tiles<BITS, WG>(r, t, c, idx, val, err, 1u << PATH_DENSE, pool, bid, nblk);
}

/* ------------------------------------------------------------------ k_encode */

/* One workgroup per chunk of `chunk` consecutive survivors of a PATH_CAND bucket: gather,
 * absmax, scale, codes, packing, indices, and the coding error left in the residual.  Every
 * floating-point step is a single correctly rounded binary32 operation.  A chunk longer than
 * ENC_BLK is gathered block by block, once for its absmax and once more for the codes.
 * Where values are whole (16 and 32 bits) its first `team` workgroups, dispatched before the others and so resident when they
 * meet, do the dense passes, so that the rest of such a call is k_band alone.  (Everything that is not staged coded here, a workgroup per 2048
 * survivors of the dense accumulator, saves two launches that nearly always have nothing to do, 3 us of 46 with one bucket of 1 Mi elements; but
 * survivors far apart are then a long chain in one workgroup: such a bucket at 0.01 with values clipped at one sigma 160 - 500 us instead
 * of 70.) */
template <int BITS, uint32_t ENC_T>
__global__ __launch_bounds__(ENC_T, 4) void k_encode(Tables t, Cand c, const uint32_t *__restrict__ chunk_b,
                                               const uint32_t *__restrict__ chunk_seg, float *__restrict__ r,
                                               uint32_t *__restrict__ idx_out, void *__restrict__ val,
                                               float *__restrict__ scales, uint32_t *__restrict__ err,
                                               uint64_t n_chunks, uint32_t *__restrict__ hist,
                                               const double *__restrict__ tile_sq, double *__restrict__ l2sq,
                                               uint32_t *__restrict__ f0, uint32_t *__restrict__ f1, uint32_t *__restrict__ f2,
                                               uint32_t first, uint32_t team)
{
    __shared__ __align__(16) uint32_t pool[2 * ENC_BLK];
    float *sv = reinterpret_cast<float *>(pool);
    uint32_t *si = pool + ENC_BLK;
    __shared__ float red[ENC_T / 64];
    __shared__ uint32_t sh, filled, meta[3 * ENC_T];       /* of segments: entries, and what lies above and at T before */
    static_assert(ENC_BLK == (uint32_t)TILE, "the pool holds a tile's survivors");
    if (blockIdx.x < first) {
        if (blockIdx.x < t.B) {
            /* The first workgroups keep the buckets' records: the norm, and what the plan was made from left clean for the next
             * call.  (In k_select_finish, whose time all of it would add to, 4 us.) */
            const uint32_t b = blockIdx.x;
            bucket_sq<ENC_T>(t, b, tile_sq, reinterpret_cast<double *>(pool), l2sq + b);
            for (uint32_t i = threadIdx.x * 4u; i < NHC * HROW; i += ENC_T * 4u) *reinterpret_cast<uint4 *>(hist + (uint64_t)b * NHC * HROW + i) = make_uint4(0u, 0u, 0u, 0u);
            if (threadIdx.x == 0) {
                if (t.k[b] == 0u) plan_empty(t, b);
                t.ovf[b] = 0u;
            }
        }
        if constexpr (BITS >= 16) {
            if (blockIdx.x >= team || t.nhard[2] == 0u || threadIdx.x >= WG) return;
            wg_sync();
            band_dense_buckets<BITS>(r, t, c, f0, f1, f2, idx_out, val, err, pool, blockIdx.x, team);
        }
        return;
    }
    const uint32_t bid = blockIdx.x - first;
    constexpr float QMAX = BITS == 8 ? 127.0f : 7.0f;
    constexpr uint32_t ENC_WAVES = ENC_T / 64;
    const uint32_t tid = threadIdx.x;
    /* A workgroup takes the chunks bid, bid + grid, ..: its only one, or up to 64 at a time, of which the lanes
     * first find those that are coded here (of a workgroup each, 2742 chunks of other paths took 15 us to skip, so 5) */
    const uint32_t grid = gridDim.x - first, lane = tid & 63;
    const bool single = grid == n_chunks;
    for (uint64_t c0 = bid; c0 < n_chunks; c0 += 64ull * grid) {
    uint64_t todo = 1ull;
    if (!single) {
        const uint64_t cl = c0 + (uint64_t)lane * grid;
        todo = __ballot(cl < n_chunks && t.fast[chunk_b[min(cl, n_chunks - 1u)]] == PATH_CAND);
    }
    for (; todo; todo &= todo - 1ull) {
    const uint64_t cid = c0 + (uint64_t)__builtin_ctzll(todo) * grid;
    const uint32_t b = chunk_b[cid];
    const uint32_t sFirst = chunk_seg[cid];          /* meaningful for PATH_CAND buckets only, like the next one */
    const uint32_t sNext = cid + 1 < n_chunks ? chunk_seg[cid + 1] : 0u;
    if (single && t.fast[b] != PATH_CAND) return;
    const uint64_t cb = cid - t.C[b];
    const uint64_t j0c = cb * t.chunk;                         /* first survivor of the chunk, bucket-local */
    const uint32_t cnt_c = (uint32_t)min((uint64_t)t.chunk, (uint64_t)t.k[b] - j0c);
    const uint32_t T = t.T[b], e_b = t.need[b];
    const uint32_t seg_lo = t.tile0[b], seg_hi = t.tile0[b + 1];
    const uint32_t sEnd = j0c + cnt_c < (uint64_t)t.k[b] ? sNext + 1u : seg_hi;      /* where the next chunk begins, or the bucket's end */
    const uint64_t lo = t.off[b], Pb = t.P[b];
    uint8_t *vb = reinterpret_cast<uint8_t *>(val) + t.V[b];

    /* a thread holds PER survivors of the block, ENC_T apart: the lanes of a wavefront hold consecutive ones */
    constexpr uint32_t PER = ENC_BLK / ENC_T;
    static_assert(PER % 4u == 0u, "coded four at a time");
    float xv[PER];
    auto fetch_values = [&](uint32_t n) {
#pragma unroll
        for (uint32_t h = 0; h < PER; ++h) { const uint32_t i = h * ENC_T + tid; xv[h] = i < n ? sv[i] : 0.0f; }
    };
    auto block_absmax = [&]() {
        float m = 0.0f;
#pragma unroll
        for (uint32_t h = 0; h < PER; ++h) m = fmaxf(m, fabsf(xv[h]));
        m = wave_max(m);
        wg_sync();
        if (lane == 0) red[tid >> 6] = m;
        wg_sync();
#pragma unroll
        for (uint32_t w = 0; w < ENC_WAVES; ++w) m = fmaxf(m, red[w]);
        return m;
    };
    auto gather = [&](uint32_t blk0, uint32_t n) {
        wg_sync();                                       /* the previous block has been consumed */
        if (tid == 0) filled = 0u;
        const uint32_t j0 = (uint32_t)j0c + blk0;
        uint32_t sA = sFirst;
        if (blk0 != 0) {
            /* a later block of a long chunk: the last segment whose first survivor is not beyond j0 */
            auto rank0 = [&](uint32_t s) { return (uint64_t)c.G[s] + (uint64_t)min(e_b, c.E[s]); };
            sA = wg_search_le<ENC_T>(seg_lo, seg_hi, (uint64_t)j0, rank0, &sh);
        }
        wg_sync();
        gather_survivors<ENC_T>(c, sA, sEnd, T, e_b, j0, n, meta, sv, si, &filled);
        wg_sync();
        if (filled == n) return true;
        if (tid == 0) err[0] = 1u;                       /* the prefixes and the entries disagree: nothing is written */
        return false;
    };

    float m = 0.0f;
    const bool long_chunk = cnt_c > ENC_BLK;
    if (BITS <= 8 && long_chunk)
        for (uint32_t blk0 = 0; blk0 < cnt_c; blk0 += ENC_BLK) {
            const uint32_t n = min(ENC_BLK, cnt_c - blk0);
            if (!gather(blk0, n)) return;                /* (same for the whole workgroup) */
            fetch_values(n);
            m = fmaxf(m, block_absmax());
        }
    for (uint32_t blk0 = 0; blk0 < cnt_c; blk0 += ENC_BLK) {
        const uint32_t n = min(ENC_BLK, cnt_c - blk0);
        if (!gather(blk0, n)) return;
        fetch_values(n);
        float scale = 0.0f;
        if (BITS <= 8) {
            if (!long_chunk) m = block_absmax();
            scale = m == 0.0f ? 0.0f : __fdiv_rn(m, QMAX);
            if (tid == 0 && blk0 == 0) scales[t.S[b] + cb] = scale;
        }
        const uint64_t jb = j0c + blk0;                        /* bucket-local number of the block's first survivor */
#pragma unroll
        for (uint32_t h0 = 0; h0 < PER; h0 += 4) {
            float x4[4];
            int q[4] = {0, 0, 0, 0};
#pragma unroll
            for (int h = 0; h < 4; ++h) x4[h] = xv[h0 + h];
            if (BITS <= 8) quantize_four<BITS>(x4, scale, q);
#pragma unroll
            for (int h = 0; h < 4; ++h) {
                const uint32_t i = (h0 + h) * ENC_T + tid;
                /* a pair's codes in one byte at 4 bits: the odd lane's comes over (0 beyond the last) */
                const int odd = BITS == 4 ? __builtin_amdgcn_mov_dpp(q[h], 0xF5, 0xF, 0xF, false) : 0;      /* lanes 1 1 3 3 */
                if (i >= n) continue;
                float deq;
                if (BITS == 32) {
                    reinterpret_cast<float *>(vb)[jb + i] = x4[h];
                    deq = x4[h];
                } else if (BITS == 16) {
                    const __half hv = __float2half_rn(x4[h]);
                    reinterpret_cast<__half *>(vb)[jb + i] = hv;
                    deq = __half2float(hv);
                } else {
                    deq = __fmul_rn((float)q[h], scale);
                    if (BITS == 8) reinterpret_cast<int8_t *>(vb)[jb + i] = (int8_t)q[h];
                    else if (!(lane & 1u)) vb[(jb + i) >> 1] = (uint8_t)((q[h] & 0xF) | ((odd & 0xF) << 4));
                }
                const uint32_t li = si[i];
                idx_out[Pb + jb + i] = li;
                r[lo + li] = __fsub_rn(x4[h], deq);
            }
        }
    }
    }
    }
}

/* ------------------------------------------------------------------ k_hard */

/* Ordered write and value coding in one pass, for the buckets whose survivors are taken from the
 * dense accumulator and whose threshold is known (PATH_BAND, PATH_ZERO), with chunks of at most
 * DENC_MAX_CHUNK survivors.  Survivors are dense here (ratios from an eighth up, or an
 * embedding whose few non-zero rows all survive), so the work is laid out by elements: a
 * workgroup streams a unit of dencTiles consecutive tiles, 4096 elements at a time (512
 * consecutive ones per wavefront); ranks come from ballots and a prefix over the eight wavefronts; the
 * survivors are put into LDS in rank order behind the ones still waiting for their chunk to
 * fill up; every chunk that is complete is coded from LDS by one wavefront (absmax, scale,
 * codes, indices, and the coding error scattered into the accumulator lines the workgroup has
 * just read, which are still in the cache).  A chunk that reaches across the unit's ends (or a
 * bucket's tiles of another unit) is written uncoded to idx / v_out, and k_quant codes exactly
 * those afterwards (same test, see chunk_coded_by_stream).  (16- and 32-bit values: band_tile.) */
/* What bounds it: the steps, not memory.  Half of 419 M elements sent as 8-bit codes take 860 - 960 us, from one machine to another, for 4.35 GB.
 * Without the scattered residual it is 708 of 948, without any store 690.  The wavefronts spend 21 % of their time issuing (37 instructions per
 * element; 59 before the counts came from comparison masks and the codes from a product), 30 % ready and waiting to issue, and 50 % waiting
 * for memory, LDS or each other, of which barriers are 26 (SQ_ACTIVE_INST_ANY, SQ_WAIT_INST_ANY, SQ_WAIT_ANY; barriers by the clock in a
 * copy).  Was 1010 with four wavefronts and two survivors per lane; four consecutive survivors per lane (16-byte index stores at 4-byte
 * alignment, residual stores 8 elements apart) 975, full residual lines 1057, non-temporal index stores 1169; the elements
 * written back when they are read, so that the errors meet whole lines in the cache, 997 (they have left it by then). */
constexpr uint32_t DENC_SMALL_CHUNK = 256;         /* up to here a wavefront codes a chunk */
constexpr uint32_t DENC_MAX_CHUNK = 2048;
constexpr uint32_t DENC_STEP = 4096;               /* elements per step: all of them can be survivors */
constexpr uint32_t HTH = 512;                      /* threads of a workgroup of k_hard */
constexpr uint32_t DENC_ROWS = DENC_STEP / HTH / 4; /* 16-byte accesses per thread and step */
constexpr uint32_t DENC_WT = DENC_STEP / (HTH / 64); /* consecutive elements of one wavefront per step */
constexpr uint32_t denc_cap(bool big) { return DENC_STEP + (big ? DENC_MAX_CHUNK : DENC_SMALL_CHUNK); }

template <int BITS, bool BIG>       /* BIG: chunks of more than DENC_SMALL_CHUNK survivors */
__device__ __forceinline__ void dense_encode_body(float *__restrict__ r, const Tables &t, const Cand &c,
                                                  uint32_t *__restrict__ idx_out, float *__restrict__ v_out,
                                                  void *__restrict__ val, float *__restrict__ scales,
                                                  float *sv, uint32_t *si, uint32_t *wtot, uint32_t *__restrict__ err,
                                                  uint32_t bid, uint32_t nblk)
{
    constexpr float QMAX = BITS == 8 ? 127.0f : 7.0f;
    const uint32_t tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t chunk = t.chunk;
    const uint32_t n_units = (t.n_tiles + t.dencTiles - 1) / t.dencTiles;
    for (uint32_t unit = bid; unit < n_units; unit += nblk) {
        uint32_t cur_b = NONE;
        /* state of the stream: one bucket's consecutive tiles inside the unit */
        uint32_t T = 0, e_b = 0, kb = 0, run_g = 0, run_e = 0, carry = 0, Rbase = 0;
        uint64_t Pb = 0;
        uint8_t *vb = nullptr;
        uint64_t Sb = 0;
        bool head = false;
        uint32_t li_stream = 0;
        /* what is left in LDS when a stream ends belongs to a chunk that goes on elsewhere */
        auto flush = [&]() {
            for (uint32_t i = tid; i < carry; i += HTH) {
                idx_out[Pb + Rbase + i] = si[i] + li_stream;
                v_out[Pb + Rbase + i] = sv[i];
            }
            carry = 0;
            wg_sync();
        };
        const uint32_t sp1 = min(t.n_tiles, (unit + 1) * t.dencTiles);
        uint32_t send = 0;
        for (uint32_t tile = unit * t.dencTiles; tile < sp1; tile = send) {
            /* the bucket's tiles of this unit: [tile, send) */
            const uint32_t b = t.tile_b[tile];
            send = min(sp1, t.tile0[b + 1]);
            const uint32_t path = t.fast[b];
            if (cur_b != NONE) flush();
            if ((path != PATH_BAND && path != PATH_ZERO) || t.k[b] == 0u) { cur_b = NONE; continue; }
            const TileGeo s = tile_geo(t, b, tile);
            cur_b = b;
            T = t.T[b]; e_b = t.need[b]; kb = t.k[b]; Pb = t.P[b];
            vb = reinterpret_cast<uint8_t *>(val) + t.V[b];
            Sb = t.S[b];
            run_g = c.G[tile]; run_e = c.E[tile];
            Rbase = run_g + min(e_b, run_e);
            carry = 0;
            head = (Rbase % chunk) != 0u;
            const uint32_t nwt = (send - tile) * (TILE / DENC_WT);
            /* the next 4096 elements are fetched while the survivors of these are coded */
            float xn[DENC_ROWS][4];
            uint32_t mn[DENC_ROWS];
            auto fetch = [&](uint32_t wt_base) {
                const uint32_t wt = wt_base + wave;
                const uint64_t wb = s.base + (uint64_t)wt * DENC_WT;
#pragma unroll
                for (int u = 0; u < (int)DENC_ROWS; ++u) {
                    const uint64_t gi = wb + (uint64_t)(u * 64 + lane) * 4;
                    mn[u] = 0;
#pragma unroll
                    for (int j = 0; j < 4; ++j) xn[u][j] = 0.0f;
                    if (wt < nwt) {
                        if (wb >= s.lo && wb + DENC_WT <= s.hi) {          /* the whole wave-tile lies inside the bucket */
                            const f4 v = *reinterpret_cast<const f4 *>(r + gi);
                            xn[u][0] = v.x; xn[u][1] = v.y; xn[u][2] = v.z; xn[u][3] = v.w;
                            mn[u] = 0xFu;
                        } else {
                            mn[u] = load_quad(r, gi, s.lo, s.hi, xn[u]);
                        }
                        if (t.pmask) mn[u] &= ~pruned_bits(t.pmask, tile, wt * (DENC_WT / 4) + u * 64 + lane);
                    }
                }
            };
            fetch(0);
            const uint32_t li_base = li_stream = (uint32_t)(s.base - s.lo);       /* bucket-local index = position from s.base + this (mod 2^32) */
            float *rb = r + s.base;
            for (uint32_t wt_base = 0; wt_base < nwt; wt_base += HTH / 64) {
                const uint32_t wt = wt_base + wave;
                const uint64_t wb = s.base + (uint64_t)wt * DENC_WT;
                if (tid == 0 && (run_g != c.G[tile + wt_base / (TILE / DENC_WT)] || run_e != c.E[tile + wt_base / (TILE / DENC_WT)]))
                    err[0] = 1u;                     /* the prefixes and the elements disagree */
                float x[DENC_ROWS][4];
                bool fg[DENC_ROWS][4];
                const bool full = wt < nwt && wb >= s.lo && wb + DENC_WT <= s.hi && !t.pmask;      /* every element counts */
                uint64_t ties = 0;
                /* Ranks: a lane's elements of a row are consecutive, so the elements before one are those of
                 * the lower lanes of its row, of the earlier rows and of the earlier wavefronts.  A
                 * comparison's result is the mask over the wavefront that counting needs. */
                uint32_t row_g[DENC_ROWS], row_e[DENC_ROWS];       /* elements above / equal to T in a row (same in all lanes) */
                uint32_t bef_g[DENC_ROWS];                         /* those above T in the lower lanes of the row */
#pragma unroll
                for (int u = 0; u < (int)DENC_ROWS; ++u) {
                    row_g[u] = row_e[u] = bef_g[u] = 0;
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        x[u][j] = xn[u][j];
                        const uint32_t key = keyof(x[u][j]);
                        const bool in = full || ((mn[u] >> j) & 1u);
                        fg[u][j] = in && key > T;
                        const uint64_t bg = __ballot(fg[u][j]), be = __ballot(in && key == T);
                        row_g[u] += (uint32_t)__popcll(bg);
                        row_e[u] += (uint32_t)__popcll(be);
                        bef_g[u] = __builtin_amdgcn_mbcnt_hi((uint32_t)(bg >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bg, bef_g[u]));
                        ties |= be;
                    }
                }
                uint32_t wsum = 0;
#pragma unroll
                for (int u = 0; u < (int)DENC_ROWS; ++u) wsum += row_g[u] | (row_e[u] << 16);      /* 4096 elements cannot carry */
                if (lane == 0) wtot[wave] = wsum;
                wg_sync();
                uint32_t woff = 0, all = 0;
                {
                    const uint32_t mine = wtot[lane & (HTH / 64 - 1)];
#pragma unroll
                    for (uint32_t w = 0; w < HTH / 64; ++w) {
                        const uint32_t v = (uint32_t)__builtin_amdgcn_readlane((int)mine, w);
                        if (w < wave) woff += v;
                        all += v;
                    }
                }
                const uint32_t all_g = all & 0xFFFFu, all_e = all >> 16;
                const uint32_t Rnext = run_g + min(e_b, run_e);               /* rank of the next survivor = Rbase + carry */
                const uint32_t nsurv = (run_g + all_g + min(e_b, run_e + all_e)) - Rnext;
                /* survivors into LDS in rank order, behind those that wait */
                auto put = [&](int u, int j, uint32_t slot) {
                    sv[slot] = x[u][j];
                    si[slot] = wt * DENC_WT + (uint32_t)(u * 64 + lane) * 4 + (uint32_t)j;
                };
                uint32_t g0 = run_g + (woff & 0xFFFFu), e0 = run_e + (woff >> 16);
#pragma unroll
                for (int u = 0; u < (int)DENC_ROWS; ++u) {
                    if (ties == 0) {                 /* none in this wavefront, the ordinary case */
                        uint32_t slot = carry + g0 + bef_g[u] + min(e_b, e0) - Rnext;
#pragma unroll
                        for (int j = 0; j < 4; ++j) {
                            if (fg[u][j]) put(u, j, slot);
                            slot += fg[u][j] ? 1u : 0u;
                        }
                    } else {
                        uint32_t pe = e0;
                        bool fe[4];
#pragma unroll
                        for (int j = 0; j < 4; ++j) {
                            fe[j] = (full || ((mn[u] >> j) & 1u)) && keyof(x[u][j]) == T;
                            const uint64_t be = __ballot(fe[j]);
                            pe = __builtin_amdgcn_mbcnt_hi((uint32_t)(be >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)be, pe));
                        }
                        uint32_t slot = carry + g0 + bef_g[u] + min(e_b, pe) - Rnext;
#pragma unroll
                        for (int j = 0; j < 4; ++j) {
                            const bool take = fg[u][j] || (fe[j] && pe < e_b);
                            if (take) put(u, j, slot);
                            slot += take ? 1u : 0u;
                            pe += fe[j] ? 1u : 0u;
                        }
                    }
                    g0 += row_g[u];
                    e0 += row_e[u];
                }
                run_g += all_g;
                run_e += all_e;
                wg_sync();
                if (wt_base + HTH / 64 < nwt) fetch(wt_base + HTH / 64);
                /* consume what is complete */
                const uint32_t total = carry + nsurv;
                uint32_t p = 0;
                {
                    if (head) {
                        /* up to the next chunk boundary: part of a chunk that began before this stream */
                        const uint32_t to_edge = chunk - (Rbase % chunk);
                        const uint32_t nh = min(total, to_edge);
                        for (uint32_t i = tid; i < nh; i += HTH) {
                            idx_out[Pb + Rbase + i] = si[i] + li_base;
                            v_out[Pb + Rbase + i] = sv[i];
                        }
                        p = nh;
                        if (nh == to_edge) head = false;
                    }
                    if (!head) {
                        const uint32_t avail = total - p;
                        const uint32_t nfull = avail / chunk, rem = avail - nfull * chunk;
                        const uint32_t ncode = nfull + ((rem != 0u && Rbase + total == kb) ? 1u : 0u);   /* the bucket's last chunk may be short */
                        /* four survivors of a chunk, `step` apart, so that the lanes of a wavefront hold consecutive
                         * ones: values and positions; then codes, indices and coding errors */
                        float xv[4];
                        uint32_t at[4];
                        auto take_four = [&](uint32_t base, uint32_t i0, uint32_t step, uint32_t cnt) {
#pragma unroll
                            for (int h = 0; h < 4; ++h) {
                                const uint32_t i = i0 + h * step;
                                xv[h] = i < cnt ? sv[base + i] : 0.0f;
                                at[h] = i < cnt ? si[base + i] : 0u;
                            }
                            return fmaxf(fmaxf(fabsf(xv[0]), fabsf(xv[1])), fmaxf(fabsf(xv[2]), fabsf(xv[3])));
                        };
                        auto code_four = [&](uint32_t rank0, uint32_t i0, uint32_t step, uint32_t cnt, float scale) {
                            int qq[4];
                            quantize_four<BITS>(xv, scale, qq);
#pragma unroll
                            for (int h = 0; h < 4; ++h) {
                                const uint32_t i = i0 + h * step;
                                /* a pair's codes in one byte at 4 bits: the odd lane's comes over */
                                const int odd = BITS == 4 ? __builtin_amdgcn_mov_dpp(qq[h], 0xF5, 0xF, 0xF, false) : 0;      /* lanes 1 1 3 3 */
                                if (i < cnt) {
                                    idx_out[Pb + rank0 + i] = at[h] + li_base;
                                    if (BITS == 8) vb[rank0 + i] = (uint8_t)qq[h];
                                    else if (!(lane & 1u)) vb[(rank0 + i) >> 1] = (uint8_t)((qq[h] & 0xF) | ((odd & 0xF) << 4));
                                    *reinterpret_cast<float *>(reinterpret_cast<char *>(rb) + at[h] * 4u) = __fsub_rn(xv[h], __fmul_rn((float)qq[h], scale));
                                }
                            }
                        };
                        if (!BIG) {
                            /* chunks of up to 256: a wavefront each */
                            for (uint32_t q = wave; q < ncode; q += HTH / 64) {
                                const uint32_t base = p + q * chunk;
                                const uint32_t cnt = min(chunk, total - base);
                                const uint32_t rank0 = Rbase + base;
                                const float mx = wave_max(take_four(base, lane, 64, cnt));
                                const float scale = mx == 0.0f ? 0.0f : __fdiv_rn(mx, QMAX);
                                if (lane == 0) scales[Sb + rank0 / chunk] = scale;
                                code_four(rank0, lane, 64, cnt, scale);
                            }
                        } else {
                            /* longer chunks: the whole workgroup on one chunk after the other */
                            for (uint32_t q = 0; q < ncode; ++q) {
                                const uint32_t base = p + q * chunk;
                                const uint32_t cnt = min(chunk, total - base);
                                const uint32_t rank0 = Rbase + base;
                                const float wm = wave_max(take_four(base, tid, HTH, cnt));
                                float *red = reinterpret_cast<float *>(wtot);
                                if (lane == 0) red[wave] = wm;
                                wg_sync();
                                float mx = 0.0f;
#pragma unroll
                                for (uint32_t w = 0; w < HTH / 64; ++w) mx = fmaxf(mx, red[w]);
                                const float scale = mx == 0.0f ? 0.0f : __fdiv_rn(mx, QMAX);
                                if (tid == 0) scales[Sb + rank0 / chunk] = scale;
                                code_four(rank0, tid, HTH, cnt, scale);
                                wg_sync();
                            }
                        }
                        p += min(avail, ncode * chunk);
                    }
                }
                wg_sync();
                /* the rest waits at the front for the next elements */
                const uint32_t left = total - p;
                constexpr uint32_t KEEP = BIG ? DENC_MAX_CHUNK / HTH : 1u;
                float keep_v[KEEP];
                uint32_t keep_i[KEEP];
#pragma unroll
                for (uint32_t u = 0; u < KEEP; ++u) {
                    const uint32_t i = tid + u * HTH;
                    keep_v[u] = 0.0f; keep_i[u] = 0u;
                    if (i < left) { keep_v[u] = sv[p + i]; keep_i[u] = si[p + i]; }
                }
                wg_sync();
#pragma unroll
                for (uint32_t u = 0; u < KEEP; ++u) {
                    const uint32_t i = tid + u * HTH;
                    if (i < left) { sv[i] = keep_v[u]; si[i] = keep_i[u]; }
                }
                Rbase += p;
                carry = left;
            }
        }
        if (cur_b != NONE) flush();
        wg_sync();
    }
}

/* Whether chunk cb (bucket-local) of a PATH_BAND / PATH_ZERO bucket b was coded by
 * dense_encode_body: its first survivor lies in tile s, and all of its survivors lie in the
 * tiles of b inside the unit of dencTiles tiles that holds s. */
__device__ __forceinline__ bool chunk_coded_by_stream(const Tables &t, const Cand &c, uint32_t b, uint64_t cb, uint32_t s)
{
    const uint32_t kb = t.k[b], e_b = t.need[b];
    const uint64_t end = min((cb + 1) * (uint64_t)t.chunk, (uint64_t)kb);
    const uint32_t next = (s / t.dencTiles + 1u) * t.dencTiles;
    uint64_t r1 = kb;
    if (next < t.tile0[b + 1]) r1 = (uint64_t)c.G[next] + min(e_b, c.E[next]);
    return end <= r1;
}

/* workgroups of k_hard per compute unit: what its LDS allows (all of them must be resident) */
constexpr uint32_t hard_wg_per_cu(bool) { return 3u; }
constexpr uint32_t hard_lds(bool big) { return 2 * denc_cap(big) + HTH / 64; }    /* words; also holds the level-1 histogram */

template <int BITS, bool BIG>
__global__ __launch_bounds__(HTH, hard_wg_per_cu(BIG) * (HTH / 256)) void k_hard(float *__restrict__ r, Tables t, Cand c, uint32_t *__restrict__ f0,
                                             uint32_t *__restrict__ f1, uint32_t *__restrict__ f2, uint32_t *__restrict__ idx,
                                             float *__restrict__ vdst, void *__restrict__ val,
                                             float *__restrict__ scales, uint32_t *__restrict__ err, int stream_coding, uint32_t team)
{
    static_assert(hard_lds(BIG) >= NB1, "the pool must hold the level-1 histogram");
    __shared__ __align__(16) uint32_t pool[hard_lds(BIG)];
    if (t.nhard[0] == 0u) return;                    /* every bucket was decided and coded from its staged elements */
    const uint32_t bid = blockIdx.x;
    uint32_t nblk = gridDim.x;
    /* band and zero-threshold buckets: survivors from the dense accumulator, threshold known */
    if constexpr (BITS <= 8)
        if (stream_coding)
            dense_encode_body<BITS, BIG>(r, t, c, idx, vdst, val, scales, reinterpret_cast<float *>(pool),
                                         pool + denc_cap(BIG), pool + 2 * denc_cap(BIG), err, bid, nblk);
    if (threadIdx.x >= WG) return;                   /* what follows is work for four wavefronts */
    if constexpr (BITS <= 8)
        if (!stream_coding) write_dense_body(r, t, c, idx, vdst, (1u << PATH_BAND) | (1u << PATH_ZERO), bid, nblk);
    /* the dense passes: the first `team` workgroups only.  They are dispatched before the others
     * of this launch, and the team is small enough (one workgroup per compute unit) to be
     * resident at once even next to the teams of other contexts; a barrier that still cannot
     * complete runs into its time limit and raises the consistency flag. */
    if (t.nhard[2] == 0u || bid >= team) return;
    wg_sync();
    nblk = team;
    if constexpr (BITS >= 16) {
        band_dense_buckets<BITS>(r, t, c, f0, f1, f2, idx, val, err, pool, bid, nblk);
    } else {
        dense_threshold(r, t, c, f0, f1, f2, pool, t.nhard + 1, bid, nblk, true, err);
        write_dense_body(r, t, c, idx, vdst, 1u << PATH_DENSE, bid, nblk);
    }
}

/* The buckets of a call with 16- or 32-bit values whose survivors come from the dense accumulator, in the order of
 * the streaming passes.  Bound by memory: 25.6 M elements, 0.13 to 0.71 of them as 32-bit values, 50 us on average (5.7 TB/s); by
 * the stream that codes narrower values, with its steps of 4096 elements and scattered errors, 66. */
constexpr uint32_t BAND_T = STH;
template <int BITS, bool PAST>
__global__ __launch_bounds__(BAND_T, 8) void k_band(float *__restrict__ r, Tables t, Cand c, uint32_t *__restrict__ idx, void *__restrict__ val, uint32_t *__restrict__ err)
{
    __shared__ __align__(16) uint32_t pool[2 * TILE];
    const uint32_t tile = grid_tile();
    if (tile >= t.n_tiles) return;
    const uint4 d = t.desc[tile];
    const uint32_t path = t.fast[d.z];
    if (path != PATH_BAND && path != PATH_ZERO) return;
    band_tile<BITS, BAND_T, PAST>(r, t, c, idx, val, err, tile, d, pool);
}
/* The same where no more than an eighth is sent, which nearly always leaves nothing to do: a grid of a few workgroups per compute unit, which look
 * for their tiles 64 at a time (a workgroup for each of 820 thousand tiles that leaves at once is a launch of 100 us and more). */
constexpr uint32_t BAND_WG_PER_CU = 4;
template <int BITS>
__global__ __launch_bounds__(BAND_T, 8) void k_band_few(float *__restrict__ r, Tables t, Cand c, uint32_t *__restrict__ idx, void *__restrict__ val, uint32_t *__restrict__ err)
{
    __shared__ __align__(16) uint32_t pool[2 * TILE];
    if (t.nhard[0] == 0u) return;                    /* every bucket was coded from its staged elements */
    band_tiles<BITS, BAND_T>(r, t, c, idx, val, err, (1u << PATH_BAND) | (1u << PATH_ZERO), pool, blockIdx.x, gridDim.x);
}

/* Value coding of the survivors the ordered writes above left uncoded in idx / vdst: every chunk
 * of a PATH_DENSE bucket, and of the band / zero-threshold buckets the chunks that the one-pass
 * coding could not complete (all of them when it was not used).  Leaves at once when every
 * bucket was coded from its staged elements.  Chunks of up to 256 survivors: a wavefront per
 * chunk, QUANT_PER_WAVE chunks per wavefront; longer chunks: a workgroup each. */
constexpr uint32_t QUANT_WAVE_CHUNK = 256;
constexpr uint32_t QUANT_BIG_PER_WG = 8;
template <int BITS>
__global__ __launch_bounds__(WG) void k_quant(const float *__restrict__ v, const uint32_t *__restrict__ idx, Tables t,
                                              Cand c, float *__restrict__ r, void *__restrict__ val,
                                              float *__restrict__ scales, const uint32_t *__restrict__ chunk_b,
                                              const uint32_t *__restrict__ chunk_seg, uint64_t n_chunks, int stream_coding)
{
    if (t.nhard[0] == 0u) return;
    if (t.chunk <= QUANT_WAVE_CHUNK) {
        /* which of the workgroup's chunks are still to be coded: one lane per chunk */
        constexpr uint32_t PER_WG = (WG / 64) * QUANT_PER_WAVE;
        __shared__ uint32_t todo_sh;
        const uint64_t cw = (uint64_t)blockIdx.x * PER_WG;
        if (threadIdx.x < 64) {
            const uint64_t cid = cw + threadIdx.x;
            bool todo = false;
            if (threadIdx.x < PER_WG && cid < n_chunks) {
                const uint32_t b = chunk_b[cid];
                const uint32_t path = t.fast[b];
                todo = path != PATH_CAND && path != PATH_LEFT;
                if (todo && stream_coding && path != PATH_DENSE)
                    todo = !chunk_coded_by_stream(t, c, b, cid - t.C[b], chunk_seg[cid]);
            }
            const uint64_t bal = __ballot(todo);
            if (threadIdx.x == 0) todo_sh = (uint32_t)bal;
        }
        wg_sync();
        const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        const uint32_t mine = (todo_sh >> (wave * QUANT_PER_WAVE)) & ((1u << QUANT_PER_WAVE) - 1u);
        if (mine) quant_wave<BITS>(v, idx, t, r, val, scales, chunk_b, cw + wave * QUANT_PER_WAVE, mine);
    } else {
        /* longer chunks: up to QUANT_BIG_PER_WG per workgroup, one after the other; which of them
         * are still to be coded is found by one lane per chunk first */
        __shared__ uint32_t todo_big;
        const uint32_t per = (uint32_t)((n_chunks + gridDim.x - 1) / gridDim.x);
        const uint64_t cw = (uint64_t)blockIdx.x * per;
        if (threadIdx.x < 64) {
            const uint64_t cid = cw + threadIdx.x;
            bool todo = false;
            if (threadIdx.x < per && cid < n_chunks) {
                const uint32_t b = chunk_b[cid];
                const uint32_t path = t.fast[b];
                todo = path != PATH_CAND && path != PATH_LEFT;
                if (todo && stream_coding && path != PATH_DENSE)
                    todo = !chunk_coded_by_stream(t, c, b, cid - t.C[b], chunk_seg[cid]);
            }
            const uint64_t bal = __ballot(todo);
            if (threadIdx.x == 0) todo_big = (uint32_t)bal;
        }
        wg_sync();
        uint32_t mask = todo_big;
        while (mask) {
            const uint32_t q = (uint32_t)__builtin_ctz(mask);
            mask &= mask - 1u;
            wg_sync();                         /* the previous chunk's use of LDS is over */
            quant_body<BITS>(v, idx, t, r, val, scales, chunk_b, cw + q);
        }
    }
}

/* ------------------------------------------------------------------ weight stage: the bitmap */

/* The staged band elements of a bucket decided from its band that are pruned get their bit in the
 * bitmap (k_whist left 0 for the whole band): below the threshold key, or equal to it and not
 * among the first e equal ones in index order (k_select_finish left T, e and, per segment, the
 * number of equal keys before it).  Sixteen lanes per staging segment, four segments per
 * wavefront. */
__device__ __forceinline__ void wfix_body(const Tables &t, const Cand &c, uint32_t *__restrict__ pmask, uint32_t bid)
{
    const uint32_t lane = threadIdx.x & 63, sub = lane >> 4, gl = lane & 15u;
    const uint32_t ss = (bid * (WG / 64) + (threadIdx.x >> 6)) * 4u + sub;
    uint32_t cnt = 0, T = 0, e_b = 0, run_e = 0, b = 0, head = 0;
    if (ss < t.n_tiles) {
        b = t.tile_b[ss];
        if (t.fast[b] == PATH_BAND && t.k[b] != 0u) {
            cnt = c.cnt[ss];
            T = t.T[b]; e_b = t.need[b]; run_e = c.E[ss];
            head = (uint32_t)(t.off[b] & 3ull);
        }
    }
    uint32_t maxcnt = cnt;
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) maxcnt = max(maxcnt, (uint32_t)__shfl_xor(maxcnt, d, 64));
    const uint64_t base = (uint64_t)ss * SEG_CAP;
    for (uint32_t i0 = 0; i0 < maxcnt; i0 += 16) {
        const uint32_t i = i0 + gl;
        const bool in = i < cnt;
        const uint32_t key = in ? keyof(c.val[base + i]) : 0u;
        const uint32_t li = in ? c.idx[base + i] : 0u;
        const bool ise = in && key == T;
        const uint32_t be = (uint32_t)(__ballot(ise) >> (sub * 16u)) & 0xFFFFu;
        const uint32_t pe = run_e + __popc(be & ((1u << gl) - 1u));
        if (in && (key < T || (ise && pe >= e_b))) {
            const uint64_t e = (uint64_t)li + head;          /* position counted from the bucket's first tile */
            const uint32_t tile = t.tile0[b] + (uint32_t)(e / TILE);
            const uint32_t inq = (uint32_t)(e % TILE);
            atomicOr(&pmask[(uint64_t)tile * (TILE / 32) + (inq >> 5)], 1u << (inq & 31u));
        }
        run_e += __popc(be);
    }
}

/* Bitmap of a bucket that went through the dense passes (T, e and the per-segment prefixes are
 * known): one wavefront per staging segment walks the weights it covers in index order; a weight
 * is kept when its key exceeds T or equals it among the first e such, everything else gets its
 * bit.  Every word of the bucket's tiles is written. */
__device__ __forceinline__ void mask_dense_body(const float *__restrict__ w, const Tables &t, const Cand &c,
                                                uint32_t *__restrict__ pmask, uint32_t bid, uint32_t nblk)
{
    const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint64_t lt = (1ull << lane) - 1ull;
    for (uint32_t ss = bid * (WG / 64) + wave; ss < t.n_tiles; ss += nblk * (WG / 64)) {
        const uint32_t b = t.tile_b[ss];
        if (t.fast[b] != PATH_DENSE || t.k[b] == 0u) continue;
        const TileGeo s = tile_geo(t, b, ss);
        const uint32_t T = t.T[b], e_b = t.need[b];
        uint32_t run_e = c.E[ss];
        constexpr uint32_t wt0 = 0, wt1 = TILE / WTILE;
        for (uint32_t wt = wt0; wt < wt1; ++wt) {
            const uint64_t wb = s.base + (uint64_t)wt * WTILE;
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const uint64_t gi = wb + (uint64_t)(u * 64 + lane) * 4;
                float x[4];
                const uint32_t m = load_quad(w, gi, s.lo, s.hi, x);
                uint32_t fe = 0, bits = 0;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const uint32_t key = keyof(x[j]);
                    if ((m >> j) & 1u) { fe |= (key == T ? 1u : 0u) << j; bits |= (key < T ? 1u : 0u) << j; }
                }
                uint32_t pe = run_e, te = 0;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const uint64_t be = __ballot((fe >> j) & 1u);
                    pe += __popcll(be & lt);
                    te += __popcll(be);
                }
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const bool ise = (fe >> j) & 1u;
                    if (ise && pe >= e_b) bits |= 1u << j;
                    pe += ise ? 1u : 0u;
                }
                run_e += te;
                uint32_t word = bits << ((lane & 7u) * 4u);
                word |= __shfl_xor(word, 1, 64);
                word |= __shfl_xor(word, 2, 64);
                word |= __shfl_xor(word, 4, 64);
                if ((lane & 7u) == 0u)
                    pmask[(uint64_t)ss * (TILE / 32) + wt * (WTILE / 32) + u * 8 + (lane >> 3)] = word;
            }
        }
    }
}

/* The weight buckets on the dense passes (no usable band, a band that missed or overflowed), by a
 * small resident team with barriers between the steps, like k_hard: list of tiles,
 * up to three histograms of |w| and their digits, counts per segment, prefixes,
 * bitmap.  Leaves at once when there is no such bucket.  k_whard: the team alone (force_dense); k_wrest: the team is the first workgroups of
 * the launch, which also keep the buckets' records (what the next call's band is built from; what the plan was made from left clean for the
 * gradient), the others complete the bitmap of the staged bands (three launches that waited for each other, 109 M weights in 199 buckets: 16.3 + 4.7 + 4.7 us). */
__device__ __forceinline__ void whard_body(const float *__restrict__ w, const Tables &t, const Cand &c, uint32_t *__restrict__ f0,
                                           uint32_t *__restrict__ f1, uint32_t *__restrict__ f2, uint32_t *__restrict__ pmask,
                                           uint32_t *__restrict__ err, uint32_t *h, uint32_t bid, uint32_t nblk)
{
    if (t.nhard[2] == 0u) return;
    dense_threshold(w, t, c, f0, f1, f2, h, t.nhard + 1, bid, nblk, false, err);
    mask_dense_body(w, t, c, pmask, bid, nblk);
}
__global__ __launch_bounds__(WG) void k_whard(const float *__restrict__ w, Tables t, Cand c, uint32_t *__restrict__ f0,
                                              uint32_t *__restrict__ f1, uint32_t *__restrict__ f2, uint32_t *__restrict__ pmask,
                                              uint32_t *__restrict__ err)
{
    __shared__ uint32_t h[NB1];
    whard_body(w, t, c, f0, f1, f2, pmask, err, h, blockIdx.x, gridDim.x);
}
/* The bitmap of the staged bands alone: many tiles are better off without the registers and the LDS of the dense passes.  Beside it k_wrest
 * takes 4 - 5 us.  One launch / two, us together: 10 thousand tiles 4.4 / 8.5, 31 thousand 10.0 / 10.3, 47 thousand 13.8 / 14.6, 53 thousand in
 * 199 buckets 22.3 / 21.1 (the call 495.4 / 495.5), 78 thousand 22.2 / 20.3, 117 thousand 32.0 / 25.7, 390 thousand 104 / 72, 3.3 M (6.7 G
 * weights) 1029 / 643. */
__global__ __launch_bounds__(WG) void k_wfix(Tables t, Cand c, uint32_t *__restrict__ pmask) { wfix_body(t, c, pmask, blockIdx.x); }
__global__ __launch_bounds__(WG) void k_wrest(const float *__restrict__ w, Tables t, Cand c, uint32_t *__restrict__ f0,
                                              uint32_t *__restrict__ f1, uint32_t *__restrict__ f2, uint32_t *__restrict__ pmask,
                                              uint32_t *__restrict__ err, uint32_t team, uint32_t *__restrict__ hist,
                                              const uint32_t *__restrict__ nband, uint32_t *__restrict__ prevT, uint32_t *__restrict__ prevHw)
{
    __shared__ uint32_t h[NB1];
    if (blockIdx.x >= team) {
        wfix_body(t, c, pmask, blockIdx.x - team);
        return;
    }
    for (uint32_t b = blockIdx.x; b < t.B; b += team) {
        for (uint32_t i = threadIdx.x * 4u; i < NHC * HROW; i += WG * 4u) *reinterpret_cast<uint4 *>(hist + (uint64_t)b * NHC * HROW + i) = make_uint4(0u, 0u, 0u, 0u);
        if (threadIdx.x == 0) {
            if (t.k[b] == 0u) plan_weights_empty(t, b);
            t.ovf[b] = 0u;
            remember_weights(t, b, nband, prevT, prevHw);
        }
    }
    wg_sync();
    whard_body(w, t, c, f0, f1, f2, pmask, err, h, blockIdx.x, team);
}

}  // namespace

#endif
