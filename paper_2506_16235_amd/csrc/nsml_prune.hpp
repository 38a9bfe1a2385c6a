/*
 * libnsml device code, part 3: weight-magnitude pruning (Algorithm 2 Step 2).
 * Included by nsml_kernels.hip (one translation unit); not a public header.
 */
#ifndef NSML_PRUNE_HPP
#define NSML_PRUNE_HPP

namespace {

/* ------------------------------------------------------------------ model pruning (optional) */

/* Algorithm 2 Step 2 on the GPU: the kept parameters of a bucket are its n_b - floor(0.5 (1 -
 * ratio) n_b) largest |weight| (ties: lower index kept).  The kept set is more than half of
 * the bucket, so "candidates above a bound" would be most of it; instead the threshold is
 * bracketed by a band of keys [lo, hi) that holds the kw-th largest key: from a sample of |w|
 * with a wide margin, or, from the second call on, a narrow one around the threshold the call
 * before found (weights move little between steps).  One pass over the weights stages the
 * elements inside the band, counts those above it and writes the pruning bitmap (1 = pruned)
 * for everything outside it; the threshold key T and the number e of admitted elements equal to
 * T come from the staged elements alone (k_select_count / k_select_finish), and k_wrest sets the
 * bits of the band elements that turn out pruned.  A bucket whose band missed or overflowed
 * takes the dense ordered passes (k_wrest's first workgroups; k_whard when they are asked for), which write its bitmap.  The
 * gradient kernels read one bit per parameter.  Pruned parameters are neither counted nor emitted, and their accumulated gradient is
 * still written to the residual: pruning is not permanent. */

/* Per bucket: the band of keys [lo, hi) to stage, from the sample histogram of |w|, and the shift of
 * its bins.  The sample histogram is left clean. */
__global__ __launch_bounds__(WG) void k_wpredict(Tables t, uint32_t *__restrict__ hist_s, int force_dense, int miss,
                                                 const uint32_t *__restrict__ prevT, const uint32_t *__restrict__ prevHw)
{
    __shared__ uint32_t tmp[WG];
    __shared__ uint32_t res[6];          /* digit, above, at for the upper and the lower rank */
    const uint32_t b = blockIdx.x, tid = threadIdx.x;
    const uint64_t nb = t.off[b + 1] - t.off[b];
    const uint32_t k = t.k[b];
    const KeyPar nothing = make_uint4(NONE, NONE, NONE, SH1);
    if (b == 0 && tid < 4) t.nhard[tid] = 0u;      /* counted anew by k_select_count ([1]: the barrier of the dense passes) */
    if (nb == 0 || k == 0 || force_dense) {
        if (tid == 0) t.par[b] = nothing;
        return;
    }
    if (prevT && prevT[b] != NONE) {                 /* (then no sample was taken) */
        /* weights move little from one step to the next: a narrow band around the threshold the
         * last call found (remember_weights chose its width); if it misses, the dense passes decide */
        if (tid == 0) {
            const uint32_t T = prevT[b], hw = prevHw[b];
            KeyPar p;
            p.x = T > hw ? T - hw : 0u;
            p.y = p.z = (uint32_t)min((uint64_t)T + hw + 1ull, 0x7FFFFFFFull);
            p.w = window_shift(p.x, p.z);
            /* whole bins only: the undecided keys are those of one bin */
            p.x &= ~((1u << p.w) - 1u);
            t.par[b] = p;
        }
        return;
    }
    DigitWalk<NB0> w;
    w.load(hist_s + (uint64_t)b * NB0, tmp);
    w.clear(hist_s + (uint64_t)b * NB0);
    const uint32_t m = w.total;
    if (m == 0) {
        if (tid == 0) t.par[b] = nothing;
        return;
    }
    const bool exact = nb < SAMPLE_ALL_BELOW;
    const double ks = (double)k * (double)m / (double)nb;      /* sample rank of the threshold, from the top */
    const double dev = exact ? 0.0 : 4.0 * sqrt(ks) + 4.0;
    double r_up = floor(ks - dev), r_dn = ceil(ks + dev);
    if (r_up < 1.0) r_up = 1.0;
    if (r_dn < 1.0) r_dn = 1.0;
    if (r_dn > (double)m) r_dn = (double)m;
    if (r_up > (double)m) r_up = (double)m;
    uint32_t digit, above, at;
    if (w.find((uint32_t)r_up, digit, above, at)) { res[0] = digit; res[1] = above; res[2] = at; }
    if (w.find((uint32_t)r_dn, digit, above, at)) { res[3] = digit; res[4] = above; res[5] = at; }
    wg_sync();
    if (tid == 0) {
        /* sample entries inside the band -> expected staged elements */
        const double in_band = (double)(res[4] + res[5]) - (double)res[1];
        const double est = in_band * (double)nb / (double)m;
        const double cap_b = (double)(t.tile0[b + 1] - t.tile0[b]) * (double)SEG_CAP;
        KeyPar p = nothing;
        /* a bucket sampled in full whose kept set is all of it needs no band either way */
        if (est <= 0.8 * cap_b) {
            p.x = res[3] << SH0;
            p.y = p.z = (res[0] + 1u) << SH0;
            /* diagnostic: a band of two digits above the right one, so that the threshold is missed */
            if (miss) { p.x = (res[0] + 1u) << SH0; p.y = p.z = (res[0] + 3u) << SH0; }
            p.w = window_shift(p.x, p.z);
        }
        t.par[b] = p;
    }
}

/* One pass over the weights, a tile per workgroup like the gradient's streaming pass.  For a bucket
 * with a band [lo, hi): every element whose key lies in the band is staged and counted in its bin;
 * the elements above the band are only counted (c.G); and the pruning bitmap gets a first version: 1
 * for the elements below the band (pruned for certain), 0 for the rest (the few band elements that
 * end up pruned are set later by k_wrest).  A bucket without a band (no usable sample, or the dense
 * passes were asked for) is left to k_wrest or k_whard.  Bound by reading w, 4 bytes per element, a third of what
 * the gradient's pass has in flight per tile: so two wavefronts take a tile, 16 tiles per compute unit
 * (109 M elements: 147 us with eight wavefronts per tile). */
constexpr int WTH = 128;
template <bool HIST>
__global__ __launch_bounds__(WTH, 8) void k_whist(const float *__restrict__ w, Tables t, uint32_t *__restrict__ hist, Cand c,
                                                  uint32_t *__restrict__ pmask)
{
    constexpr int Q = TILE / (4 * WTH);
    __shared__ StageShared<HIST> sm;
    const uint32_t tile = grid_tile();
    if (tile >= t.n_tiles) return;
    const uint4 d = t.desc[tile];
    const uint32_t tid = threadIdx.x, lane = tid & 63, first = d.w & 0xFFFFu, last = d.w >> 16;
    const uint64_t g0 = ((uint64_t)d.y << 32) | d.x;
    const uint32_t b = d.z;
    const KeyPar p = t.par[b];
    if (p.x == NONE) {                                    /* same for the whole workgroup */
        if (tid == 0) { c.cnt[tile] = 0u; c.G[tile] = 0u; }
        return;
    }
    float a[Q][4];
    uint32_t m[Q];
    if (first == 0u && last == (uint32_t)TILE) {
        f4 x[Q];
#pragma unroll
        for (int u = 0; u < Q; ++u) x[u] = __builtin_nontemporal_load(reinterpret_cast<const f4 *>(w + g0 + (u * WTH + tid) * 4u));
#pragma unroll
        for (int u = 0; u < Q; ++u) { a[u][0] = x[u].x; a[u][1] = x[u].y; a[u][2] = x[u].z; a[u][3] = x[u].w; m[u] = 0xFu; }
    } else {
#pragma unroll
        for (int u = 0; u < Q; ++u) {
            m[u] = 0;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint32_t e = (u * WTH + tid) * 4u + j;
                a[u][j] = 0.0f;
                if (e >= first && e < last) { a[u][j] = w[g0 + e]; m[u] |= 1u << j; }
            }
        }
    }
#pragma unroll
    for (int u = 0; u < Q; ++u) {
        uint32_t bits = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) bits |= (((m[u] >> j) & 1u) && keyof(a[u][j]) < p.x ? 1u : 0u) << j;
        /* eight lanes share a word of the bitmap (four bits per quad): lane 8g collects the
         * words of lanes 8g .. 8g+7 by shifts inside its row of 16 lanes */
        uint32_t word = bits << ((lane & 7u) * 4u);
        word |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)word, 0x101, 0xF, 0xF, true);     /* from lane + 1 */
        word |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)word, 0x102, 0xF, 0xF, true);     /* from lane + 2 */
        word |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)word, 0x104, 0xF, 0xF, true);     /* from lane + 4 */
        if ((lane & 7u) == 0u) pmask[(uint64_t)tile * (TILE / 32) + ((u * WTH + tid) >> 3)] = word;
    }
    stage_tile<WTH, HIST>(a, m, p, b, tile, (uint32_t)(g0 - t.off[b]), c, hist, t.ovf + b, sm);
}

/* The plan of a bucket of weights, from the exact counts as plan_bucket has them for the gradient: the staged band decides the rest iff the kw-th
 * largest lies inside it, no staging segment overflowed and the list of undecided keys holds them, otherwise the
 * bucket takes the dense passes. */
__device__ __forceinline__ Plan plan_weights(const Tables &t, const KeyPar &p, uint32_t want, bool found, uint32_t bin, uint32_t above, uint32_t at,
                                             uint32_t ovf, uint32_t segs)
{
    const uint32_t top = (p.z - 1u) >> p.w;
    const bool known = p.x != NONE && found && !(bin == (uint32_t)NHB - 1u && (p.x >> p.w) != top - bin);      /* (not in the open last bin) */
    Plan q = {PATH_DENSE, 0u, want, SH_NONE, 0u};
    if (known) {
        q.T = top - bin; q.need = want - above; q.sh = p.w;
        if (!ovf && list_pays(at, segs, t.n_tiles)) q.path = PATH_BAND;
    }
    return q;
}
/* Its record (one thread per bucket). */
__device__ __forceinline__ void plan_weights_store(const Tables &t, uint32_t b, const Plan &q)
{
    t.T[b] = q.T;
    t.need[b] = q.need;
    t.sh[b] = q.sh;
    t.fast[b] = q.path;
    if (q.path == PATH_DENSE) atomicAdd(t.nhard + 2, 1u);      /* the dense passes have work */
    if (q.path == PATH_DENSE && q.sh == SH_NONE) atomicAdd(t.nhard + 3, 1u);
}
__device__ __forceinline__ void plan_weights_empty(const Tables &t, uint32_t b) { t.T[b] = NONE; t.need[b] = 0; t.fast[b] = PATH_BAND; t.sh[b] = SH0; }

/* The plan when every bucket is sent to the dense passes (force_dense): no band, so the next call has nothing to go by. */
__global__ __launch_bounds__(WG) void k_wplan_dense(Tables t, uint32_t *__restrict__ prevT)
{
    const uint32_t b = blockIdx.x * WG + threadIdx.x;
    if (b >= t.B) return;
    prevT[b] = NONE;
    if (t.k[b] == 0u) plan_weights_empty(t, b);
    else plan_weights_store(t, b, Plan{PATH_DENSE, 0u, t.k[b], SH_NONE, 0u});
}

/* What the next call's band is built from, per bucket: the threshold key this call found, and a
 * half-width that would have staged about 0.2 % of the bucket (at least 4096 elements, but no more
 * than a sixteenth of the bucket: a staging segment holds a quarter of its tile) at the
 * density of keys this call's band had.  A bucket that took the dense passes remembers nothing. */
__device__ __forceinline__ void remember_weights(const Tables &t, uint32_t b, const uint32_t *__restrict__ nband, uint32_t *__restrict__ prevT,
                                                 uint32_t *__restrict__ prevHw)
{
    const uint64_t nb = t.off[b + 1] - t.off[b];
    const KeyPar p = t.par[b];
    if (!t.fast[b] || t.k[b] == 0u || t.T[b] == NONE || p.x == NONE) { prevT[b] = NONE; return; }
    const uint64_t width = (uint64_t)p.z - p.x;
    const uint64_t some = nb / 16 < 4096 ? nb / 16 + 1 : 4096;
    const uint64_t target = nb / 512 > some ? nb / 512 : some;
    uint64_t hw = nband[b] ? width * target / (2ull * nband[b]) : width;
    hw = hw < 256 ? 256 : (hw > (1ull << 24) ? (1ull << 24) : hw);
    prevT[b] = t.T[b];
    prevHw[b] = (uint32_t)hw;
}

}  // namespace

#endif
