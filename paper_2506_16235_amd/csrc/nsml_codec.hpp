/*
 * libnsml device code, part 4: value coding of the survivors and the decompress kernels.
 * Included by nsml_kernels.hip (one translation unit); not a public header.
 */
#ifndef NSML_CODEC_HPP
#define NSML_CODEC_HPP

namespace {

/* ------------------------------------------------------------------ value coding */

/* The coding of quant_body (below) for chunks of at most 256 survivors, one wavefront per chunk and QUANT_PER_WAVE
 * chunks per wavefront, all of whose values and indices are fetched before any is used (with a
 * workgroup per small chunk the step is bound by the latency of its chain of dependent loads,
 * not by bandwidth).  A lane takes up to two pairs of consecutive survivors of each chunk. */
constexpr uint32_t QUANT_PER_WAVE = 4;
template <int BITS>
__device__ __forceinline__ void quant_wave(const float *__restrict__ v, const uint32_t *__restrict__ idx,
                                           const Tables &t, float *__restrict__ r, void *__restrict__ val,
                                           float *__restrict__ scales, const uint32_t *__restrict__ chunk_b,
                                           uint64_t c0, uint32_t todo)
{
    constexpr float QMAX = BITS == 8 ? 127.0f : 7.0f;
    const uint32_t lane = threadIdx.x & 63;
    uint32_t bq[QUANT_PER_WAVE], cnt[QUANT_PER_WAVE];
    uint64_t j0[QUANT_PER_WAVE], jg[QUANT_PER_WAVE], cbq[QUANT_PER_WAVE];
#pragma unroll
    for (uint32_t q = 0; q < QUANT_PER_WAVE; ++q) bq[q] = ((todo >> q) & 1u) ? chunk_b[c0 + q] : NONE;   /* bit q: chunk c0 + q is to be coded */
#pragma unroll
    for (uint32_t q = 0; q < QUANT_PER_WAVE; ++q) {
        cnt[q] = 0; j0[q] = jg[q] = cbq[q] = 0;
        if (bq[q] != NONE) {
            cbq[q] = c0 + q - t.C[bq[q]];
            j0[q] = cbq[q] * t.chunk;
            cnt[q] = (uint32_t)min((uint64_t)t.chunk, (uint64_t)t.k[bq[q]] - j0[q]);
            jg[q] = t.P[bq[q]] + j0[q];
        }
    }
    float x[QUANT_PER_WAVE][2][2];
    uint32_t li[QUANT_PER_WAVE][2][2];
#pragma unroll
    for (uint32_t q = 0; q < QUANT_PER_WAVE; ++q)
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int hh = 0; hh < 2; ++hh) {
                const uint32_t i = 2 * (lane + u * 64) + hh;
                x[q][u][hh] = i < cnt[q] ? v[jg[q] + i] : 0.0f;
                li[q][u][hh] = i < cnt[q] ? idx[jg[q] + i] : 0u;
            }
#pragma unroll
    for (uint32_t q = 0; q < QUANT_PER_WAVE; ++q) {
        if (cnt[q] == 0) continue;                             /* same for the whole wavefront */
        const uint32_t b = bq[q];
        const uint64_t lo = t.off[b];
        uint8_t *vb = reinterpret_cast<uint8_t *>(val) + t.V[b];
        float m = fmaxf(fmaxf(fabsf(x[q][0][0]), fabsf(x[q][0][1])), fmaxf(fabsf(x[q][1][0]), fabsf(x[q][1][1])));
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) m = fmaxf(m, __shfl_xor(m, d, 64));
        const float scale = m == 0.0f ? 0.0f : __fdiv_rn(m, QMAX);
        if (lane == 0) scales[t.S[b] + cbq[q]] = scale;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const uint32_t i0 = 2 * (lane + u * 64);
            if (i0 >= cnt[q]) continue;
            const int have = (i0 + 1 < cnt[q]) ? 2 : 1;
            float res[2] = {0.0f, 0.0f};
            int qq[2] = {0, 0};
#pragma unroll
            for (int hh = 0; hh < 2; ++hh) {
                if (hh >= have) continue;
                const float xv = x[q][u][hh];
                if (scale != 0.0f) {
                    float tq = rintf(__fdiv_rn(xv, scale));
                    tq = fminf(fmaxf(tq, -QMAX), QMAX);
                    qq[hh] = (int)tq;
                }
                if (BITS == 8) reinterpret_cast<int8_t *>(vb)[j0[q] + i0 + hh] = (int8_t)qq[hh];
                res[hh] = __fsub_rn(xv, __fmul_rn((float)qq[hh], scale));
            }
            if (BITS == 4) vb[(j0[q] + i0) >> 1] = (uint8_t)((qq[0] & 0xF) | ((qq[1] & 0xF) << 4));
#pragma unroll
            for (int hh = 0; hh < 2; ++hh)
                if (hh < have) r[lo + li[q][u][hh]] = res[hh];
        }
    }
}

/* A workgroup's work on one chunk of `chunk` consecutive survivors of a bucket whose survivors
 * were written by k_hard's ordered pass (not PATH_CAND): absmax, scale,
 * codes, packing, and the coding error left in the residual.  Every floating-point step is a
 * single correctly rounded binary32 operation (divide, round-to-nearest-even, multiply,
 * subtract); nothing may be contracted into an fma. */
template <int BITS>
__device__ __forceinline__ void quant_body(const float *__restrict__ v, const uint32_t *__restrict__ idx,
                                           const Tables &t, float *__restrict__ r, void *__restrict__ val,
                                           float *__restrict__ scales, const uint32_t *__restrict__ chunk_b,
                                           uint64_t c)
{
    __shared__ float red[WG / 64];
    const uint32_t tid = threadIdx.x;
    const uint32_t b = chunk_b[c];
    if (t.fast[b] == PATH_CAND) return;                     /* coded by k_encode */
    const uint64_t cb = c - t.C[b];
    const uint64_t j0 = cb * t.chunk;                         /* first survivor of the chunk, bucket-local */
    const uint32_t cnt = (uint32_t)min((uint64_t)t.chunk, (uint64_t)t.k[b] - j0);
    const uint64_t jg = t.P[b] + j0;                          /* same, global */
    const uint64_t lo = t.off[b];
    uint8_t *vb = reinterpret_cast<uint8_t *>(val) + t.V[b];
    /* A thread takes pairs of consecutive survivors (so a 4-bit pair is one byte store), up to
     * four pairs per block of 2048; the values and indices of a block are fetched before any is
     * used.  A chunk of up to 2048 is one block and its values are read once; a longer chunk
     * first takes its absmax in a pass of its own. */
    constexpr uint32_t BLK = WG * 8;
    const bool one_block = cnt <= BLK;
    float scale = 0.0f;
    if (!one_block) {
        float m = 0.0f;
        for (uint32_t i = tid; i < cnt; i += WG) m = fmaxf(m, fabsf(v[jg + i]));
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) m = fmaxf(m, __shfl_xor(m, d, 64));
        if ((tid & 63) == 0) red[tid >> 6] = m;
        wg_sync();
        m = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
        constexpr float QMAX = BITS == 8 ? 127.0f : 7.0f;
        scale = m == 0.0f ? 0.0f : __fdiv_rn(m, QMAX);
        if (tid == 0) scales[t.S[b] + cb] = scale;
    }
    for (uint32_t b0 = 0; b0 < cnt; b0 += BLK) {
        float x[4][2];
        uint32_t li[4][2];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
#pragma unroll
            for (int hh = 0; hh < 2; ++hh) {
                const uint32_t i = b0 + 2 * (tid + u * WG) + hh;
                x[u][hh] = i < cnt ? v[jg + i] : 0.0f;
                li[u][hh] = i < cnt ? idx[jg + i] : 0u;
            }
        }
        if (one_block) {
            float m = 0.0f;
#pragma unroll
            for (int u = 0; u < 4; ++u) m = fmaxf(m, fmaxf(fabsf(x[u][0]), fabsf(x[u][1])));   /* absent ones are 0 */
#pragma unroll
            for (int d = 32; d >= 1; d >>= 1) m = fmaxf(m, __shfl_xor(m, d, 64));
            if ((tid & 63) == 0) red[tid >> 6] = m;
            wg_sync();
            m = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
            constexpr float QMAX = BITS == 8 ? 127.0f : 7.0f;
            scale = m == 0.0f ? 0.0f : __fdiv_rn(m, QMAX);
            if (tid == 0) scales[t.S[b] + cb] = scale;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const uint32_t i0 = b0 + 2 * (tid + u * WG);
            if (i0 >= cnt) continue;
            const int have = (i0 + 1 < cnt) ? 2 : 1;
            float res[2] = {0.0f, 0.0f};
            int q[2] = {0, 0};
#pragma unroll
            for (int hh = 0; hh < 2; ++hh) {
                if (hh >= have) continue;
                const float xv = x[u][hh];
                constexpr float QMAX = BITS == 8 ? 127.0f : 7.0f;
                if (scale != 0.0f) {
                    float tq = rintf(__fdiv_rn(xv, scale));
                    tq = fminf(fmaxf(tq, -QMAX), QMAX);
                    q[hh] = (int)tq;
                }
                if (BITS == 8) reinterpret_cast<int8_t *>(vb)[j0 + i0 + hh] = (int8_t)q[hh];
                res[hh] = __fsub_rn(xv, __fmul_rn((float)q[hh], scale));
            }
            if (BITS == 4) vb[(j0 + i0) >> 1] = (uint8_t)((q[0] & 0xF) | ((q[1] & 0xF) << 4));
#pragma unroll
            for (int hh = 0; hh < 2; ++hh)
                if (hh < have) r[lo + li[u][hh]] = res[hh];
        }
    }
}

/* ------------------------------------------------------------------ decompress */

template <int BITS>
__device__ __forceinline__ float decode(const uint8_t *__restrict__ vb, const float *__restrict__ sc,
                                        uint64_t j, uint32_t chunk, uint32_t chunkSh)
{
    if (BITS == 32) return reinterpret_cast<const float *>(vb)[j];
    if (BITS == 16) return __half2float(reinterpret_cast<const __half *>(vb)[j]);
    int q;
    if (BITS == 8) q = reinterpret_cast<const int8_t *>(vb)[j];
    else {
        const uint32_t byte = vb[j >> 1];
        const int nib = (j & 1) ? (int)(byte >> 4) : (int)(byte & 0xFu);
        q = nib >= 8 ? nib - 16 : nib;
    }
    /* the usual chunk lengths are powers of two: a shift instead of a 64-bit division */
    return __fmul_rn((float)q, sc[chunkSh < 64u ? (j >> chunkSh) : j / chunk]);
}

/* Where each tile's survivors start in its bucket's ascending index list: ts[tile0[b] + b + i]
 * = number of survivors of bucket b with an index below tile i (i = 0..tiles_b).  A thread
 * takes TS_PER consecutive survivors (8 for long payloads, 2 for short ones, which need the
 * threads more); a survivor whose tile differs from its predecessor's writes the entries of
 * the tiles that begin between the two, and the last survivor of a bucket also closes the
 * bucket's remaining tiles. */

__device__ __forceinline__ void tilestart_one(const uint32_t *__restrict__ idx, const Tables &t, uint32_t b,
                                              uint64_t j, uint32_t *__restrict__ ts)
{
    const uint32_t tiles_b = t.tile0[b + 1] - t.tile0[b];
    const uint32_t kb = t.k[b];
    const uint32_t jj = (uint32_t)(j - t.P[b]);
    uint32_t *tsb = ts + t.tile0[b] + b;
    const uint32_t head = (uint32_t)(t.off[b] & 3ull);
    /* tile of a local index; indices beyond the bucket (invalid payload) count as the last tile */
    uint32_t tcur = (uint32_t)(((uint64_t)idx[j] + head) / TILE);
    tcur = min(tcur, tiles_b - 1);
    uint32_t tfrom = 0;                         /* first tile this survivor fills */
    if (jj > 0) {
        uint32_t tprev = (uint32_t)(((uint64_t)idx[j - 1] + head) / TILE);
        tprev = min(tprev, tiles_b - 1);
        tfrom = tprev + 1;
    }
    for (uint32_t tt = tfrom; tt <= tcur; ++tt) tsb[tt] = jj;
    if (jj == kb - 1)
        for (uint32_t tt = tcur + 1; tt <= tiles_b; ++tt) tsb[tt] = kb;
}

/* P: the buckets' first survivors, in memory or in LDS */
template <uint32_t TS_PER>
__device__ __forceinline__ void tilestart_walk(const uint32_t *__restrict__ idx, const Tables &t, const uint64_t *P, uint64_t K,
                                               uint32_t *__restrict__ ts)
{
    const uint64_t stride = (uint64_t)gridDim.x * WG * TS_PER;
    for (uint64_t j0 = ((uint64_t)blockIdx.x * WG + threadIdx.x) * TS_PER; j0 < K; j0 += stride) {
        const uint32_t b = find_bucket<uint64_t>(P, t.B, j0);
        const uint64_t Pb = P[b], Pn = P[b + 1];
        if (j0 > Pb && j0 + TS_PER < Pn) {
            /* all of them inside one bucket, none its first or last survivor: only tile changes matter */
            const uint32_t tiles_b = t.tile0[b + 1] - t.tile0[b];
            const uint32_t head = (uint32_t)(t.off[b] & 3ull);
            uint32_t *tsb = ts + t.tile0[b] + b;
            uint32_t v[TS_PER + 1];
#pragma unroll
            for (uint32_t i = 0; i <= TS_PER; ++i) v[i] = idx[j0 - 1 + i];
#pragma unroll
            for (uint32_t i = 0; i <= TS_PER; ++i) v[i] = min((uint32_t)(((uint64_t)v[i] + head) / TILE), tiles_b - 1);
            if (v[0] != v[TS_PER]) {
                const uint32_t jj0 = (uint32_t)(j0 - Pb);
#pragma unroll
                for (uint32_t i = 1; i <= TS_PER; ++i)
                    for (uint32_t tt = v[i - 1] + 1; tt <= v[i]; ++tt) tsb[tt] = jj0 + i - 1;
            }
        } else {
            for (uint64_t j = j0; j < min(K, j0 + TS_PER); ++j)
                tilestart_one(idx, t, j < Pn ? b : find_bucket<uint64_t>(P, t.B, j), j, ts);
        }
    }
}

template <uint32_t TS_PER>
__global__ __launch_bounds__(WG) void k_tilestart(const uint32_t *__restrict__ idx, Tables t,
                                                  uint64_t K, uint32_t *__restrict__ ts)
{
    constexpr uint32_t LDS_B = 2047;
    __shared__ uint64_t sP[LDS_B + 1];
    if (t.B <= LDS_B) {
        for (uint32_t i = threadIdx.x; i <= t.B; i += WG) sP[i] = t.P[i];
        wg_sync();
        tilestart_walk<TS_PER>(idx, t, sP, K, ts);
    } else {
        tilestart_walk<TS_PER>(idx, t, t.P, K, ts);
    }
}

/* The same table by binary search, one thread per tile: cheaper than walking the whole index
 * list once a tile holds many survivors (high ratios).  An index list that is not ascending (an
 * invalid payload) gives entries that are wrong but still within [0, k_b]. */
__device__ __forceinline__ void tilestart_find(const uint32_t *__restrict__ idx, const Tables &t, uint32_t g, uint32_t *__restrict__ ts)
{
    const uint32_t b = find_bucket<uint32_t>(t.tile0, t.B, g);
    const uint32_t i = g - t.tile0[b], tiles_b = t.tile0[b + 1] - t.tile0[b];
    const uint32_t kb = t.k[b];
    const uint32_t *ib = idx + t.P[b];
    const uint64_t head = t.off[b] & 3ull;
    const uint64_t edge = (uint64_t)i * TILE;           /* survivors with index + head below this come first */
    uint32_t lo = 0, hi = kb;                           /* first j in [0, kb] with ib[j] + head >= edge */
    while (lo < hi) {
        const uint32_t mid = lo + ((hi - lo) >> 1);
        if ((uint64_t)ib[mid] + head < edge) lo = mid + 1; else hi = mid;
    }
    uint32_t *tsb = ts + t.tile0[b] + b;
    tsb[i] = lo;
    if (i + 1 == tiles_b) tsb[tiles_b] = kb;
}
__global__ __launch_bounds__(WG) void k_tilestart_search(const uint32_t *__restrict__ idx, Tables t, uint32_t n_tiles,
                                                         uint32_t *__restrict__ ts)
{
    const uint32_t g = blockIdx.x * WG + threadIdx.x;
    if (g < n_tiles) tilestart_find(idx, t, g, ts);
}

/* One of its entries by a wavefront: the first j in [0, kb] with ib[j] + head >= edge.  per: survivors per element of the bucket.
 * Bound by round trips, by the lines they fetch, and in short lists by its instructions (edge and list are the same for the wavefront: scalar).
 * In lists of more than two rounds of 64 probes the first round probes where the rounds after it can resolve the distance.  All tiles of
 * the bucket probe the same lines there, and it shows how the survivors lie.
 * Where they are spread evenly the edge's place is then known to a few of them after one or two looks at 64 neighbours, three lines each.
 * Where they are clustered the rounds of probes, a line each, go on: no round is lost to them.
 * (Up to 65536 survivors the probes lie 1024 apart, so that one look nearly always does.)
 * Short lists look first: it may be the only round.
 * The kernel in a worker's round, us, by probes alone / looks before any probe / this.  ResNet-50's shape at 0.2: normal values 29.7 / 24.9 / 26.2,
 * nine rows of 768 in ten zero 24.4 / 29.3 / 23.9, clipped at one sigma (of the equal ones the first are sent) 29.2 / 31.5 / 28.8; 30 M in
 * one bucket at 0.01 25.6 / 21.8 / 22.0; 110 M in 250 buckets at 0.01 88.4 / 87.4 / 82.9, but lists not in the caches 83.0 / 92.8 / 89.0 (the probes
 * of one tile fetch its neighbours' lines); 60 Ki in 24 buckets, rows, at 0.05 4.3 / 4.9 / 4.6.
 * A list that is not ascending (an invalid payload) gives entries that are wrong but still within [0, kb]. */
__device__ __forceinline__ uint32_t tilestart_wave(const uint32_t *__restrict__ ib, uint32_t kb, uint32_t head, uint64_t edge, float per)
{
    if (edge <= head) return 0u;
    const uint32_t lane = threadIdx.x & 63, e = (uint32_t)(edge - head);       /* (an element of the bucket, or their number) */
    uint32_t lo = 0, hi = kb;
    float want = (float)e * per, span = (float)kb;       /* where the edge should be; off by half the root of span at most, if survivors are spread evenly */
    uint32_t looks = 2;
    bool even = true;
    if (kb > 4160u) {
        const uint32_t step = kb <= 65536u ? 1024u : kb <= 266304u ? 4161u : kb <= 17043520u ? 266305u : 17043521u;
        const uint32_t p = lane * step, v = ib[min(p, kb - 1u)];
        const uint64_t beyond = __ballot(p >= kb || v >= e);
        const uint32_t f = beyond ? (uint32_t)__builtin_ctzll(beyond) : 64u;      /* the first probe at or beyond the edge */
        if (f == 0u) return 0u;
        const float d = (float)v * per - (float)p;
        even = !__any(p < kb && d * d > 4.0f * span + 4096.0f);
        hi = f < 64u ? min(kb, f * step) : kb;
        lo = (f - 1u) * step + 1u;
        want = (float)lo + (float)(uint32_t)__builtin_amdgcn_readlane((int)(e - v), (int)(f - 1u)) * per;
        span = (float)step;
        looks = 3;
    }
#pragma unroll 1
    for (; even && looks && hi - lo > 64u; --looks) {
        /* 64 neighbours, half of them before it */
        const uint32_t at = min(max((uint32_t)fminf(fmaxf(want - 32.0f, 0.0f), 4294966784.0f), lo), hi - 64u), v = ib[at + lane];
        const uint64_t beyond = __ballot(v >= e);
        if (beyond && !(beyond & 1ull)) return at + (uint32_t)__builtin_ctzll(beyond);
        const uint32_t to = beyond ? at : at + 64u;      /* the edge is not beyond it, or not before */
        const int diff = __builtin_amdgcn_readlane((int)(e - v), beyond ? 0 : 63);
        const float off = (beyond ? -(float)(0u - (uint32_t)diff) : (float)(uint32_t)diff) * per;
        if (beyond) hi = to; else lo = to;
        want = (float)to + off;
        even = off * off <= 4.0f * span + 1024.0f;
        span = fabsf(off);
    }
    while (lo < hi) {                                    /* (the range shrinks every round, whatever the list holds) */
        const uint32_t n = hi - lo, step = (n - 1u) / 64u + 1u, p = lane * step;
        const uint64_t beyond = __ballot(p >= n || ib[lo + min(p, n - 1u)] >= e);
        const uint32_t f = beyond ? (uint32_t)__builtin_ctzll(beyond) : 64u;
        hi = lo + min(n, f * step);
        if (f) lo += (f - 1u) * step + 1u;
    }
    return lo;
}

/* Four consecutive values j0 .. j0 + 3 of a bucket's value stream, decoded; 8- and 32-bit ones in one
 * load (the stream of a bucket starts at any byte, so the address is not aligned; global loads need
 * not be). */
template <int BITS>
__device__ __forceinline__ void decode4(const uint8_t *__restrict__ vb, const float *__restrict__ sc, uint64_t j0,
                                        uint32_t chunk, uint32_t chunkSh, float (&x)[4])
{
    if (BITS == 32) {
        f4 v;
        __builtin_memcpy(&v, vb + 4 * j0, 16);
        x[0] = v.x; x[1] = v.y; x[2] = v.z; x[3] = v.w;
    } else if (BITS == 8) {
        uint32_t w4;
        __builtin_memcpy(&w4, vb + j0, 4);
        const uint64_t c0 = chunkSh < 64u ? (j0 >> chunkSh) : j0 / chunk;
        const uint64_t c3 = chunkSh < 64u ? ((j0 + 3) >> chunkSh) : (j0 + 3) / chunk;
        const float s0 = sc[c0], s3 = c3 == c0 ? s0 : sc[c3];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint64_t cj = chunkSh < 64u ? ((j0 + j) >> chunkSh) : (j0 + j) / chunk;
            x[j] = __fmul_rn((float)(int)(int8_t)(w4 >> (8 * j)), cj == c0 ? s0 : s3);
        }
    } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) x[j] = decode<BITS>(vb, sc, j0 + j, chunk, chunkSh);
    }
}

/* Dense output, a tile per workgroup: every output line is written once, past the caches (with plain stores
 * half of 4 M elements into one of nine buffers 19.0 us, so 15.8; 25 M at ratio 0.05 36.2 and 27.4).  An empty
 * tile is zeros at once.  Otherwise the tile is assembled in LDS (zeros, then the decoded survivors that fall
 * inside it, found through the tile-start table, or with few tiles by a search of its own: see launch_decompress).  Where a tile has four survivors and more for every thread, a
 * thread takes four consecutive ones at a time, indices and codes each in one load (419 M elements at ratio 0.9:
 * 8-bit codes 642 us, one by one 776; for 32-bit values, whose loads are as wide either way, 852 and 839, so not
 * there).  A bucket of which every element was sent needs neither LDS nor its index list: its output is the
 * decoded value stream.  Bound by the 4 bytes per element written; the chain tile -> survivors' place ->
 * survivors -> LDS is four memory round trips long, so a compute unit has to hold many tiles.  NTH: see
 * launch_decompress.  MAP: type of the tile -> bucket table (16 bits for the entry point without a context). */
template <int BITS, typename MAP, int NTH>
__global__ __launch_bounds__(NTH, 8) void k_decomp(const uint32_t *__restrict__ idx, const void *__restrict__ val,
                                                   const float *__restrict__ scales, Tables t, const MAP *__restrict__ tile_b,
                                                   const uint32_t *__restrict__ ts, float *__restrict__ dense)
{
    constexpr int U = TILE / (4 * NTH);          /* 16-byte stores per thread */
    constexpr int S = TILE / NTH < 8 ? TILE / NTH : 8;      /* survivors a thread has in flight */
    __shared__ float slots[TILE];
    const uint32_t tile = grid_tile();
    if (tile >= t.n_tiles) return;
    const uint32_t tid = threadIdx.x;
    const uint32_t b = tile_b[tile];
    const TileGeo s = tile_geo(t, b, tile);
    const uint32_t kb = t.k[b], nb = (uint32_t)(s.hi - s.lo);
    const uint32_t *ib = idx + t.P[b];
    const uint8_t *vb = reinterpret_cast<const uint8_t *>(val) + t.V[b];
    const float *sb = BITS <= 8 ? scales + t.S[b] : nullptr;
    f4 out[U];
#pragma unroll
    for (int u = 0; u < U; ++u) out[u] = f4{0.f, 0.f, 0.f, 0.f};
    if (kb == nb) {
        /* every element of the bucket was sent (ratio 1, or a bucket of one element): survivor j is
         * element j, so the index list (which can only be 0 .. n_b - 1) is not read */
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint64_t gi = s.base + (u * NTH + tid) * 4u;
            float x[4];
            if (gi >= s.lo && gi + 4 <= s.hi) {
                decode4<BITS>(vb, sb, gi - s.lo, t.chunk, t.chunkSh, x);
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    x[j] = (gi + j >= s.lo && gi + j < s.hi) ? decode<BITS>(vb, sb, gi + j - s.lo, t.chunk, t.chunkSh) : 0.0f;
            }
            out[u] = f4{x[0], x[1], x[2], x[3]};
        }
    } else {
        uint32_t j0, j1;
        if (ts) {
            j0 = min(ts[tile + b], kb); j1 = min(ts[tile + b + 1], kb);
        } else {
            /* no table: a wavefront each for the tile's first survivor and the one after its last */
            __shared__ uint32_t place[2];
            const uint32_t w = __builtin_amdgcn_readfirstlane(tid >> 6), i = tile - t.tile0[b] + w, tiles_b = t.tile0[b + 1] - t.tile0[b];
            if (w < 2u) {
                const uint32_t at = i >= tiles_b ? kb : tilestart_wave(ib, kb, (uint32_t)(s.lo & 3ull), (uint64_t)i * TILE, (float)kb / (float)nb);
                if ((tid & 63u) == 0u) place[w] = at;
            }
            wg_sync();
            j0 = place[0]; j1 = place[1];
        }
        if (j0 < j1) {                                   /* same for the whole workgroup */
            const uint64_t shift = s.lo - s.base;        /* slot = local index + lo - base */
#pragma unroll
            for (int u = 0; u < U; ++u) *reinterpret_cast<f4 *>(&slots[(u * NTH + tid) * 4]) = out[u];
            wg_sync();
            uint32_t one = j0;                           /* from here on one by one */
            if (BITS <= 16 && j1 - j0 >= 4u * NTH) {
                constexpr int V = TILE / (4 * NTH) < 2 ? 1 : 2;      /* groups a thread has in flight */
                const uint32_t ngrp = (j1 - j0) / 4u;
                one = j0 + 4u * ngrp;
                for (uint32_t q0 = 0; q0 < ngrp; q0 += V * NTH) {
                    uint4 li[V];
                    float x[V][4];
#pragma unroll
                    for (int v = 0; v < V; ++v) {
                        const uint32_t q = q0 + v * NTH + tid;
                        li[v] = make_uint4(NONE, NONE, NONE, NONE);
                        x[v][0] = x[v][1] = x[v][2] = x[v][3] = 0.0f;
                        if (q < ngrp) {
                            const uint64_t j = (uint64_t)j0 + 4ull * q;
                            __builtin_memcpy(&li[v], ib + j, 16);        /* (aligned to 4) */
                            decode4<BITS>(vb, sb, j, t.chunk, t.chunkSh, x[v]);
                        }
                    }
#pragma unroll
                    for (int v = 0; v < V; ++v) {
                        const uint32_t l4[4] = {li[v].x, li[v].y, li[v].z, li[v].w};
#pragma unroll
                        for (int u = 0; u < 4; ++u) {
                            const uint64_t slot = (uint64_t)l4[u] + shift;
                            if (l4[u] < nb && slot < TILE) slots[slot] = x[v][u];
                        }
                    }
                }
            }
            for (uint64_t jb = one; jb < j1; jb += S * NTH) {
                uint32_t li[S];
                float x[S];
#pragma unroll
                for (int u = 0; u < S; ++u) {
                    const uint64_t j = jb + (uint64_t)u * NTH + tid;
                    li[u] = NONE;
                    x[u] = 0.0f;
                    if (j < j1) { li[u] = ib[j]; x[u] = decode<BITS>(vb, sb, j, t.chunk, t.chunkSh); }
                }
#pragma unroll
                for (int u = 0; u < S; ++u) {
                    /* an index outside the bucket or outside this tile (invalid payload) is dropped */
                    const uint64_t slot = (uint64_t)li[u] + shift;
                    if (li[u] < nb && slot < TILE) slots[slot] = x[u];
                }
            }
            wg_sync();
#pragma unroll
            for (int u = 0; u < U; ++u) out[u] = *reinterpret_cast<const f4 *>(&slots[(u * NTH + tid) * 4]);
        }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const uint64_t gi = s.base + (u * NTH + tid) * 4u;
        if (gi >= s.lo && gi + 4 <= s.hi) {
            st_out<true>(reinterpret_cast<f4 *>(dense + gi), out[u]);
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (gi + j >= s.lo && gi + j < s.hi) dense[gi + j] = out[u][j];
        }
    }
}

/* ------------------------------------------------------------------ everything is sent */

/* The whole of a compress call in which every element of every bucket is sent (ratio 1, the
 * controller's cap): nothing is selected, survivor j of a bucket is its element j.  One pass: a = g + r,
 * indices, values or codes, and the coding error over the residual.  A workgroup takes tile i of a
 * bucket counted from the bucket's own start, so that chunks of 2048 / 2^x survivors (the host checks)
 * nest in tiles and a scale needs one exchange inside the workgroup.  Bound by HBM: 8 bytes read and
 * 8 + payload per element written (419 M elements, 32-bit values: 1.35 ms in one bucket, 1.43 in 16, 5.9 - 6.2
 * TB/s; selection, dense encode and the launches between took 2.25).
 * By-products as from the streaming pass: |grad|^2 and the number of zeros per tile. */
template <int BITS, bool NT>
__global__ __launch_bounds__(STH, 8) void k_full(const float *__restrict__ g, float *__restrict__ r, Tables t, Cand c,
                                                 double *__restrict__ tile_sq, uint32_t *__restrict__ idx_out,
                                                 void *__restrict__ val, float *__restrict__ scales)
{
    constexpr float QMAX = BITS == 8 ? 127.0f : 7.0f;
    __shared__ double sq_w[STH / 64];
    __shared__ uint32_t z_w[STH / 64];
    __shared__ float red[STH / 64];
    const uint32_t tile = grid_tile();
    if (tile >= t.n_tiles) return;
    const uint32_t b = t.tile_b[tile];
    const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint64_t lo = t.off[b];
    const uint32_t nb = (uint32_t)(t.off[b + 1] - lo);
    const uint64_t e64 = (uint64_t)(tile - t.tile0[b]) * TILE + tid * 4u;      /* local index of this thread's first element */
    const uint32_t have = e64 >= nb ? 0u : (uint32_t)min((uint64_t)4, nb - e64);
    const uint32_t e0 = (uint32_t)e64;
    float a[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    double sq = 0.0;
    f4 x, y;
    if (have == 4u) {
        /* (a bucket may start at any element: 16-byte accesses that are aligned to 4) */
        if (NT) {
            x = __builtin_nontemporal_load(reinterpret_cast<const f4 *>(g + lo + e0));
            y = __builtin_nontemporal_load(reinterpret_cast<const f4 *>(r + lo + e0));
        } else {
            __builtin_memcpy(&x, g + lo + e0, 16);
            __builtin_memcpy(&y, r + lo + e0, 16);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) a[j] = __fadd_rn(x[j], y[j]);
        sq = (double)(__fmaf_rn(x.x, x.x, __fmul_rn(x.y, x.y)) + __fmaf_rn(x.z, x.z, __fmul_rn(x.w, x.w)));
    } else {
#pragma unroll
        for (uint32_t j = 0; j < 4; ++j)
            if (j < have) {
                const float xv = g[lo + e0 + j];
                a[j] = __fadd_rn(xv, r[lo + e0 + j]);
                sq += (double)__fmul_rn(xv, xv);
            }
    }
    uint32_t zeros = 0;
#pragma unroll
    for (uint32_t j = 0; j < 4; ++j) zeros += __popcll(__ballot(j < have && keyof(a[j]) == 0u));
    sq = wave_sum_last(sq);
    if (lane == 63) { sq_w[wave] = sq; z_w[wave] = zeros; }
    uint8_t *vb = reinterpret_cast<uint8_t *>(val) + t.V[b];
    const uint64_t Pb = t.P[b];
    float scale = 0.0f;
    if (BITS <= 8) {
        float m = 0.0f;
#pragma unroll
        for (int j = 0; j < 4; ++j) m = fmaxf(m, fabsf(a[j]));
        const uint32_t cq = t.chunk / 4u;                   /* threads per chunk: a power of two from 2 to 512 */
        for (uint32_t d = 1; d < 64u && d < cq; d <<= 1) m = fmaxf(m, __shfl_xor(m, (int)d, 64));
        if (lane == 0) red[wave] = m;
        wg_sync();
        if (cq > 64u) {
            const uint32_t wpc = cq / 64u, w0 = wave & ~(wpc - 1u);
            for (uint32_t w = w0; w < w0 + wpc; ++w) m = fmaxf(m, red[w]);
        }
        scale = m == 0.0f ? 0.0f : __fdiv_rn(m, QMAX);
        if (have && tid % cq == 0u) scales[t.S[b] + e0 / t.chunk] = scale;
    } else {
        wg_sync();
    }
    if (tid == 0) {
        double tot = 0.0;
        uint32_t z = 0;
#pragma unroll
        for (uint32_t w = 0; w < STH / 64; w += 4) {
            tot += (sq_w[w] + sq_w[w + 1]) + (sq_w[w + 2] + sq_w[w + 3]);
            z += (z_w[w] + z_w[w + 1]) + (z_w[w + 2] + z_w[w + 3]);
        }
        tile_sq[tile] = tot;
        c.E[tile] = z;
    }
    float left[4];
    int q[4];
    uint16_t hbits[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        float deq = a[j];
        q[j] = 0; hbits[j] = 0;
        if (BITS == 16) {
            const __half hv = __float2half_rn(a[j]);
            hbits[j] = __half_as_ushort(hv);
            deq = __half2float(hv);
        } else if (BITS <= 8) {
            if (scale != 0.0f) {
                float tq = rintf(__fdiv_rn(a[j], scale));
                tq = fminf(fmaxf(tq, -QMAX), QMAX);
                q[j] = (int)tq;
            }
            deq = __fmul_rn((float)q[j], scale);
        }
        left[j] = __fsub_rn(a[j], deq);        /* 32 bits: nothing is left behind (NaN where no value was) */

    }
    if (have == 4u) {
        const f4 rv = {left[0], left[1], left[2], left[3]}, av = {a[0], a[1], a[2], a[3]};
        const uint4 iv = make_uint4(e0, e0 + 1u, e0 + 2u, e0 + 3u);
        if (NT) {
            f4 fi;
            __builtin_memcpy(&fi, &iv, 16);
            __builtin_nontemporal_store(rv, reinterpret_cast<f4 *>(r + lo + e0));
            __builtin_nontemporal_store(fi, reinterpret_cast<f4 *>(idx_out + Pb + e0));
            if (BITS == 32) __builtin_nontemporal_store(av, reinterpret_cast<f4 *>(vb + 4ull * e0));
        } else {
            __builtin_memcpy(r + lo + e0, &rv, 16);
            __builtin_memcpy(idx_out + Pb + e0, &iv, 16);
            if (BITS == 32) __builtin_memcpy(vb + 4ull * e0, &av, 16);
        }
        if (BITS == 16) __builtin_memcpy(vb + 2ull * e0, hbits, 8);
        if (BITS == 8) {
            const uint32_t w = (uint32_t)(q[0] & 0xFF) | ((uint32_t)(q[1] & 0xFF) << 8) | ((uint32_t)(q[2] & 0xFF) << 16) | ((uint32_t)(q[3] & 0xFF) << 24);
            __builtin_memcpy(vb + e0, &w, 4);
        }
        if (BITS == 4) {
            const uint16_t w = (uint16_t)((q[0] & 0xF) | ((q[1] & 0xF) << 4) | ((q[2] & 0xF) << 8) | ((q[3] & 0xF) << 12));
            __builtin_memcpy(vb + (e0 >> 1), &w, 2);
        }
    } else {
#pragma unroll
        for (uint32_t j = 0; j < 4; ++j)
            if (j < have) {
                r[lo + e0 + j] = left[j];
                idx_out[Pb + e0 + j] = e0 + j;
                if (BITS == 32) reinterpret_cast<float *>(vb)[e0 + j] = a[j];
                if (BITS == 16) reinterpret_cast<uint16_t *>(vb)[e0 + j] = hbits[j];
                if (BITS == 8) vb[e0 + j] = (uint8_t)q[j];
                if (BITS == 4 && (j & 1u) == 0u) vb[(e0 + j) >> 1] = (uint8_t)((q[j] & 0xF) | (j + 1 < have ? (q[j + 1] & 0xF) << 4 : 0));
            }
    }
}

/* The per-bucket records of such a call: |grad|^2 and the selection state (threshold key 0, the zeros
 * admitted as its ties).  Bound by the latency of its loads: a thread's four at a time, 1024 threads for buckets of
 * more than STATE_BIG elements (one of 419 M: 36 us, with 256 threads and one load at a time 228), 256 otherwise (20000 of
 * 100: 1024 threads add 50 us). */
constexpr uint64_t STATE_BIG = 1ull << 22;
template <uint32_t NT>
__global__ __launch_bounds__(NT) void k_full_state(Tables t, Cand c, const double *__restrict__ tile_sq, double *__restrict__ l2sq)
{
    __shared__ double red[NT / 64];
    __shared__ uint32_t redz[NT / 64];
    const uint32_t b = blockIdx.x, tid = threadIdx.x, t1 = t.tile0[b + 1];
    double acc = 0.0;
    uint32_t z = 0;
#pragma unroll 4
    for (uint32_t s = t.tile0[b] + tid; s < t1; s += NT) { acc += tile_sq[s]; z += c.E[s]; }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) { acc += __shfl_xor(acc, d, 64); z += __shfl_xor(z, d, 64); }
    if ((tid & 63) == 0) { red[tid >> 6] = acc; redz[tid >> 6] = z; }
    wg_sync();
    if (tid != 0) return;
    const bool empty = t.k[b] == 0u;
    double tot = 0.0;
    uint32_t zeros = 0;
    for (uint32_t w = 0; w < NT / 64; w += 4) {
        tot += (red[w] + red[w + 1]) + (red[w + 2] + red[w + 3]);
        zeros += (redz[w] + redz[w + 1]) + (redz[w + 2] + redz[w + 3]);
    }
    l2sq[b] = tot;
    t.T[b] = empty ? NONE : 0u;
    t.need[b] = zeros;
    t.fast[b] = empty ? PATH_CAND : PATH_ZERO;
    t.sh[b] = SH0;
    t.why[b] = 0u;
    t.par[b] = empty ? make_uint4(NONE, NONE, NONE, SH1) : make_uint4(1u, 1u, 1u, SH1);
}

/* Zeros, for the dense output that few survivors are then stored into: 16 bytes per thread in the
 * streaming kernels' order (7.1 TB/s on 6.7 GB; a kilobyte per thread group further apart 5.9). */
constexpr uint32_t ZERO_T = 1024;
template <bool NT>
__global__ __launch_bounds__(ZERO_T, 8) void k_zero(float *__restrict__ dense, uint64_t n)
{
    const uint64_t i = (uint64_t)grid_tile() * (ZERO_T * 4u) + threadIdx.x * 4u;
    if (i + 4 <= n) st_out<NT>(reinterpret_cast<f4 *>(dense + i), f4{0.f, 0.f, 0.f, 0.f});
    else for (uint64_t j = i; j < n; ++j) dense[j] = 0.0f;
}

/* One payload's decoded survivors stored into a dense gradient of zeros, or (ADD) added into one that
 * is being accumulated (the receiver side of an all-gather of payloads); nothing else is touched.
 * The indices of a payload are distinct, so plain read-modify-write needs no atomics.  Bound by the
 * partly written lines; what helps is that the lines in flight lie close together: a wavefront's
 * 64 survivors are consecutive (four consecutive ones per thread: 53 us for 1.1 M survivors of 109 M
 * elements against 41).  A workgroup takes blocks of 256 survivors gridDim.x apart; the host picks the
 * grid and the direction (scatter_grid). */
template <int BITS, bool ADD, bool BACK>
__global__ __launch_bounds__(WG) void k_scatter(const uint32_t *__restrict__ idx, const void *__restrict__ val,
                                                const float *__restrict__ scales, Tables t, uint64_t K,
                                                float *__restrict__ dense)
{
    constexpr uint32_t LDS_B = 2047;
    __shared__ uint64_t sP[LDS_B + 1];
    const bool in_lds = t.B <= LDS_B;
    const uint64_t n_blk = (K + WG - 1) / WG;
    if (in_lds) {
        for (uint32_t i = threadIdx.x; i <= t.B; i += WG) sP[i] = t.P[i];
        wg_sync();
    }
    for (uint64_t q = blockIdx.x; q < n_blk; q += gridDim.x) {
        const uint64_t j = (BACK ? n_blk - 1u - q : q) * WG + threadIdx.x;
        if (j >= K) continue;
        const uint32_t li = idx[j];                       /* fetched while its bucket is searched for */
        const uint32_t b = in_lds ? find_bucket<uint64_t>(sP, t.B, j) : find_bucket<uint64_t>(t.P, t.B, j);
        const uint64_t lo = t.off[b], nb = t.off[b + 1] - lo;
        if (li >= nb) continue;                           /* invalid payload: never leave the bucket */
        float *at = dense + lo + li;
        float y = 0.0f;
        if (ADD && BACK) y = *at;                         /* few survivors: the long way first */
        const float x = decode<BITS>(reinterpret_cast<const uint8_t *>(val) + t.V[b], BITS <= 8 ? scales + t.S[b] : nullptr,
                                     j - t.P[b], t.chunk, t.chunkSh);
        if (ADD && !BACK) y = *at;
        *at = ADD ? __fadd_rn(y, x) : x;
    }
}

}  // namespace

#endif
