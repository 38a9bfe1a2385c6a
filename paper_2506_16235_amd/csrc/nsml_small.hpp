/*
 * libnsml device code, part 6: whole compress calls of small buckets, a workgroup per bucket.
 * Included by nsml_kernels.hip (one translation unit); not a public header.
 */
#ifndef NSML_SMALL_HPP
#define NSML_SMALL_HPP

namespace {

/* A bucket that fits the registers of one workgroup needs none of the passes over memory that the long
 * chain of kernels is made of, and with small buckets the chain's eight launches of 4 - 10 us each are
 * all that a call costs.  Gradient and residual are read once into registers (a wavefront holds consecutive
 * elements, four of a row per lane), the k-th key is found digit by digit with histograms in LDS, ranks
 * come from ballots, chunk maxima from LDS, and payload and residual are written once.
 * Bound by the instructions of the passes over the registers (3 us for every 4096 elements) on top of about 8 us, so only the
 * first digit is counted over all elements; the few keys that share it are listed, and the rest of the search is theirs.  Four
 * rows of loads are in flight, and a phase keeps none of the last one's masks.  60007 elements in 24 buckets, 10 %, fp16: 19.8 us
 * (25.2 with three passes and a row of loads at a time; by the chain 52); one of 32764, 1 % as 8-bit codes 31.4 (39.3), of 500 9.5 (13.2). */
constexpr uint32_t SMALL_T = 1024;
constexpr uint32_t SMALL_ROWS = 8;                                   /* rows of four elements per lane, at most */
constexpr uint32_t SMALL_MAX = SMALL_T * SMALL_ROWS * 4 - 4;         /* elements, less the ones a bucket may start before a multiple of 4 */
constexpr uint32_t SMALL_WAVES = SMALL_T / 64;
constexpr uint32_t SMALL_LIST = 4096;                                /* undecided keys that are searched in a list */
constexpr uint32_t SMALL_CHUNKS = SMALL_T * SMALL_ROWS * 4 / 8;      /* chunks have at least 8 survivors */

template <int BITS>
__global__ __launch_bounds__(SMALL_T) void k_small(const float *__restrict__ g, float *__restrict__ r, Tables t, double *__restrict__ l2sq,
                                                   uint32_t *__restrict__ idx_out, void *__restrict__ val, float *__restrict__ scales)
{
    constexpr float QMAX = BITS == 8 ? 127.0f : 7.0f;     /* (unused for 16 / 32 bits) */
    constexpr bool CODED = BITS <= 8;
    __shared__ __align__(16) uint32_t hist[NB0];
    __shared__ uint32_t cmax[CODED ? SMALL_CHUNKS : 1];   /* a chunk's largest magnitude, then its scale */
    __shared__ uint32_t code[CODED ? SMALL_T * SMALL_ROWS : SMALL_LIST];      /* first the undecided keys, then the codes */
    __shared__ uint32_t tmp[SMALL_WAVES], wg_[SMALL_WAVES], we_[SMALL_WAVES], res[3], listed;
    __shared__ double red[SMALL_WAVES];
    const uint32_t b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint64_t lo = t.off[b], hi = t.off[b + 1], base = lo & ~3ull;
    const uint32_t kb = t.k[b], chunk = t.chunk;
    uint32_t *list = code;
    if (hi == lo) {
        if (tid == 0) {
            l2sq[b] = 0.0;
            t.T[b] = NONE; t.need[b] = 0u; t.fast[b] = PATH_CAND; t.sh[b] = SH0; t.why[b] = 0u;
            t.par[b] = make_uint4(NONE, NONE, NONE, SH1);
        }
        return;
    }
    const uint32_t quads = (uint32_t)((hi - base + 3) / 4);
    const uint32_t rows = (quads + SMALL_T - 1) / SMALL_T;               /* 1 .. SMALL_ROWS, the same in every thread */
    const uint32_t q0 = wave * rows * 64 + lane;                         /* this lane's first quad */

    float x[SMALL_ROWS][4];
    uint32_t valid = 0;                                                  /* four bits per row */
    double sq = 0.0;
    constexpr uint32_t FLY = 4;                                          /* rows in flight */
#pragma unroll
    for (uint32_t u0 = 0; u0 < SMALL_ROWS; u0 += FLY) {
        f4 y[FLY], z[FLY];
#pragma unroll
        for (uint32_t u = 0; u < FLY; ++u) {
            const uint64_t gi = base + (uint64_t)(q0 + (u0 + u) * 64) * 4;
            y[u] = z[u] = f4{0.f, 0.f, 0.f, 0.f};
            if (u0 + u < rows && gi >= lo && gi + 4 <= hi) {
                y[u] = *reinterpret_cast<const f4 *>(g + gi);
                z[u] = *reinterpret_cast<const f4 *>(r + gi);
                valid |= 0xFu << (4 * (u0 + u));
            }
        }
#pragma unroll
        for (uint32_t u = 0; u < FLY; ++u) {
            const uint64_t gi = base + (uint64_t)(q0 + (u0 + u) * 64) * 4;
            if (u0 + u < rows && gi < hi && !((valid >> (4 * (u0 + u))) & 1u)) {
                /* the bucket's first and last quad may be partly another's */
                float ya[4], za[4];
                valid |= load_quad(g, gi, lo, hi, ya) << (4 * (u0 + u));
                load_quad(r, gi, lo, hi, za);
                y[u] = f4{ya[0], ya[1], ya[2], ya[3]};
                z[u] = f4{za[0], za[1], za[2], za[3]};
            }
            sq += (double)(__fmaf_rn(y[u].x, y[u].x, __fmul_rn(y[u].y, y[u].y)) + __fmaf_rn(y[u].z, y[u].z, __fmul_rn(y[u].w, y[u].w)));
#pragma unroll
            for (int j = 0; j < 4; ++j) x[u0 + u][j] = __fadd_rn(y[u][j], z[u][j]);
        }
    }
    sq = wave_sum_last(sq);
    if (lane == 63) red[wave] = sq;
    /* Keys, comparisons and masks of one phase are not kept for the next (the compiler would, and spill them). */
    auto anew = [&]() {
        asm volatile("" : "+v"(valid));
#pragma unroll
        for (uint32_t u = 0; u < SMALL_ROWS; ++u)
#pragma unroll
            for (int j = 0; j < 4; ++j) asm volatile("" : "+v"(x[u][j]));
    };

    /* The k-th largest key, a digit of 12, 12 and 7 bits at a time: the first over all elements, and the next as well as long as
     * more keys are undecided than the list holds; then those keys are listed and the remaining digits come from the list. */
    uint32_t T = 0, want = kb, psh = 31u, at = 0;        /* T: the bits from psh up */
#pragma unroll 1
    while (true) {
        const uint32_t dsh = psh == 31u ? (uint32_t)SH0 : psh == (uint32_t)SH0 ? (uint32_t)SH1 : 0u;
        const uint32_t nbin = dsh == 0u ? (uint32_t)NB2 : (uint32_t)NB0;
        for (uint32_t i = tid; i < nbin; i += SMALL_T) hist[i] = 0u;
        wg_sync();
        anew();
#pragma unroll
        for (uint32_t u = 0; u < SMALL_ROWS; ++u) {
            if (u >= rows) continue;
            uint32_t d[4], hit = 0;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint32_t key = keyof(x[u][j]);
                d[j] = (key >> dsh) & (nbin - 1u);
                if (((valid >> (4 * u + j)) & 1u) && (key >> psh) == T) hit |= 1u << j;
            }
            /* runs of equal keys (zeros): one addition for the wavefront */
            const uint32_t fd = __builtin_amdgcn_readfirstlane(d[0]);
            if (__all(hit == 0xFu && d[0] == fd && d[1] == fd && d[2] == fd && d[3] == fd)) {
                if (lane == 0) atomicAdd(&hist[fd], 256u);
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if ((hit >> j) & 1u) atomicAdd(&hist[d[j]], 1u);
            }
        }
        if (tid == 0) listed = 0u;
        wg_sync();
        (void)(dsh == 0u ? find_digit_lds<NB2>(hist, want, tmp, res) : find_digit_lds<NB0>(hist, want, tmp, res));
        T = (T << (psh == 31u ? 12u : psh - dsh)) | res[0];
        want -= res[1];
        at = res[2];
        psh = dsh;
        wg_sync();
        if (psh == 0u || at <= SMALL_LIST) break;
    }

    /* keys above T's bits per wavefront, those that share them into the list (its order does not matter; when T is complete they are counted) */
    {
        uint32_t ng = 0, ne = 0;
        anew();
#pragma unroll
        for (uint32_t u = 0; u < SMALL_ROWS; ++u) {
            if (u >= rows) continue;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint32_t key = keyof(x[u][j]);
                const bool is = ((valid >> (4 * u + j)) & 1u) && (key >> psh) == T;
                ng += (uint32_t)__popcll(__ballot((key >> psh) > T));      /* (what is not valid has key 0) */
                const uint64_t be = __ballot(is);
                if (!be) continue;
                if (psh == 0u) { ne += (uint32_t)__popcll(be); continue; }
                uint32_t p = 0;
                if (lane == 0) p = atomicAdd(&listed, (uint32_t)__popcll(be));
                p = __builtin_amdgcn_readfirstlane(p);
                p = __builtin_amdgcn_mbcnt_hi((uint32_t)(be >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)be, p));
                if (is) list[p] = (key & ((1u << psh) - 1u)) | (wave << SH0);        /* at most 19 undecided bits, then the wavefront */
            }
        }
        if (lane == 0) { wg_[wave] = ng; we_[wave] = ne; }
    }
    if (psh) {
        const uint32_t low = (1u << psh) - 1u, T0 = T;
        if (psh > (uint32_t)SH1) {
            for (uint32_t i = tid; i < (uint32_t)NB1; i += SMALL_T) hist[i] = 0u;
            wg_sync();
            for (uint32_t i = tid; i < at; i += SMALL_T) atomicAdd(&hist[(list[i] & low) >> SH1], 1u);
            wg_sync();
            (void)find_digit_lds<NB1>(hist, want, tmp, res);
            T = (T << (psh - SH1)) | res[0];
            want -= res[1];
            wg_sync();
        }
        if (tid < (uint32_t)NB2) hist[tid] = 0u;
        wg_sync();
        for (uint32_t i = tid; i < at; i += SMALL_T) {
            const uint32_t k = list[i] & low;
            if (((T0 << psh) | k) >> SH1 == T) atomicAdd(&hist[k & (NB2 - 1u)], 1u);
        }
        wg_sync();
        (void)find_digit_lds<NB2>(hist, want, tmp, res);
        T = (T << SH1) | res[0];
        want -= res[1];
        for (uint32_t i = tid; i < at; i += SMALL_T) {
            const uint32_t e = list[i], k = (T0 << psh) | (e & low);
            if (k >= T) atomicAdd(k > T ? &wg_[e >> SH0] : &we_[e >> SH0], 1u);
        }
    }
    const uint32_t e_b = want;                           /* of the keys equal to T the first so many survive */
    wg_sync();
    /* ranks: survivors before this wavefront, then row by row */
    uint32_t all;
    uint32_t g0 = scan_totals(wg_, all), e0 = scan_totals(we_, all);
    if (CODED) {
        for (uint32_t i = tid; i < (kb + chunk - 1) / chunk; i += SMALL_T) cmax[i] = 0u;
        wg_sync();
    }
    const uint64_t Pb = t.P[b];
    uint8_t *vb = reinterpret_cast<uint8_t *>(val) + t.V[b];
    uint8_t *code8 = reinterpret_cast<uint8_t *>(code);
    auto chunk_of = [&](uint32_t rank) { return t.chunkSh < 64u ? rank >> t.chunkSh : rank / chunk; };
    /* survivors of row u: which of the lane's four, the rank of its first; g_run, e_run: keys above / equal to T before the row */
    auto row_ranks = [&](uint32_t u, uint32_t &g_run, uint32_t &e_run, uint32_t &first) {
        uint32_t pg = g_run, pe = e_run, took = 0;
        bool fg[4], fe[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const bool in = (valid >> (4 * u + j)) & 1u;
            fg[j] = in && keyof(x[u][j]) > T;
            fe[j] = in && keyof(x[u][j]) == T;
            const uint64_t bg = __ballot(fg[j]), be = __ballot(fe[j]);
            pg = __builtin_amdgcn_mbcnt_hi((uint32_t)(bg >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bg, pg));
            pe = __builtin_amdgcn_mbcnt_hi((uint32_t)(be >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)be, pe));
            g_run += (uint32_t)__popcll(bg);
            e_run += (uint32_t)__popcll(be);
        }
        first = pg + min(e_b, pe);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (fg[j] || (fe[j] && pe < e_b)) took |= 1u << j;
            pe += fe[j] ? 1u : 0u;
        }
        return took;
    };
    if (CODED) {
        uint32_t g1 = g0, e1 = e0;
        anew();
#pragma unroll
        for (uint32_t u = 0; u < SMALL_ROWS; ++u) {
            if (u >= rows) continue;
            const uint32_t r0 = g1 + min(e_b, e1);
            uint32_t rank;
            const uint32_t took = row_ranks(u, g1, e1, rank);
            const uint32_t r1 = g1 + min(e_b, e1);
            if (r0 == r1) continue;
            uint32_t key[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                key[j] = (took >> j) & 1u ? keyof(x[u][j]) : 0u;
                if (key[j] > 0x7F800000u) key[j] = 0u;       /* a chunk's largest magnitude passes NaN over */
            }
            const uint32_t c0 = chunk_of(r0);
            if (c0 == chunk_of(r1 - 1)) {                /* the row lies in one chunk */
                const float m = wave_max(__uint_as_float(max(max(key[0], key[1]), max(key[2], key[3]))));
                if (lane == 0) atomicMax(&cmax[c0], __float_as_uint(m));
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if ((took >> j) & 1u) { atomicMax(&cmax[chunk_of(rank)], key[j]); ++rank; }
            }
        }
        wg_sync();
        for (uint32_t i = tid; i < (kb + chunk - 1) / chunk; i += SMALL_T) {
            const float m = __uint_as_float(cmax[i]);
            const float scale = m == 0.0f ? 0.0f : __fdiv_rn(m, QMAX);
            scales[t.S[b] + i] = scale;
            cmax[i] = __float_as_uint(scale);
        }
        if (tid == 0 && (kb & 1u)) code8[kb] = 0u;       /* what fills the last byte of an odd number of 4-bit codes */
        wg_sync();
    }
    anew();
#pragma unroll
    for (uint32_t u = 0; u < SMALL_ROWS; ++u) {
        if (u >= rows) continue;
        uint32_t rank;
        const uint32_t took = row_ranks(u, g0, e0, rank);
        const uint64_t gi = base + (uint64_t)(q0 + u * 64) * 4;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (!((took >> j) & 1u)) continue;
            const float xv = x[u][j];
            idx_out[Pb + rank] = (uint32_t)(gi - lo) + (uint32_t)j;
            if (BITS == 32) {
                reinterpret_cast<float *>(vb)[rank] = xv;
                x[u][j] = __fsub_rn(xv, xv);             /* nothing is left behind (NaN where no value was) */
            } else if (BITS == 16) {
                const __half hv = __float2half_rn(xv);
                reinterpret_cast<__half *>(vb)[rank] = hv;
                x[u][j] = __fsub_rn(xv, __half2float(hv));
            } else {
                const float scale = __uint_as_float(cmax[chunk_of(rank)]);
                /* (the product with the reciprocal gives the quotient's code away from the middle of two: see quantize_four) */
                const float y = __fmul_rn(xv, __builtin_amdgcn_rcpf(scale));
                float wq = rintf(y);
                if (!(fabsf(__fsub_rn(y, wq)) < 0.4999f)) wq = scale != 0.0f ? rintf(__fdiv_rn(xv, scale)) : 0.0f;
                const int q = (int)fminf(fmaxf(wq, -QMAX), QMAX);
                code8[rank] = (uint8_t)q;
                x[u][j] = __fsub_rn(xv, __fmul_rn((float)q, scale));
            }
            ++rank;
        }
        const uint32_t m = (valid >> (4 * u)) & 0xFu;
        if (m == 0xFu) {
            *reinterpret_cast<f4 *>(r + gi) = f4{x[u][0], x[u][1], x[u][2], x[u][3]};
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if ((m >> j) & 1u) r[gi + j] = x[u][j];
        }
    }
    if (CODED) {
        wg_sync();
        const uint32_t bytes = BITS == 8 ? kb : (kb + 1) / 2;
        for (uint32_t i = tid; i < bytes; i += SMALL_T)
            vb[i] = BITS == 8 ? code8[i] : (uint8_t)((code8[2 * i] & 0xFu) | (code8[2 * i + 1] << 4));
    }
    if (tid == 0) {
        double tot = 0.0;
        for (uint32_t w = 0; w < SMALL_WAVES; ++w) tot += red[w];
        l2sq[b] = tot;
        t.T[b] = T; t.need[b] = e_b; t.fast[b] = PATH_CAND; t.sh[b] = SH0; t.why[b] = 0u;
        t.par[b] = make_uint4(T, T, T, SH1);
    }
}

}  // namespace

#endif
