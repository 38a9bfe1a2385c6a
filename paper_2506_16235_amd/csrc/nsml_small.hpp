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
 * elements, four of a row per lane, four rows of loads in flight), payload and residual are written once.
 * Bound by the instructions of the passes over the registers and by their barriers, so where no more than a quarter is sent only two
 * such passes are made, over a sample of the elements and for the list of those that may survive; all else is
 * done with the list.  The 23185 elements of the largest of 24 buckets, 10 % as 16-bit values: 13 us a call, one call after the other, 15 - 16 in a
 * kernel trace; of them 2.6 loads, 2.4 bound, 3.2 list, 0.7 the bin of the threshold, 0.9 its key, 1.5 ranks, 0.5 payload.  Digit by digit over all
 * elements 18 a call.  With more sent, or a list that does
 * not fit, the k-th key is found digit by digit with histograms in LDS, the first digit over all elements; a phase keeps none of the last
 * one's masks.
 * us, compress, so / digit by digit: 60000 elements in 24 buckets, 10 %, 8 bits 15.5 / 24.1, 16 bits 13.1 / 17.3, 1 % 13.6 / 21.5; one
 * of 5000 11.2 / 13.5, 1000 of them 44.6 / 52.3. */
constexpr uint32_t SMALL_T = 1024;
constexpr uint32_t SMALL_ROWS = 8;                                   /* rows of four elements per lane, at most */
constexpr uint32_t SMALL_MAX = SMALL_T * SMALL_ROWS * 4 - 4;         /* elements, less the ones a bucket may start before a multiple of 4 */
constexpr uint32_t SMALL_WAVES = SMALL_T / 64;
constexpr uint32_t SMALL_LIST = 4096;                                /* undecided keys that are searched in a list */
constexpr uint32_t SMALL_CHUNKS = SMALL_T * SMALL_ROWS * 4 / 8;      /* chunks have at least 8 survivors */
constexpr uint32_t SMALL_CAND = 8192;                                /* candidates (two workgroups' LDS fits a compute unit: one starts while another ends) */
static_assert(SMALL_CHUNKS == (uint32_t)NB0, "the candidates' bins and the chunks' maxima are one array");

/* Two digits of an LDS histogram of NB0 bins at once, see find_digit_lds: res[0 .. 2] for the want-th entry, res[3] the digit of the want2-th. */
__device__ __forceinline__ void find_two_digits_lds(const uint32_t *h, uint32_t want, uint32_t want2, uint32_t *tmp, uint32_t *res)
{
    const int top = NB0 - 1 - (int)threadIdx.x * 4;
    const uint4 v = *reinterpret_cast<const uint4 *>(h + top - 3);
    const uint32_t cnt[4] = {v.w, v.z, v.y, v.x}, sum = (v.x + v.y) + (v.z + v.w);
    uint32_t total, incl = wave_incl_scan(sum);
    if ((threadIdx.x & 63u) == 63u) tmp[threadIdx.x >> 6] = incl;
    wg_sync();
    incl += scan_totals(tmp, total);
    uint32_t acc = incl - sum;
    if ((acc < want && want <= incl) || (acc < want2 && want2 <= incl)) {
#pragma unroll
        for (uint32_t i = 0; i < 4; ++i) {
            if (acc < want && want <= acc + cnt[i]) { res[0] = (uint32_t)top - i; res[1] = acc; res[2] = cnt[i]; }
            if (acc < want2 && want2 <= acc + cnt[i]) res[3] = (uint32_t)top - i;
            acc += cnt[i];
        }
    }
    wg_sync();
}

/* The digit of 256 bins that holds the want-th entry from the top, found by every wavefront for itself: no barrier.  above: entries in higher digits. */
__device__ __forceinline__ uint32_t find_digit_wave(const uint32_t *h, uint32_t want, uint32_t &above)
{
    const uint32_t lane = threadIdx.x & 63;
    const uint4 v = *reinterpret_cast<const uint4 *>(h + 252u - 4u * lane);
    const uint32_t cnt[4] = {v.w, v.z, v.y, v.x}, sum = (v.x + v.y) + (v.z + v.w), incl = wave_incl_scan(sum);
    const uint64_t here = __ballot(incl >= want);
    uint32_t acc = incl - sum, i = 0;
#pragma unroll
    for (uint32_t u = 0; u < 3; ++u) if (i == u && acc + cnt[u] < want) { acc += cnt[u]; ++i; }
    const int l = here ? (int)__builtin_ctzll(here) : 63;
    above = (uint32_t)__builtin_amdgcn_readlane((int)acc, l);
    return 255u - 4u * (uint32_t)l - (uint32_t)__builtin_amdgcn_readlane((int)i, l);
}

/* LDS of the candidates' way. */
struct SmallCand {
    __align__(16) uint32_t h[3 * 256];                   /* the last digits, 8 bits at a time */
    __align__(16) float v[SMALL_CAND];                                 /* the candidates, a wavefront's side by side in the order of its elements */
    uint16_t i[SMALL_CAND];
    uint32_t few[64], n_few, n_all;
};

/* The rest of a bucket's call from its candidates: n of them, from `first` on, this wavefront's, kb and more in all.  h1: the counts of the candidates' bins
 * ((key - low) >> s, the last one open above), `d` the bin of the k-th key, `want` of its `at` keys are wanted.  The undecided keys
 * are those of that bin: up to 64 are searched bit by bit, by every wavefront for itself. */
template <int BITS, typename CHUNK, typename RECORD>
__device__ __forceinline__ void small_candidates(SmallCand &c, uint32_t first, uint32_t n, uint32_t kb, uint32_t chunk, uint32_t low, uint32_t s, uint32_t d, uint32_t want, uint32_t at,
                                                 const Tables &t, uint32_t b, uint32_t *cmax, uint8_t *code8, uint32_t *tot,
                                                 uint32_t *__restrict__ idx_out, uint8_t *__restrict__ vb, float *__restrict__ scales, float *__restrict__ rb,
                                                 CHUNK chunk_of, RECORD record)
{
    constexpr float QMAX = BITS == 8 ? 127.0f : 7.0f;     /* (unused for 16 / 32 bits) */
    constexpr bool CODED = BITS <= 8;
    const uint32_t tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const float *cv = c.v + first;
    const uint16_t *ci = c.i + first;
    /* f(whether there is one, candidate, its number) for the wavefront's candidates, 64 at a time: the first 256 from registers */
    float v[4];
    auto fetch = [&](uint32_t q, float (&x)[4]) {
#pragma unroll
        for (uint32_t u = 0; u < 4; ++u) { const uint32_t i = q + u * 64u + lane; x[u] = i < n ? cv[i] : 0.0f; }
    };
    fetch(0u, v);
    auto rows = [&](auto f) __attribute__((always_inline)) {
#pragma unroll
        for (uint32_t u = 0; u < 4; ++u)
            if (u * 64u < n) f(u * 64u + lane < n, v[u], u * 64u + lane);
        for (uint32_t q = 256u; q < n; q += 64u) { const uint32_t i = q + lane; f(i < n, i < n ? cv[i] : 0.0f, i); }
    };
    if (CODED) *reinterpret_cast<uint4 *>(cmax + tid * 4u) = make_uint4(0u, 0u, 0u, 0u);      /* (the counts have been read) */
    const uint32_t rest_mask = (1u << s) - 1u;
    auto undecided = [&](bool in, float x, uint32_t &rest) {
        const uint32_t k = keyof(x) - low;
        rest = k & rest_mask;
        return in && min(k >> s, (uint32_t)NB0 - 1u) == d;
    };
    uint32_t T = 0;
    if (at <= 64u) {
        rows([&](bool in, float x, uint32_t) {
            uint32_t rest;
            const bool is = undecided(in, x, rest);
            const uint64_t bal = __ballot(is);
            if (!bal) return;
            uint32_t p = 0;
            if (lane == 0) p = atomicAdd(&c.n_few, (uint32_t)__popcll(bal));
            p = __builtin_amdgcn_readfirstlane(p);
            p = __builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bal, p));
            if (is && p < 64u) c.few[p] = rest;
        });
        wg_sync();
        const uint32_t y = lane < at ? c.few[lane] : 0u;
        uint64_t who = at < 64u ? (1ull << at) - 1ull : ~0ull;
        for (uint32_t bit = s; bit-- > 0u;) {
            const uint64_t ones = __ballot((y >> bit) & 1u) & who;
            const uint32_t cnt = (uint32_t)__popcll(ones);
            if (want <= cnt) { who = ones; T |= 1u << bit; }
            else { want -= cnt; who &= ~ones; }
        }
    } else {
        uint32_t *h = c.h;
        for (uint32_t rem = s; rem;) {
            const uint32_t sh = rem > 8u ? rem - 8u : 0u, mask = (1u << (rem - sh)) - 1u;
            rows([&](bool in, float x, uint32_t) {
                uint32_t rest;
                if (undecided(in, x, rest) && rest >> rem == T >> rem) add_shared(h, (rest >> sh) & mask, 1u);
            });
            wg_sync();
            uint32_t above;
            T |= find_digit_wave(h, want, above) << sh;
            want -= above;
            rem = sh;
            h += 256;
        }
    }
    T += low + (d << s);
    const uint32_t e_b = want;                           /* of the keys equal to T the first so many survive */
    uint32_t ng = 0, ne = 0;
    rows([&](bool in, float x, uint32_t) {
        ng += (uint32_t)__popcll(__ballot(in && keyof(x) > T));
        ne += (uint32_t)__popcll(__ballot(in && keyof(x) == T));
    });
    if (lane == 0) tot[wave] = ng | (ne << 16);          /* (no more than 32764 of either in all) */
    wg_sync();
    uint32_t all;
    const uint32_t before = scan_totals(tot, all);
    /* the candidate's rank, NONE: no survivor; g_run, e_run: keys above / equal to T before the row */
    auto rank_of = [&](bool in, float x, uint32_t &g_run, uint32_t &e_run) {
        const bool isg = in && keyof(x) > T, ise = in && keyof(x) == T;
        const uint64_t bg = __ballot(isg), be = __ballot(ise);
        const uint32_t pg = __builtin_amdgcn_mbcnt_hi((uint32_t)(bg >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bg, g_run));
        const uint32_t pe = __builtin_amdgcn_mbcnt_hi((uint32_t)(be >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)be, e_run));
        g_run += (uint32_t)__popcll(bg);
        e_run += (uint32_t)__popcll(be);
        return isg || (ise && pe < e_b) ? pg + min(pe, e_b) : NONE;
    };
    if (CODED) {
        uint32_t g_run = before & 0xFFFFu, e_run = before >> 16;
        rows([&](bool in, float x, uint32_t) {
            /* the chunks' largest magnitudes, which pass NaN over */
            const uint32_t rank = rank_of(in, x, g_run, e_run);
            const uint64_t who = __ballot(rank != NONE);
            if (!who) return;
            const uint32_t first = chunk_of((uint32_t)__builtin_amdgcn_readlane((int)rank, (int)__builtin_ctzll(who)));
            const uint32_t last = chunk_of((uint32_t)__builtin_amdgcn_readlane((int)rank, (int)(63 - __builtin_clzll(who))));
            const float y = rank != NONE && !(x != x) ? fabsf(x) : 0.0f;
            if (first == last) {
                const float m = wave_max(y);
                if (lane == 0) atomicMax(&cmax[first], __float_as_uint(m));
            } else if (rank != NONE) {
                atomicMax(&cmax[chunk_of(rank)], __float_as_uint(y));
            }
        });
        wg_sync();
        for (uint32_t i = tid; i < (kb + chunk - 1) / chunk; i += SMALL_T) {
            const float m = __uint_as_float(cmax[i]), sc = m == 0.0f ? 0.0f : __fdiv_rn(m, QMAX);
            scales[t.S[b] + i] = sc;
            cmax[i] = __float_as_uint(sc);
        }
        if (BITS == 4 && tid == 0 && (kb & 1u)) code8[kb] = 0u;      /* what fills the last byte of an odd number of 4-bit codes */
    }
    __builtin_amdgcn_s_waitcnt(0);                       /* the elements that were written back come before the errors */
    wg_sync();
    uint32_t g_run = before & 0xFFFFu, e_run = before >> 16;
    rows([&](bool in, float xv, uint32_t i) {
        const uint32_t rank = rank_of(in, xv, g_run, e_run);
        if (rank == NONE) return;
        const uint32_t li = ci[i];
        float left;
        idx_out[rank] = li;
        if (BITS == 32) {
            reinterpret_cast<float *>(vb)[rank] = xv;
            left = __fsub_rn(xv, xv);                    /* nothing is left behind (NaN where no value was) */
        } else if (BITS == 16) {
            const __half hv = __float2half_rn(xv);
            reinterpret_cast<__half *>(vb)[rank] = hv;
            left = __fsub_rn(xv, __half2float(hv));
        } else {
            const float scale = __uint_as_float(cmax[chunk_of(rank)]);
            /* (the product with the reciprocal gives the quotient's code away from the middle of two: see quantize_four) */
            const float y = __fmul_rn(xv, __builtin_amdgcn_rcpf(scale));
            float wq = rintf(y);
            if (!(fabsf(__fsub_rn(y, wq)) < 0.4999f)) wq = scale != 0.0f ? rintf(__fdiv_rn(xv, scale)) : 0.0f;
            const int code = (int)fminf(fmaxf(wq, -QMAX), QMAX);
            if (BITS == 8) vb[rank] = (uint8_t)code;
            else code8[rank] = (uint8_t)code;
            left = __fsub_rn(xv, __fmul_rn((float)code, scale));
        }
        rb[li] = left;
    });
    if (BITS == 4) {
        wg_sync();
        for (uint32_t i = tid; i < (kb + 1) / 2; i += SMALL_T) vb[i] = (uint8_t)((code8[2 * i] & 0xFu) | (code8[2 * i + 1] << 4));
    }
    if (tid == 0) record(T, e_b);
}

template <int BITS>
__global__ __launch_bounds__(SMALL_T) void k_small(const float *__restrict__ g, float *__restrict__ r, Tables t, double *__restrict__ l2sq,
                                                   uint32_t *__restrict__ idx_out, void *__restrict__ val, float *__restrict__ scales)
{
    constexpr float QMAX = BITS == 8 ? 127.0f : 7.0f;     /* (unused for 16 / 32 bits) */
    constexpr bool CODED = BITS <= 8;
    __shared__ __align__(16) uint32_t cmax[SMALL_CHUNKS];       /* a chunk's largest magnitude, then its scale; before that the counts of digits and bins */
    __shared__ uint8_t code4[BITS == 4 ? SMALL_CAND / 2 + 4 : 4];      /* the candidates' way: codes of 4 bits */
    uint32_t *hist = cmax;
    __shared__ uint32_t tmp[SMALL_WAVES], wg_[SMALL_WAVES], we_[SMALL_WAVES], res[4], listed;
    __shared__ SmallCand sc;
    uint32_t *draw = reinterpret_cast<uint32_t *>(sc.v);      /* the sample's digits */
    uint32_t *code = draw;      /* first the undecided keys, then the codes */
    static_assert(sizeof sc.v >= SMALL_T * SMALL_ROWS * 4, "a byte per element");
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

    const uint32_t nb = (uint32_t)(hi - lo);
    /* the candidates' way where they may fit (what it counts in is cleared while the loads are on their way) */
    const bool some = kb <= nb / 4u && kb <= SMALL_CAND / 2u;
    const bool sampled = nb > SMALL_T * 4u;
    if (some) {
        *reinterpret_cast<uint4 *>(hist + tid * 4u) = *reinterpret_cast<uint4 *>(draw + tid * 4u) = make_uint4(0u, 0u, 0u, 0u);
        if (tid < 192u) *reinterpret_cast<uint4 *>(sc.h + tid * 4u) = make_uint4(0u, 0u, 0u, 0u);
        if (tid == 0) sc.n_few = sc.n_all = 0u;
    }
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

    const uint64_t Pb = t.P[b];
    uint8_t *vb = reinterpret_cast<uint8_t *>(val) + t.V[b];
    uint8_t *code8 = reinterpret_cast<uint8_t *>(code);
    auto chunk_of = [&](uint32_t rank) { return t.chunkSh < 64u ? rank >> t.chunkSh : rank / chunk; };
    auto record = [&](uint32_t T, uint32_t e_b) {
        double tot = 0.0;
        for (uint32_t w = 0; w < SMALL_WAVES; ++w) tot += red[w];
        l2sq[b] = tot;
        t.T[b] = T; t.need[b] = e_b; t.fast[b] = PATH_CAND; t.sh[b] = SH0; t.why[b] = 0u;
        t.par[b] = make_uint4(T, T, T, SH1);
    };

    /* The candidates' way: a lower bound of the k-th key from every fourth element (the first of each lane's four, so that runs of large values
     * weigh what they do); the elements from there up go into LDS, a wavefront's side by side, and are counted in bins that are fine where the
     * k-th key must lie; the rest is theirs.  A bound that leaves too many or too few leads to the way below. */
    bool found = false;                                  /* the k-th key's digit, or all of it, without the digits of all elements */
    uint32_t zeros = 0, crowded = NONE;                  /* crowded: a digit with more keys than the list holds, which seems to be the k-th key's */
    if (some) {
        uint32_t low = 0, s = SH0;                       /* keys from low up, bins of 2^s keys */
        bool fits = true;
        wg_sync();
        if (sampled) {
#pragma unroll
            for (uint32_t u = 0; u < SMALL_ROWS; ++u) {
                if (u >= rows) continue;
                const bool in = (valid >> (4 * u)) & 1u;
                const uint32_t d = keyof(x[u][0]) >> SH0, fd = __builtin_amdgcn_readfirstlane(d);
                if (__all(in && d == fd)) {
                    if (lane == 0) atomicAdd(&draw[fd], 64u);
                } else if (in) {
                    atomicAdd(&draw[d], 1u);
                }
            }
            wg_sync();
            const uint32_t drawn = quads - ((lo & 3ull) ? 1u : 0u);      /* quads whose first element is the bucket's */
            const float ks = (float)kb * ((float)drawn / (float)nb), dev = 4.0f * sqrtf(ks) + 4.0f, up = floorf(ks - dev);
            const uint32_t want = (uint32_t)ceilf(ks + dev);
            fits = want <= drawn;
            if (fits) {
                find_two_digits_lds(draw, want, up < 1.0f ? 1u : (uint32_t)up, tmp, res);
                low = max(res[0] << SH0, 1u);            /* (zeros are no candidates: see below) */
                fits = (res[1] + (low > 1u ? res[2] : 0u)) * 4u <= SMALL_CAND * 7u / 8u;
                if (!fits && ks > (float)res[1]) crowded = res[0];
                /* two digits above the one that the k-th key will not exceed */
                s = (uint32_t)SH1;
                while (s < (uint32_t)SH0 && ((res[3] - res[0] + 3u) << SH0) > ((uint32_t)NB0 << s)) ++s;
            }
        }
        if (fits) {
            auto bin_of = [&](uint32_t key) { return min((key - low) >> s, (uint32_t)NB0 - 1u); };
            auto flags = [&](uint32_t u, uint64_t (&bal)[4]) {
                const uint32_t m = (valid >> (4 * u)) & 0xFu;
                if (__ballot(m == 0xFu) == ~0ull) {
#pragma unroll
                    for (int j = 0; j < 4; ++j) bal[j] = __ballot(keyof(x[u][j]) >= low);
                } else {
#pragma unroll
                    for (int j = 0; j < 4; ++j) bal[j] = __ballot(((m >> j) & 1u) && keyof(x[u][j]) >= low);
                }
            };
            /* a wavefront of up to 512 elements has a part for all of them, more are counted first */
            static_assert(SMALL_CAND / SMALL_WAVES >= 512u, "two rows");
            const bool counted = rows > 2u;
            uint32_t n = 0, first = wave * (SMALL_CAND / SMALL_WAVES), room = 512u, n_all = 0;
            if (counted) {
                anew();
#pragma unroll
                for (uint32_t u = 0; u < SMALL_ROWS; ++u) {
                    if (u >= rows) continue;
                    uint64_t bal[4];
                    flags(u, bal);
#pragma unroll
                    for (int j = 0; j < 4; ++j) n += (uint32_t)__popcll(bal[j]);
                }
                if (lane == 0) tmp[wave] = n;
                wg_sync();
                first = scan_totals(tmp, n_all);
                room = first + n <= SMALL_CAND ? n : 0u;
            }
            float *cv = sc.v + first;
            uint16_t *ci = sc.i + first;
            uint32_t put = 0;
            anew();
#pragma unroll
            for (uint32_t u = 0; u < SMALL_ROWS; ++u) {
                if (u >= rows) continue;
                const uint64_t gi = base + (uint64_t)(q0 + u * 64) * 4;
                const uint32_t m = (valid >> (4 * u)) & 0xFu;
                uint64_t bal[4];
                uint32_t at = put;
                flags(u, bal);
                if (bal[0] | bal[1] | bal[2] | bal[3]) {
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        at = __builtin_amdgcn_mbcnt_hi((uint32_t)(bal[j] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bal[j], at));
                        put += (uint32_t)__popcll(bal[j]);
                    }
                    if (put <= room) {                   /* (uniform) */
#pragma unroll
                        for (int j = 0; j < 4; ++j)
                            if ((bal[j] >> lane) & 1ull) {
                                cv[at] = x[u][j];
                                ci[at] = (uint16_t)((uint32_t)(gi - lo) + (uint32_t)j);
                                ++at;
                            }
                    }
                }
                /* what is not sent is left as it is; the survivors' errors come after */
                if (m == 0xFu) {
                    *reinterpret_cast<f4 *>(r + gi) = f4{x[u][0], x[u][1], x[u][2], x[u][3]};
                } else {
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        if ((m >> j) & 1u) r[gi + j] = x[u][j];
                }
            }
            put = __builtin_amdgcn_readfirstlane(put);       /* (its lanes read what others of it wrote) */
            if (!counted) {
                n = put;
                if (lane == 0 && n) atomicAdd(&sc.n_all, n);
            }
            if (n <= room)
                for (uint32_t i = lane; i < n; i += 64u) atomicAdd(&hist[bin_of(keyof(cv[i]))], 1u);
            wg_sync();
            if (!counted) n_all = sc.n_all;
            if (n_all <= SMALL_CAND && find_digit_lds<NB0>(hist, kb, tmp, res)) {         /* the same in every thread */
                if (counted) {
                    /* from here on as many for each wavefront: those of a run would be one wavefront's chain (20 buckets of 20 thousand elements, nine
                     * rows of 768 in ten zero, 8 bits: at 0.15 27.7 us, so 22.9, digit by digit 25.3; normal values 18.4, so 17.9) */
                    const uint32_t share = (n_all + SMALL_WAVES - 1u) / SMALL_WAVES;
                    first = min(wave * share, n_all);
                    n = min(share, n_all - first);
                }
                if (res[0] == (uint32_t)NB0 - 1u && s < (uint32_t)SH0) {
                    /* above all that was expected: whole digits */
                    s = SH0;
                    wg_sync();
                    *reinterpret_cast<uint4 *>(hist + tid * 4u) = make_uint4(0u, 0u, 0u, 0u);
                    wg_sync();
                    for (uint32_t i = lane; i < n; i += 64u) atomicAdd(&hist[bin_of(keyof(sc.v[first + i]))], 1u);
                    wg_sync();
                    (void)find_digit_lds<NB0>(hist, kb, tmp, res);
                }
                small_candidates<BITS>(sc, first, n, kb, chunk, low, s, res[0], kb - res[1], res[2], t, b, cmax, code4, wg_, idx_out + Pb, vb, scales, r + lo, chunk_of, record);
                return;
            }
            found = low == 1u && n_all < kb;             /* fewer values than survivors: the first zeros survive as well */
            zeros = kb - n_all;
            wg_sync();                                   /* LDS is written again */
        }
    }

    /* The k-th largest key, a digit of 12, 12 and 7 bits at a time: the first over all elements, and the next as well as long as
     * more keys are undecided than the list holds; then those keys are listed and the remaining digits come from the list. */
    uint32_t T = 0, want = kb, psh = 31u, at = 0;        /* T: the bits from psh up */
    if (found) { want = zeros; psh = 0u; }
    if (crowded != NONE) {
        /* The first digit without a histogram, in which equal digits wait for each other (60 thousand elements in 24 buckets, 1 % as 8-bit codes: of two
         * magnitudes and zero 49.9 us, so 37.9, with no sample taken 45.3; of one magnitude 24.2, 22.8, 22.6). */
        uint32_t ng = 0, ne = 0, all;
        anew();
#pragma unroll
        for (uint32_t u = 0; u < SMALL_ROWS; ++u) {
            if (u >= rows) continue;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint32_t d = keyof(x[u][j]) >> SH0;
                ng += (uint32_t)__popcll(__ballot(d > crowded));           /* (what is not valid has key 0) */
                ne += (uint32_t)__popcll(__ballot(((valid >> (4 * u + j)) & 1u) && d == crowded));
            }
        }
        if (lane == 0) tmp[wave] = ng | (ne << 16);      /* (no more than 32764 of either in all) */
        if (tid == 0) listed = 0u;
        wg_sync();
        (void)scan_totals(tmp, all);
        if ((all & 0xFFFFu) < kb && kb <= (all & 0xFFFFu) + (all >> 16)) { T = crowded; want = kb - (all & 0xFFFFu); at = all >> 16; psh = SH0; found = at <= SMALL_LIST; }
    }
#pragma unroll 1
    while (!found) {
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
    if (tid == 0) record(T, e_b);
}

}  // namespace

#endif
