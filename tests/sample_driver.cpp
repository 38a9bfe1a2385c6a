/*
 * k_presample on the CPU against a plain histogram of the elements it is to sample: what it leaves for the streaming
 * pass, and, of buckets that are sampled whole, the digit and the count the dense passes start from.
 */
#include "simt.hpp"

#include "nsml.h"

#include "nsml_device_common.hpp"
#include "nsml_select.hpp"

struct Layout {
    std::vector<uint64_t> off;
    std::vector<uint32_t> tile0, k, T, need, margin, kw, pmask;
    std::vector<uint64_t> P, V, S, C;
    std::vector<uint4> par;
    uint32_t nhard[4];
    Tables t;
    explicit Layout(const std::vector<uint64_t> &off_) : off(off_)
    {
        const size_t B = off.size() - 1;
        tile0.assign(B + 1, 0);
        for (size_t b = 0; b < B; ++b) {
            const uint64_t lo = off[b] & ~3ull;
            tile0[b + 1] = tile0[b] + (uint32_t)(off[b + 1] > off[b] ? (off[b + 1] - lo + TILE - 1) / TILE : 0);
        }
        for (auto *v : {&k, &T, &need, &margin, &kw}) v->assign(B, 0);
        for (auto *v : {&P, &V, &S, &C}) v->assign(B + 1, 0);
        par.assign(B, uint4{0, 0, 0, 0});
        pmask.assign((size_t)tile0[B] * (TILE / 32), 0u);
        memset(&t, 0, sizeof t);
        t.off = off.data(); t.tile0 = tile0.data(); t.k = k.data(); t.kw = kw.data(); t.T = T.data(); t.need = need.data();
        t.margin = margin.data(); t.par = par.data(); t.P = P.data(); t.V = V.data(); t.S = S.data(); t.C = C.data();
        t.nhard = nhard; t.B = (uint32_t)B; t.n_tiles = tile0[B]; t.chunk = 256; t.chunkSh = 8;
    }
};

/* predict_bucket on counts made elsewhere */
static uint32_t digit_up, digit_dn;       /* of the band it tried last */
static void from_counts(const Tables &t, uint32_t b, uint64_t nb, uint32_t k, double pop, bool exact, uint32_t wide, const uint32_t *counts)
{
    static uint32_t tmp[PRE_T / 64], res[10];
    DigitWalk1024 w;
    w.load(counts, tmp);
    predict_bucket(t, b, nb, k, pop, exact, wide, w, res);
    digit_up = res[3]; digit_dn = res[6];
}

static uint64_t rng_state = 88172645463325252ull;
static uint32_t rnd() { rng_state ^= rng_state << 13; rng_state ^= rng_state >> 7; rng_state ^= rng_state << 17; return (uint32_t)(rng_state >> 20); }
static float uniform() { return (float)(rnd() & 0xFFFFFF) / 16777216.0f; }

static int failures, checked, whole, handed, again;

static void check(uint64_t lead, uint64_t nb, int values, uint32_t tail, double ratio, bool pruned)
{
    const std::vector<uint64_t> off = {0, lead, lead + nb};
    Layout a(off), w(off);
    const uint64_t lo = lead, n = lead + nb, a0 = lo & ~3ull;
    std::vector<float> gs(n + 8), rs(n + 8, 0.0f);
    /* values: 0 one magnitude, 1 zeros, 2 continuous, 3 two magnitudes in turn by run of 16, 4 two in five of one magnitude above the others; the last `tail` are larger */
    for (uint64_t i = 0; i < n; ++i) {
        float v = values == 0 ? 1e-3f : values == 1 ? 0.0f : values == 2 ? (uniform() - 0.5f) * 1e-3f : values == 3 ? ((i / 16) % 3 ? 1e-3f : 3e-3f)
                : i % 5 < 2 ? 1e-3f : uniform() * 1e-3f;
        if (i + tail >= n) v = 2.0f * 1e-3f;
        gs[i] = (rnd() & 1) ? v : -v;
    }
    if (pruned) {
        a.t.pmask = w.t.pmask = a.pmask.data();
        for (auto &x : a.pmask) x = values == 1 ? 0u : rnd() & rnd() & rnd();
    }
    const uint32_t b = 1;
    const uint32_t k = (uint32_t)survivors_dev(ratio, nb);
    double pop = (double)nb;
    if (pruned) pop = (double)kept_dev(ratio, nb);
    const bool all = lead < 262144 && nb < 262144;       /* no bucket is too large to be sampled whole */
    simt::run(PRE_T, dim3(b), dim3(2), [&] { k_presample(gs.data(), rs.data(), a.t, ratio, 8, all, 0, nullptr); });
    /* a small sample, and where that leaves nothing to stage all of the bucket, or a larger one */
    std::vector<uint32_t> h;
    bool exact = false;
    for (uint64_t stride = pre_stride(nb), again_at = all ? 1u : std::max<uint64_t>(nb < 262144 ? 1u : 64u, nb / 32768);; stride = again_at) {
        const uint64_t run_elems = SAMPLE_RUN * stride;
        h.assign(NB0, 0);
        for (uint64_t i = lo; i < n; ++i) {
            const uint64_t rel = i - a0;
            const bool out = pruned && (a.pmask[(size_t)a.tile0[b] * (TILE / 32) + rel / 32] >> (rel % 32)) & 1u;
            if (rel % run_elems < SAMPLE_RUN && !out) ++h[keyof(gs[i] + rs[i]) >> SH0];
        }
        exact = stride == 1u;
        simt::run(PRE_T, dim3(b), dim3(2), [&] {
            from_counts(w.t, b, nb, k, pop, exact, nb < SAMPLE_ALL_BELOW && (uint64_t)k * 8u <= nb ? 2u : 1u, h.data());
        });
        if (w.par[b].x != NONE || stride <= again_at || (!all && digit_up == digit_dn)) break;
        ++again;
    }
    bool ok = memcmp(&a.par[b], &w.par[b], sizeof(uint4)) == 0 && a.T[b] == w.T[b] && a.need[b] == w.need[b];
    const bool hands_over = exact && a.par[b].x == NONE && a.par[b].w == (uint32_t)SH0;
    if (hands_over) {
        /* exactly the elements above that digit are settled */
        uint32_t above = 0;
        for (uint32_t d = a.T[b] + 1; d < (uint32_t)NB0; ++d) above += h[d];
        ok = ok && a.T[b] < (uint32_t)NB0 && above < k && above + h[a.T[b]] >= k && a.need[b] == k - above;
    }
    ++checked; whole += exact; handed += hands_over;
    if (!ok) {
        ++failures;
        printf("lead %llu n %llu values %d tail %u ratio %g pruned %d: L %x H %x W %x s %u T %u need %u, by a plain histogram L %x H %x W %x s %u T %u need %u\n",
               (unsigned long long)lead, (unsigned long long)nb, values, tail, ratio, pruned, a.par[b].x, a.par[b].y, a.par[b].z, a.par[b].w, a.T[b], a.need[b],
               w.par[b].x, w.par[b].y, w.par[b].z, w.par[b].w, w.T[b], w.need[b]);
    }
}

int main()
{
    const double ratios[] = {0.3, 0.1, 0.5, 0.2};
    int turn = 0;
    /* whole runs: every number of them in the last turn of a wavefront, on a multiple of 4 and beside one */
    for (uint32_t j = 26; j <= 1023; j += (j % 16) ? 15 : 16)
        for (int values = 0; values < 4; ++values, ++turn)
            check(turn % 5 ? 40000 : 40001, 16ull * j, values, values == 2 ? 0 : 16u * (1 + turn % (j % 16 ? j % 16 : 16)), ratios[turn % 4], turn % 7 == 0);
    /* the last quad short, the first one another's, buckets of which a part is sampled */
    for (uint64_t nb : {8207ull, 8208ull, 8209ull, 7840ull, 4112ull, 16383ull, 16384ull, 16400ull, 24592ull, 40016ull, 70000ull, 262143ull, 262144ull, 600000ull})
        for (int values = 0; values < 4; ++values)
            for (uint64_t lead : {40000ull, 40003ull}) check(lead, nb, values, 16, ratios[turn++ % 4], false);
    for (uint64_t nb : {8208ull, 40016ull, 70000ull, 200000ull})
        for (int values = 0; values < 5; ++values) check(300000, nb, values, 16, ratios[turn++ % 4], values == 3);
    /* set-up beside the sampling: the tables of two buckets and the chunks of both */
    {
        Layout a({0, 40001, 48209});
        std::vector<uint32_t> map(400, NONE);
        const uint64_t n_chunks = (survivors_dev(0.3, 40001) + 255) / 256 + (survivors_dev(0.3, 8208) + 255) / 256;
        for (uint32_t wg = 0; wg < 2; ++wg)
            simt::run(PRE_T, dim3(2 + wg), dim3(4), [&] { k_presample(nullptr, nullptr, a.t, 0.3, 8, true, n_chunks, map.data()); });
        const uint64_t k0 = survivors_dev(0.3, 40001), c0 = (k0 + 255) / 256;
        bool ok = a.k[0] == k0 && a.k[1] == survivors_dev(0.3, 8208) && a.P[2] == a.k[0] + a.k[1] && a.C[1] == c0 && a.C[2] == n_chunks;
        for (uint64_t c = 0; c < n_chunks; ++c) ok = ok && map[c] == (c >= c0);
        if (!ok) { ++failures; printf("tables or chunk map\n"); }
    }
    printf("checked %d, whole %d, handed to the dense passes %d, sampled again %d, failures %d\n", checked, whole, handed, again, failures);
    return failures ? 1 : handed > 40 && again > 8 ? 0 : 2;
}
