/*
 * The dense passes on the CPU (a team of one workgroup) and the coding behind them, from leading bits of the threshold that
 * are right, and from numbers of wanted keys that are not: those have to be noticed before anything is written for
 * the bucket, since the coding stores to where the index list says.  Then beside empty buckets.
 */
#include "simt.hpp"

#include "nsml.h"

#include "nsml_device_common.hpp"
#include "nsml_select.hpp"
#include "nsml_prune.hpp"
#include "nsml_codec.hpp"
#include "nsml_tail.hpp"

static int failures;
static uint64_t rng_state = 88172645463325252ull;
static uint32_t rnd() { rng_state ^= rng_state << 13; rng_state ^= rng_state >> 7; rng_state ^= rng_state << 17; return (uint32_t)(rng_state >> 20); }

/* Two buckets, the second on the dense passes with `wrong` added to the number of keys it is to find. */
template <bool BIG>
static void check(uint64_t lead, uint64_t nb, double ratio, uint32_t chunk, int wrong, bool weights)
{
    const std::vector<uint64_t> off = {0, lead, lead + nb};
    const uint64_t n = lead + nb;
    constexpr uint32_t GUARD = 64;
    std::vector<float> r(n + 8 + GUARD, 7.0f);
    for (uint64_t i = 0; i < n; ++i) r[i] = (rnd() & 1 ? 1.0f : -1.0f) * (i + 48 < n ? 1e-3f + (i % 5 ? 0.0f : 1e-9f * (float)(rnd() % 64)) : 2e-3f);
    const std::vector<float> before = r;
    std::vector<uint32_t> tile0 = {0, 0, 0}, tile_b;
    for (uint32_t b = 0; b < 2; ++b) {
        tile0[b + 1] = tile0[b] + (uint32_t)((off[b + 1] - (off[b] & ~3ull) + TILE - 1) / TILE);
        tile_b.resize(tile0[b + 1], b);
    }
    const uint32_t nt = tile0[2];
    uint32_t k[2], T[2] = {0, 0}, need[2] = {0, 0}, fast[2] = {PATH_CAND, PATH_DENSE}, sh[2] = {SH0, SH0}, margin[2] = {}, why[2] = {}, ovf[2] = {}, ftile0[3] = {};
    uint32_t nhard[4] = {1, 0, 1, 0}, err = 0;
    uint64_t P[3] = {}, V[3] = {}, S[3] = {}, C[3] = {};
    for (uint32_t b = 0; b < 2; ++b) {
        k[b] = (uint32_t)survivors_dev(ratio, off[b + 1] - off[b]);
        P[b + 1] = P[b] + k[b]; V[b + 1] = V[b] + k[b]; S[b + 1] = C[b + 1] = C[b] + (k[b] + chunk - 1) / chunk;
    }
    std::vector<uint32_t> chunk_b(C[2]), chunk_seg(C[2], 0u), G(nt), E(nt), cnt(nt), pmask((size_t)nt * (TILE / 32), 0u);
    for (uint64_t c = 0; c < C[2]; ++c) chunk_b[c] = c >= C[1];
    /* the digit of the k-th key, and how many of it are wanted */
    std::vector<uint32_t> h(NB0, 0);
    for (uint64_t i = lead; i < n; ++i) ++h[keyof(r[i]) >> SH0];
    uint32_t above = 0, d = NB0 - 1;
    while (above + h[d] < k[1]) above += h[d--];
    T[1] = d; need[1] = (uint32_t)((int)(k[1] - above) + wrong);
    Tables t = {};
    t.off = off.data(); t.tile0 = tile0.data(); t.tile_b = tile_b.data(); t.k = k; t.P = P; t.V = V; t.S = S; t.C = C; t.T = T; t.need = need; t.fast = fast;
    t.sh = sh; t.margin = margin; t.why = why; t.ovf = ovf; t.ftile0 = ftile0; t.nhard = nhard; t.B = 2; t.n_tiles = nt; t.chunk = chunk; t.chunkSh = NONE;
    t.dencTiles = 2;
    Cand c = {nullptr, nullptr, cnt.data(), G.data(), E.data()};
    std::vector<uint32_t> f0(2 * NB0, 0), f1(2 * NB1, 0), f2(2 * NB2, 0), idx(P[2] + GUARD, (uint32_t)nb + 16u);      /* (an unwritten place points behind the bucket) */
    std::vector<float> v(P[2] + GUARD, 5.0f), scales(C[2] + GUARD, 5.0f);
    std::vector<int8_t> val(V[2] + GUARD, 99);
    if (weights) {
        simt::run(WG, dim3(0), dim3(1), [&] { k_whard(r.data(), t, c, f0.data(), f1.data(), f2.data(), pmask.data(), &err); });
        uint64_t gone = 0;
        for (uint64_t i = 0; i < nb; ++i) {
            const uint64_t at = i + (lead & 3ull);
            gone += (pmask[(size_t)tile0[1] * (TILE / 32) + at / 32] >> (at % 32)) & 1u;
        }
        if ((err != 0) != (wrong != 0) || (!wrong && gone != nb - k[1])) { ++failures; printf("weights: n %llu wrong %d: flag %u, %llu pruned\n", (unsigned long long)nb, wrong, err, (unsigned long long)gone); }
        return;
    }
    simt::run(HTH, dim3(0), dim3(1), [&] {
        k_hard<8, BIG>(r.data(), t, c, f0.data(), f1.data(), f2.data(), idx.data(), v.data(), val.data(), scales.data(), &err, chunk <= DENC_MAX_CHUNK, 1);
    });
    const uint32_t per = chunk <= QUANT_WAVE_CHUNK ? (WG / 64) * QUANT_PER_WAVE : 1u, grid = (uint32_t)((C[2] + per - 1) / per);
    for (uint32_t b = 0; b < grid; ++b)
        simt::run(WG, dim3(b), dim3(grid), [&] {
            k_quant<8>(v.data(), idx.data(), t, c, r.data(), val.data(), scales.data(), chunk_b.data(), chunk_seg.data(), C[2], chunk <= DENC_MAX_CHUNK);
        });
    /* what is right: the k largest, equal ones by the lower place; codes of each chunk; the error left behind */
    std::vector<float> rest = before;
    std::vector<uint32_t> want(P[2] + GUARD, (uint32_t)nb + 16u);
    std::vector<int8_t> codes(V[2] + GUARD, 99);
    std::vector<float> sc(C[2] + GUARD, 5.0f);
    if (!wrong) {
        std::vector<uint32_t> order(nb);
        for (uint32_t i = 0; i < nb; ++i) order[i] = i;
        std::stable_sort(order.begin(), order.end(), [&](uint32_t x, uint32_t y) { return keyof(before[lead + x]) > keyof(before[lead + y]); });
        order.resize(k[1]);
        std::sort(order.begin(), order.end());
        for (uint32_t j0 = 0; j0 < k[1]; j0 += chunk) {
            const uint32_t j1 = std::min(k[1], j0 + chunk);
            float m = 0.0f;
            for (uint32_t j = j0; j < j1; ++j) m = fmaxf(m, fabsf(before[lead + order[j]]));
            const float s = m / 127.0f;
            sc[S[1] + j0 / chunk] = s;
            for (uint32_t j = j0; j < j1; ++j) {
                const float x = before[lead + order[j]], q = fminf(fmaxf(rintf(x / s), -127.0f), 127.0f);
                want[P[1] + j] = order[j]; codes[V[1] + j] = (int8_t)q; rest[lead + order[j]] = x - q * s;
            }
        }
    }
    const bool same = r == rest && idx == want && val == codes && scales == sc;
    if ((err != 0) != (wrong != 0) || !same) {
        ++failures;
        printf("lead %llu n %llu ratio %g chunk %u wrong %d: flag %u, outputs %s\n", (unsigned long long)lead, (unsigned long long)nb, ratio, chunk, wrong, err,
               same ? "as they should be" : r != rest ? "differ, the residual too" : "differ");
    }
}

/* Whole values by the dense passes beside empty buckets, before and behind, whose words hold what another layout left there (a dense
 * bucket's): other workgroups of the same launch write them, in no order with the team, so nothing may be taken from them. */
static void check_empty(uint32_t stale_need, uint32_t stale_sh)
{
    constexpr uint32_t B = 4, GUARD = 64;
    const uint64_t nb = 9001;
    const std::vector<uint64_t> off = {0, 0, nb, nb, nb};
    std::vector<float> r(nb + 8 + GUARD, 7.0f);
    for (uint64_t i = 0; i < nb; ++i) r[i] = (rnd() & 1 ? 1.0f : -1.0f) * (1e-3f + (i % 5 ? 0.0f : 1e-9f * (float)(rnd() % 64)));
    const std::vector<float> before = r;
    const uint32_t nt = (uint32_t)((nb + TILE - 1) / TILE), kb = (uint32_t)survivors_dev(0.3, nb);
    std::vector<uint32_t> tile0 = {0, 0, nt, nt, nt}, tile_b(nt, 1u), G(nt), E(nt), cnt(nt);
    std::vector<uint4> desc(nt);
    for (uint32_t i = 0; i < nt; ++i) desc[i] = make_uint4(i * (uint32_t)TILE, 0u, 1u, std::min<uint32_t>(TILE, (uint32_t)nb - i * TILE) << 16);
    uint32_t k[B] = {0, kb, 0, 0}, T[B] = {5, 0, 5, 5}, need[B] = {stale_need, kb, stale_need, stale_need}, fast[B] = {}, sh[B] = {stale_sh, SH_NONE, stale_sh, stale_sh};
    uint32_t margin[B] = {}, why[B] = {}, ovf[B] = {}, ftile0[B + 1] = {}, nhard[4] = {1, 0, 1, 1}, err = 0;
    uint64_t P[B + 1] = {0, 0, kb, kb, kb}, V[B + 1] = {0, 0, 4 * kb, 4 * kb, 4 * kb}, S[B + 1] = {}, C[B + 1] = {};
    Tables t = {};
    t.off = off.data(); t.tile0 = tile0.data(); t.tile_b = tile_b.data(); t.desc = desc.data(); t.k = k; t.P = P; t.V = V; t.S = S; t.C = C; t.T = T; t.need = need;
    t.fast = fast; t.sh = sh; t.margin = margin; t.why = why; t.ovf = ovf; t.ftile0 = ftile0; t.nhard = nhard; t.B = B; t.n_tiles = nt; t.chunk = 2048; t.chunkSh = 11;
    Cand c = {nullptr, nullptr, cnt.data(), G.data(), E.data()};
    std::vector<uint32_t> f0(B * NB0, 0), f1(B * NB1, 0), f2(B * NB2, 0), idx(kb + GUARD, 77u), pool(2 * TILE);
    std::vector<float> val(kb + GUARD, 5.0f);
    simt::run(WG, dim3(0), dim3(1), [&] { band_dense_buckets<32>(r.data(), t, c, f0.data(), f1.data(), f2.data(), idx.data(), val.data(), &err, pool.data(), 0, 1); });
    std::vector<uint32_t> order(nb), want(kb + GUARD, 77u);
    std::vector<float> values(kb + GUARD, 5.0f), rest = before;
    for (uint32_t i = 0; i < nb; ++i) order[i] = i;
    std::stable_sort(order.begin(), order.end(), [&](uint32_t x, uint32_t y) { return keyof(before[x]) > keyof(before[y]); });
    order.resize(kb);
    std::sort(order.begin(), order.end());
    for (uint32_t j = 0; j < kb; ++j) { want[j] = order[j]; values[j] = before[order[j]]; rest[order[j]] = 0.0f; }
    const bool same = r == rest && idx == want && val == values;
    if (err || !same) { ++failures; printf("empty buckets, left there: need %u sh %u: flag %u, outputs %s\n", stale_need, stale_sh, err, same ? "as they should be" : "differ"); }
}

int main()
{
    setvbuf(stdout, nullptr, _IONBF, 0);
    for (int wrong : {0, -240, -1, 1, 5000})
        for (uint64_t nb : {4112ull, 8208ull, 9001ull}) {
            check<false>(5000, nb, 0.3, 256, wrong, false);
            check<true>(5001, nb, 0.3, 264, wrong, false);
            check<true>(5002, nb, 0.5, 4096, wrong, false);
            check<false>(5003, nb, 0.6, 256, wrong, true);
        }
    for (uint32_t need : {0u, 1u, 7u})
        for (uint32_t sh : {(uint32_t)SH_NONE, (uint32_t)SH0, (uint32_t)SH1}) check_empty(need, sh);
    printf("failures %d\n", failures);
    return failures != 0;
}
