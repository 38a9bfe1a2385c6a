/*
 * A tile's first survivor as the decoder's wavefronts look for it, on the CPU: against a plain search for ascending lists
 * (even, clustered, up to what 32 bits hold), and within [0, k] for lists that are not ascending.  Rounds (each a trip to memory): two where
 * survivors are even; where they are clustered no more than a search by 64 probes a round takes, two more in short lists.
 */
#include "simt.hpp"

static uint32_t rounds;
#undef __ballot
#define __ballot(p) (rounds += simt::lane() == 0, simt::ballot(p, __LINE__))

#include "nsml.h"

#include "nsml_device_common.hpp"
#include "nsml_codec.hpp"

static uint64_t rng_state = 88172645463325252ull;
static uint32_t rnd() { rng_state ^= rng_state << 13; rng_state ^= rng_state >> 7; rng_state ^= rng_state << 17; return (uint32_t)(rng_state >> 20); }

static uint32_t rounds_of_probes(uint32_t k)
{
    uint32_t n = 0;
    for (; k; ++n) k = (k + 63) / 64 - 1;
    return n;
}

int main()
{
    int failures = 0, checked = 0;
    for (uint32_t k : {0u, 1u, 2u, 63u, 64u, 65u, 66u, 127u, 128u, 129u, 1000u, 5000u, 70001u, (1u << 21) + 70u})
        for (int kind = 0; kind < 6; ++kind) {
            const uint64_t nb = kind == 3 ? 0xFFFFF000ull : kind == 2 ? k : 40ull * k;
            std::vector<uint32_t> idx(k);
            uint64_t at = 0;
            for (uint32_t j = 0; j < k; ++j) {
                if (kind == 0 || kind == 5) idx[j] = (uint32_t)((nb - 40) * j / k + rnd() % 40);                      /* even; 5: not ascending */
                else if (kind == 1) { at += j % 300 ? 1 : 1 + rnd() % 10000; idx[j] = (uint32_t)std::min<uint64_t>(at, nb - k + j); }      /* runs */
                else if (kind == 2) idx[j] = j;
                else if (kind == 3) idx[j] = j < k / 2 ? j : (uint32_t)(nb - k + j);                                  /* the two ends */
                else idx[j] = (uint32_t)(nb - k + j);
            }
            if (kind != 5) std::sort(idx.begin(), idx.end());
            else for (uint32_t j = 0; j < k; ++j) std::swap(idx[j], idx[rnd() % k]);
            for (uint32_t turn = 0; turn < 40; ++turn) {
                const uint32_t head = turn % 4;
                const uint64_t edge = turn == 0 ? 0 : turn == 1 ? nb + head : turn == 2 ? (nb + head) / TILE * TILE
                                    : turn < 20 && k ? (uint64_t)idx[rnd() % k] + head + turn % 3 : rnd() % (nb + head + 1);
                const uint64_t want = std::partition_point(idx.begin(), idx.end(), [&](uint32_t i) { return (uint64_t)i + head < edge; }) - idx.begin();
                uint32_t got[64];
                rounds = 0;
                simt::run(64, dim3(0), dim3(1), [&] { got[threadIdx.x] = tilestart_wave(idx.data(), k, head, edge, nb ? (float)k / (float)nb : 0.0f); });
                bool ok = true;
                for (uint32_t l = 0; l < 64; ++l) ok = ok && got[l] == got[0] && (kind == 5 ? got[l] <= k : got[l] == want);
                const uint32_t most = kind == 0 || kind == 2 ? 2 : kind == 3 || kind == 4 ? rounds_of_probes(k) + (k > 64 && k <= 4160 ? 2 : 0) : rounds_of_probes(k) + 3;
                ++checked;
                if (!ok || (kind != 5 && rounds > most)) {
                    ++failures;
                    printf("k %u kind %d edge %llu: %u in %u rounds, by a plain search %llu, rounds at most %u\n", k, kind, (unsigned long long)edge, got[0], rounds, (unsigned long long)want, most);
                }
            }
        }
    printf("checked %d, failures %d\n", checked, failures);
    return failures ? 1 : 0;
}
