/*
 * libnsml GPU path for gfx950 (MI355X): hand-written HIP kernels and their C-ABI entry points.
 *
 * One compress call = error-feedback accumulation, exact top-k by magnitude per bucket
 * (Sec. 4.2 Step 3 / Algorithm 2 Step 3), value coding and payload packing; one decompress
 * call = payload -> dense gradient.  Nothing here is a dense contraction: every kernel is a
 * streaming pass bound by HBM bandwidth (or, for the small ones, by launch and dependent-load
 * latency), so the work is organised around coalesced 16-byte accesses, LDS histograms, 64-lane
 * ballots and as few dependent launches as possible, not MFMA.
 *
 * Selection is an exact radix select on the 31-bit magnitude key (binary32 pattern with the
 * sign cleared), digits of 12 + 12 + 7 bits, arranged so that the gradient is read ONCE:
 *
 *   sample    level-0 histogram of a 1/64 sample of grad + residual (small buckets: all of it)
 *   predict   per bucket, what the streaming pass stages: everything from a key L_b up that lies,
 *             with a wide margin, below the k-th largest ("candidates", ratios up to an eighth);
 *             a band [L_b, H_b) of keys around the k-th largest (larger ratios); nothing, when
 *             the k-th largest is a zero (sparse embeddings, ratio 1)
 *             (presample: both in one launch, a workgroup per bucket, unless buckets are many or large)
 *   ef_emit   acc = grad + residual (written over residual), the staged elements in index order to a
 *             segment per tile, how many lie above the window of keys around the expected
 *             threshold, and the window's bins (from 16384 tiles up by a kernel of their own, bins) 12 B/element
 *   select_count, select_finish   per bucket the plan: the window's bin that holds the k-th key, and the path: PATH_CAND,
 *             PATH_BAND, PATH_ZERO when the staged elements and the counts can decide it, else PATH_DENSE; then
 *             the staged entries against those bits: counts per segment, the
 *             few undecided keys set aside, then per bucket (one workgroup of 1024 threads) the
 *             remaining bits in LDS -> threshold key T_b, e_b = how many elements equal to T_b
 *             are admitted (lowest indices first), and every segment's place in the survivor order
 *   encode    PATH_CAND: one workgroup per chunk of survivors gathers them from the segments and
 *             codes them (absmax scale, codes, packing, indices, coding error into the residual)
 *             (16- and 32-bit values: PATH_DENSE as well)
 *   band      16- and 32-bit values, PATH_BAND / PATH_ZERO: survivors taken from the dense accumulator tile by tile
 *   hard      codes, PATH_BAND / PATH_ZERO: survivors taken from the dense
 *             accumulator and coded in one streaming pass; PATH_DENSE (an unlucky sample, a
 *             staging segment that overflowed, huge groups of equal keys): all radix steps over
 *             the dense accumulator, in a small resident grid with barriers between the steps
 *   quant     codes what hard left uncoded (chunks that straddle its work units; PATH_DENSE)
 *   tilestart, decomp    payload -> dense, each output line written once (with few tiles decomp looks for
 *             its survivors itself; few survivors: zeros, then the survivors stored over them)
 * Two kinds of call need none of the selection: small buckets (small: a workgroup per bucket does the
 * whole call) and ratio 1 (full: one streaming pass).
 * Every path gives the same bytes.
 *
 * With weights (Algorithm 2 Step 2) a weight pass comes first: sample of |w| -> band around the
 * threshold of the kept set (from the second call on: around the threshold the call before
 * found) -> one pass over w that stages the band, counts what lies above it and writes the
 * pruning bitmap for everything outside the band -> threshold and ties from the band with the
 * same select_count / select_finish -> bitmap bits of the band; the gradient kernels then read
 * one bit per element instead of the weight.
 *
 * Geometry: a bucket [lo, hi) is cut into tiles of 2048 elements starting at lo rounded down
 * to a multiple of 4, so every 16-byte access is aligned; elements of an edge tile outside
 * [lo, hi) are masked.  A tile is one workgroup of the streaming kernels and one staging segment.
 *
 * One translation unit: the device code lives in nsml_device_common.hpp (tables, geometry,
 * histogram helpers), nsml_select.hpp (sample .. plan, the radix steps over the dense
 * accumulator), nsml_prune.hpp (weight pass), nsml_codec.hpp (value coding of leftover chunks,
 * decompress, ratio 1), nsml_tail.hpp (select_count .. quant, the bitmap kernels) and nsml_small.hpp; this file holds
 * the context, the launch sequences and the C-ABI entry points.
 */
#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>

#include <math.h>
#include <stdint.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <new>
#include <vector>

#include "nsml.h"

#include "nsml_device_common.hpp"
#include "nsml_select.hpp"
#include "nsml_prune.hpp"
#include "nsml_codec.hpp"
#include "nsml_tail.hpp"
#include "nsml_small.hpp"

/* ====================================================================== host side */

struct nsml_ctx {
    int device;
    uint64_t max_n;
    uint32_t max_buckets;
    uint32_t chunk;
    int last_hip;
    uint64_t ws_bytes;
    uint32_t max_tiles;
    uint64_t max_cand;     /* staging entries */

    /* device workspace */
    uint64_t *d_off, *d_P, *d_V, *d_S, *d_C;
    uint32_t *d_tile0, *d_samp0, *d_tile_b, *d_k, *d_T, *d_need, *d_fast, *d_ftile0;
    uint4 *d_desc;         /* per tile: where it starts, its bucket, its valid slots */
    KeyPar *d_par, *d_wpar;        /* per bucket: what the streaming pass stages (gradient, weights) */
    uint32_t *d_sel0;      /* B+1 prefix of the workgroups per bucket of k_select_count */
    uint4 *d_selw;         /* per workgroup of k_select_count: bucket, first and last segment */
    uint32_t *d_chunk_b;   /* per chunk of the payload: its bucket (fixed by layout, ratio, bits) */
    uint32_t *d_chunk_seg; /* per chunk: the staging segment that holds its first survivor */
    uint32_t *d_sh, *d_why, *d_margin, *d_wprevT, *d_wprevHw, *d_wnband;
    uint2 *d_part;         /* per workgroup of k_select_count: its part of the bucket's list of undecided keys */
    uint32_t *d_lkey;      /* the lists */
    uint64_t max_chunks; uint32_t max_sel;
    uint32_t *d_zero;      /* cleared by every compress call: histograms and overflow flags */
    uint32_t *d_ccnt, *d_cG, *d_cE, *d_cidx;   /* candidate staging */
    float *d_cval;
    float *d_v;            /* survivor values in final order (not used for bits == 32) */
    uint32_t *d_ts;        /* decompress: where each tile's survivors start */
    uint32_t *d_pmask;     /* pruning bitmap, TILE / 32 words per tile */
    uint32_t *d_kw, *d_Tw, *d_needw;              /* pruning stage: kept counts, threshold search state */
    uint32_t *d_wfast;                            /* pruning stage: how each bucket was decided */
    uint32_t *h_flags;     /* pinned, mapped: [0] consistency flag of the selection, [1] of the pruning stage */
    uint32_t *d_flags;     /* the same two words as the kernels see them */
    double max_ratio;      /* largest ratio the survivor-value buffer was sized for */
    bool have_prune;                              /* the last compress call had weights */
    bool none_pruned;                             /* ... but its ratio prunes nothing: the weights were not read */
    uint64_t max_nb;                              /* largest bucket of the layout */
    bool off_mult4;                               /* every bucket of it starts at a multiple of 4 elements */
    double *d_tile_sq;     /* per tile: sum of grad^2 */
    double *d_l2sq;        /* per bucket: sum of grad^2 of the last compress call */
    bool have_l2;

    /* host copies / caches */
    std::vector<uint64_t> h_off;
    uint32_t B;
    uint64_t n;
    uint32_t n_tiles, n_samp, n_sel;
    uint32_t selSh;        /* log2 of the tiles per workgroup of k_select_count */
    bool tables_valid;
    double t_ratio; int t_bits;       /* what d_k/d_P/... were computed for */
    uint64_t K, NC;                   /* totals for (layout, t_ratio, t_bits) */
    uint64_t NC_cand;                 /* ... and the chunks of the buckets that may be decided from candidates */
    void *pinned; size_t pinned_bytes;
    int decomp_variant;    /* decompress: 1 zeros then survivors, 0 tiles assembled in LDS, -1 by the share of survivors */
    int force_dense;
    int unit_tiles;        /* tiles per work unit of the one-pass dense encode, 0 by gradient size */
    int sel_waves;         /* 16: 64 tiles per workgroup of k_select_count, 4, 8: 16 of them, 0 by gradient size */
    int built_sel_waves;   /* ... when the layout tables were made */
    int nt_acc, nt_dense;  /* accumulator / zeros of the dense output past the caches: 1, 0, -1 by size */
    bool zero_clean; uint32_t zero_B;   /* the per-call histograms and flags were left zeroed (for this many buckets) */
    int n_cu;
    int hard_occ[2];       /* workgroups of k_hard that fit a compute unit at once (short / long chunks) */
    int whistory;          /* the weight band follows the threshold of the last call (1, default) or always comes from a sample (0) */
    int wfix_apart;        /* the staged weight bands' bitmap by a launch of its own: 1, 0, -1 (default) = by gradient size */
    int wband_miss;        /* diagnostic: the weight band is placed beside the threshold, so every bucket takes the dense passes */
    int force_rescan;      /* diagnostic: k_select_finish in small windows; small buckets by the chain of kernels */

    /* profiling */
    bool prof;
    struct Rec { int kid; hipEvent_t a, b; };
    std::vector<Rec> recs;
    std::vector<hipEvent_t> pool;
};

namespace {

struct DeviceGuard {
    int prev; bool ok;
    explicit DeviceGuard(int dev) : prev(-1), ok(false) {
        if (hipGetDevice(&prev) != hipSuccess) prev = -1;
        ok = hipSetDevice(dev) == hipSuccess;
    }
    ~DeviceGuard() { if (prev >= 0) (void)hipSetDevice(prev); }
};

#define NSML_HIP(ctx, call)                                                        \
    do {                                                                           \
        hipError_t e_ = (call);                                                    \
        if (e_ != hipSuccess) { if (ctx) (ctx)->last_hip = (int)e_; return NSML_EHIP; } \
    } while (0)

template <typename T>
int dev_alloc(nsml_ctx *c, T **p, uint64_t count)
{
    const uint64_t bytes = (count ? count : 1) * sizeof(T);
    NSML_HIP(c, hipMalloc(reinterpret_cast<void **>(p), bytes));
    c->ws_bytes += bytes;
    return NSML_OK;
}

/* words of the area that is zero between calls: sample histogram, bins of the window, histograms of
 * the dense passes, overflow flags */
uint64_t zero_words(uint64_t B) { return B * (uint64_t)(NB0 + NHC * HROW + NB0 + NB1 + NB2 + 2) + 16; }   /* 16 spare words: counters */

struct Hists { uint32_t *hs, *hw, *f0, *f1, *f2, *ovf, *cursor, *nhard; };
Hists hists_of(const nsml_ctx *c, uint32_t B)
{
    Hists h;
    h.hs = c->d_zero;
    h.hw = h.hs + (uint64_t)B * NB0;
    h.f0 = h.hw + (uint64_t)B * NHC * HROW;
    h.f1 = h.f0 + (uint64_t)B * NB0;
    h.f2 = h.f1 + (uint64_t)B * NB1;
    h.ovf = h.f2 + (uint64_t)B * NB2;
    h.cursor = h.ovf + B;          /* k_select_count: length of the bucket's list of undecided keys */
    h.nhard = h.cursor + B;      /* k_select_count: buckets not on the candidate path */
    return h;
}

static uint32_t chunk_shift(uint32_t chunk)
{
    if (chunk == 0 || (chunk & (chunk - 1)) != 0) return NONE;
    uint32_t sh = 0;
    while ((1u << sh) != chunk) ++sh;
    return sh;
}

/* Tiles per work unit of the one-pass dense encode: a chunk that straddles units is coded by a kernel
 * of its own, so units are as large as leaves a few of them for every workgroup of its grid. */
static uint32_t denc_tiles(uint32_t n_tiles)
{
    return n_tiles >= 65536u ? 32u : n_tiles >= 32768u ? 16u : n_tiles >= 8192u ? 8u : n_tiles >= 2048u ? 4u : 2u;
}

Tables tables_of(const nsml_ctx *c)
{
    Tables t;
    t.off = c->d_off; t.tile0 = c->d_tile0; t.samp0 = c->d_samp0;
    t.tile_b = c->d_tile_b; t.desc = c->d_desc;
    t.k = c->d_k; t.P = c->d_P; t.V = c->d_V; t.S = c->d_S; t.C = c->d_C;
    t.T = c->d_T; t.need = c->d_need; t.par = c->d_par; t.fast = c->d_fast; t.sh = c->d_sh; t.why = c->d_why; t.margin = c->d_margin;
    t.ovf = hists_of(c, c->B).ovf; t.ftile0 = c->d_ftile0; t.nhard = hists_of(c, c->B).nhard;
    t.kw = c->d_kw; t.pmask = nullptr;
    t.B = c->B; t.n_tiles = c->n_tiles; t.chunk = c->chunk; t.chunkSh = chunk_shift(c->chunk);
    t.dencTiles = c->unit_tiles > 0 ? (uint32_t)c->unit_tiles : denc_tiles(c->n_tiles);
    return t;
}

Cand cand_of(const nsml_ctx *c)
{
    Cand k;
    k.idx = c->d_cidx; k.val = c->d_cval; k.cnt = c->d_ccnt; k.G = c->d_cG; k.E = c->d_cE;
    return k;
}

/* Profiling brackets */
int prof_begin(nsml_ctx *c, int kid, hipStream_t st, bool *recorded)
{
    *recorded = false;
    if (!c || !c->prof || c->recs.size() >= 4096) return NSML_OK;
    nsml_ctx::Rec r; r.kid = kid;
    for (hipEvent_t *e : {&r.a, &r.b}) {
        if (!c->pool.empty()) { *e = c->pool.back(); c->pool.pop_back(); }
        else NSML_HIP(c, hipEventCreate(e));
    }
    NSML_HIP(c, hipEventRecord(r.a, st));
    c->recs.push_back(r);
    *recorded = true;
    return NSML_OK;
}
/* closes the record prof_begin opened for this launch (and only if it opened one) */
int prof_end(nsml_ctx *c, bool recorded, hipStream_t st)
{
    if (!recorded) return NSML_OK;
    NSML_HIP(c, hipEventRecord(c->recs.back().b, st));
    return NSML_OK;
}

#define LAUNCHB(ctx, kid, st, kernel, grid, block, ...)                             \
    do {                                                                            \
        bool rec_ = false;                                                          \
        int rc_ = prof_begin(ctx, kid, st, &rec_);                                  \
        if (rc_) return rc_;                                                        \
        hipLaunchKernelGGL(kernel, dim3(grid), dim3(block), 0, st, __VA_ARGS__);    \
        NSML_HIP(ctx, hipGetLastError());                                           \
        rc_ = prof_end(ctx, rec_, st);                                              \
        if (rc_) return rc_;                                                        \
    } while (0)
#define LAUNCH(ctx, kid, st, kernel, grid, ...) LAUNCHB(ctx, kid, st, kernel, grid, WG, __VA_ARGS__)

bool aligned(const void *p, uintptr_t a) { return (reinterpret_cast<uintptr_t>(p) & (a - 1)) == 0; }

/* Validate a bucket layout; (re)build the layout tables if it differs from the cached one. */
int ensure_layout(nsml_ctx *c, uint64_t n, const uint64_t *off, uint32_t B, hipStream_t st)
{
    if (!off || B == 0 || n == 0) return NSML_EINVAL;
    if (B > c->max_buckets || n > c->max_n) return NSML_ECAP;
    if (off[0] != 0 || off[B] != n) return NSML_EINVAL;
    for (uint32_t b = 0; b < B; ++b) {
        if (off[b + 1] < off[b]) return NSML_EINVAL;
        if (off[b + 1] - off[b] > 0xFFFFFFFFull) return NSML_EINVAL;
    }
    if (c->B == B && c->n == n && c->built_sel_waves == c->sel_waves && c->h_off.size() == (size_t)B + 1 &&
        memcmp(c->h_off.data(), off, sizeof(uint64_t) * ((size_t)B + 1)) == 0)
        return NSML_OK;

    /* new layout: tiles start at the bucket start rounded down to a multiple of 4 */
    const size_t B1 = (size_t)B + 1;
    std::vector<uint32_t> tile0(B1), samp0(B1), sel0(B1);
    uint64_t nt = 0, nsamp = 0, nsel = 0;
    /* 64 tiles per workgroup of k_select_count once that leaves four workgroups per compute unit, else 16
     * (12 K tiles of a hundred entries: 35 us with 64, 10 with 16) */
    const uint32_t selSh = c->sel_waves ? (c->sel_waves == 16 ? 6u : 4u) : n >= 4ull * 64ull * 256ull * TILE ? 6u : 4u;
    for (uint32_t b = 0; b < B; ++b) {
        tile0[b] = (uint32_t)nt;
        samp0[b] = (uint32_t)nsamp;
        sel0[b] = (uint32_t)nsel;
        const uint64_t lo = off[b], hi = off[b + 1];
        if (hi > lo) {
            const uint64_t len = hi - (lo & ~3ull);
            const uint64_t tiles = (len + TILE - 1) / TILE;
            nt += tiles;
            nsel += (tiles + (1u << selSh) - 1) >> selSh;
            const uint64_t run_elems = SAMPLE_RUN * sample_stride(hi - lo);
            const uint64_t runs = (len + run_elems - 1) / run_elems;
            nsamp += (runs + RUNS_PER_WG - 1) / RUNS_PER_WG;
        }
        if (nt > c->max_tiles || nsel > c->max_sel) return NSML_ECAP;
    }
    tile0[B] = (uint32_t)nt;
    samp0[B] = (uint32_t)nsamp;
    sel0[B] = (uint32_t)nsel;

    /* the stream may still be using the old tables */
    NSML_HIP(c, hipStreamSynchronize(st));
    c->tables_valid = false;
    c->B = 0;
    const size_t need = sizeof(uint64_t) * B1 + 3 * sizeof(uint32_t) * B1;
    if (need > c->pinned_bytes) return NSML_ECAP;
    uint8_t *hp = static_cast<uint8_t *>(c->pinned);
    uint8_t *hp_t = hp + sizeof(uint64_t) * B1;
    uint8_t *hp_m = hp_t + sizeof(uint32_t) * B1;
    uint8_t *hp_l = hp_m + sizeof(uint32_t) * B1;
    memcpy(hp, off, sizeof(uint64_t) * B1);
    memcpy(hp_t, tile0.data(), sizeof(uint32_t) * B1);
    memcpy(hp_m, samp0.data(), sizeof(uint32_t) * B1);
    memcpy(hp_l, sel0.data(), sizeof(uint32_t) * B1);
    NSML_HIP(c, hipMemcpyAsync(c->d_off, hp, sizeof(uint64_t) * B1, hipMemcpyHostToDevice, st));
    NSML_HIP(c, hipMemcpyAsync(c->d_tile0, hp_t, sizeof(uint32_t) * B1, hipMemcpyHostToDevice, st));
    NSML_HIP(c, hipMemcpyAsync(c->d_samp0, hp_m, sizeof(uint32_t) * B1, hipMemcpyHostToDevice, st));
    NSML_HIP(c, hipMemcpyAsync(c->d_sel0, hp_l, sizeof(uint32_t) * B1, hipMemcpyHostToDevice, st));
    {
        Tables t;
        memset(&t, 0, sizeof t);
        t.off = c->d_off; t.tile0 = c->d_tile0; t.B = B; t.n_tiles = (uint32_t)nt;
        LAUNCH(c, KID_TILEMAP, st, k_tilemap, (uint32_t)((nt + WG - 1) / WG), t, c->d_tile_b, c->d_desc);
    }
    LAUNCH(c, KID_TILEMAP, st, k_selmap, (uint32_t)((nsel + WG - 1) / WG), (const uint32_t *)c->d_sel0,
           (const uint32_t *)c->d_tile0, B, (uint32_t)nsel, selSh, c->d_selw);
    NSML_HIP(c, hipMemsetAsync(c->d_wprevT, 0xFF, sizeof(uint32_t) * B1, st));     /* other buckets: nothing remembered */
    NSML_HIP(c, hipMemsetAsync(c->d_margin, 0, sizeof(uint32_t) * B1, st));
    NSML_HIP(c, hipStreamSynchronize(st));

    c->h_off.assign(off, off + B + 1);
    c->max_nb = 0; c->off_mult4 = true;
    for (uint32_t b = 0; b < B; ++b) c->off_mult4 = c->off_mult4 && off[b] % 4 == 0;
    for (uint32_t b = 0; b < B; ++b) c->max_nb = off[b + 1] - off[b] > c->max_nb ? off[b + 1] - off[b] : c->max_nb;
    c->B = B; c->n = n;
    c->n_tiles = (uint32_t)nt; c->n_samp = (uint32_t)nsamp;
    c->n_sel = (uint32_t)nsel; c->selSh = selSh; c->built_sel_waves = c->sel_waves;
    return NSML_OK;
}

/* K and NC of (ratio, bits) for the cached layout; stale: d_k / d_P / d_V / d_S / d_C are those of another. */
int plan_tables(nsml_ctx *c, double ratio, int bits, bool &stale)
{
    if (!(ratio > 0.0 && ratio <= 1.0)) return NSML_EINVAL;
    if (bits != 4 && bits != 8 && bits != 16 && bits != 32) return NSML_EINVAL;
    stale = !(c->tables_valid && c->t_ratio == ratio && c->t_bits == bits);
    if (!stale) return NSML_OK;
    c->tables_valid = false;
    uint64_t K = 0, nc = 0, cand = 0;
    {
        std::vector<uint64_t> kb(c->B);
        int rc = nsml_payload_layout(c->h_off.data(), c->B, ratio, bits, c->chunk, kb.data(), &K, nullptr, nullptr);
        if (rc) return rc;
        for (uint32_t b = 0; b < c->B; ++b) {
            const uint64_t lo = c->h_off[b], hi = c->h_off[b + 1], chunks = (kb[b] + c->chunk - 1) / c->chunk;
            nc += chunks;
            if (kb[b] < hi - lo && candidates_fit(kb[b], (hi - (lo & ~3ull) + TILE - 1) / TILE)) cand += chunks;
        }
    }
    if (nc >= 0x7FFFFFFFull || nc > c->max_chunks) return NSML_ECAP;
    c->K = K; c->NC = nc; c->NC_cand = cand;
    c->t_ratio = ratio; c->t_bits = bits;
    return NSML_OK;
}

/* Workgroups (of `threads`) that make the tables, and the chunks they map */
uint32_t setup_grid(const nsml_ctx *c, uint32_t threads, uint64_t &chunks)
{
    chunks = c->B <= SETUP_MAX_B ? c->NC : 0u;
    return (uint32_t)std::min<uint64_t>(1024u, std::max<uint64_t>(1u, (chunks + threads - 1) / threads));
}
int chunk_map(nsml_ctx *c, hipStream_t st)
{
    if (c->NC && c->B > SETUP_MAX_B)
        LAUNCH(c, KID_SETUP, st, k_chunkmap, (uint32_t)((c->NC + WG - 1) / WG), (const uint64_t *)c->d_C, c->B, c->NC, c->d_chunk_b);
    c->tables_valid = true;
    return NSML_OK;
}

/* Make the tables match (ratio, bits) in a launch of their own. */
int make_tables(nsml_ctx *c, hipStream_t st)
{
    uint64_t chunks;
    const uint32_t grid = setup_grid(c, WG, chunks);
    LAUNCH(c, KID_SETUP, st, k_setup, grid, tables_of(c), c->t_ratio, c->t_bits, chunks, c->d_chunk_b);
    return chunk_map(c, st);
}
int ensure_tables(nsml_ctx *c, double ratio, int bits, hipStream_t st)
{
    bool stale;
    const int rc = plan_tables(c, ratio, bits, stale);
    return rc || !stale ? rc : make_tables(c, st);
}

/* A device-side consistency check that tripped during an earlier call is reported once, by the
 * next GPU entry point (the kernels raise the flag in host memory they can reach; reading it
 * needs no synchronisation, so the report comes one call late). */
bool pending_internal_error(nsml_ctx *c)
{
    volatile uint32_t *f = c->h_flags;
    if (!f || (f[0] | f[1]) == 0u) return false;
    f[0] = 0u; f[1] = 0u;
    c->zero_clean = false;
    return true;
}

}  // namespace

extern "C" {

int nsml_create(nsml_ctx **out, int device, uint64_t max_n, uint32_t max_buckets, uint32_t chunk)
{
    return nsml_create_ex(out, device, max_n, max_buckets, chunk, 1.0);
}

int nsml_create_ex(nsml_ctx **out, int device, uint64_t max_n, uint32_t max_buckets, uint32_t chunk,
                   double max_ratio)
{
    if (!out || max_n == 0 || max_buckets == 0 || chunk == 0 || chunk % 8 != 0) return NSML_EINVAL;
    if (!(max_ratio > 0.0 && max_ratio <= 1.0)) return NSML_EINVAL;
    *out = nullptr;
    nsml_ctx *c = new (std::nothrow) nsml_ctx();
    if (!c) return NSML_ENOMEM;
    c->device = device; c->max_n = max_n; c->max_buckets = max_buckets; c->chunk = chunk;
    c->last_hip = 0; c->ws_bytes = 0; c->B = 0; c->n = 0; c->tables_valid = false;
    c->prof = false; c->pinned = nullptr; c->pinned_bytes = 0;
    c->d_off = c->d_P = c->d_V = c->d_S = c->d_C = nullptr;
    c->d_tile0 = c->d_samp0 = c->d_tile_b = c->d_k = c->d_T = c->d_need = nullptr;
    c->d_fast = c->d_ftile0 = c->d_zero = nullptr; c->d_desc = nullptr; c->d_par = c->d_wpar = nullptr;
    c->d_sel0 = nullptr; c->d_selw = nullptr; c->d_chunk_b = c->d_chunk_seg = c->d_sh = c->d_why = c->d_margin = c->d_wprevT = c->d_wprevHw = c->d_wnband = nullptr;
    c->d_part = nullptr; c->d_lkey = nullptr;
    c->d_ccnt = c->d_cG = c->d_cE = c->d_cidx = nullptr;
    c->d_cval = nullptr; c->d_v = nullptr; c->d_ts = nullptr; c->d_tile_sq = c->d_l2sq = nullptr; c->have_l2 = false;
    c->d_pmask = c->d_kw = c->d_Tw = c->d_needw = c->d_wfast = nullptr;
    c->h_flags = c->d_flags = nullptr;
    c->have_prune = false; c->none_pruned = false; c->max_nb = 0;
    c->max_ratio = max_ratio;
    /* tuning switches: the measured defaults (see nsml_set_option) */
    c->zero_clean = false; c->zero_B = 0;
    c->n_cu = 256; c->decomp_variant = -1;
    c->unit_tiles = c->sel_waves = c->built_sel_waves = 0; c->nt_acc = c->nt_dense = -1;
    c->force_dense = 0; c->force_rescan = 0; c->wband_miss = 0; c->whistory = 1; c->wfix_apart = -1;

    int ndev = 0;
    if (hipGetDeviceCount(&ndev) != hipSuccess || device < 0 || device >= ndev) {
        c->last_hip = (int)hipErrorInvalidDevice;
        delete c;
        return NSML_EHIP;
    }
    DeviceGuard guard(device);
    if (!guard.ok) { delete c; return NSML_EHIP; }
    {
        int cus = 0;
        if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device) == hipSuccess && cus > 0) c->n_cu = cus;
        /* k_hard's workgroups meet at barriers, so its grid must fit the device at once: ask the
         * runtime how many of them a compute unit holds (the variants per width use the same LDS) */
        int occ = 0;
        c->hard_occ[0] = c->hard_occ[1] = 1;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, k_hard<8, false>, (int)HTH, 0) == hipSuccess && occ > 0)
            c->hard_occ[0] = occ < (int)hard_wg_per_cu(false) ? occ : (int)hard_wg_per_cu(false);
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, k_hard<8, true>, (int)HTH, 0) == hipSuccess && occ > 0)
            c->hard_occ[1] = occ < (int)hard_wg_per_cu(true) ? occ : (int)hard_wg_per_cu(true);
        (void)hipGetLastError();
    }

    /* every bucket can add one partial tile at each end */
    const uint64_t mt = max_n / TILE + 2ull * max_buckets + 2;
    if (mt >= 0x3FFFFFFFull) { delete c; return NSML_ECAP; }
    c->max_tiles = (uint32_t)mt;
    /* staging: a quarter of the elements every tile covers */
    c->max_cand = mt * SEG_CAP;
    const uint64_t B1 = (uint64_t)max_buckets + 1;
    int rc = NSML_OK;
    auto A = [&](int r) { if (rc == NSML_OK) rc = r; };
    A(dev_alloc(c, &c->d_off, B1)); A(dev_alloc(c, &c->d_P, B1)); A(dev_alloc(c, &c->d_V, B1));
    A(dev_alloc(c, &c->d_S, B1)); A(dev_alloc(c, &c->d_C, B1));
    A(dev_alloc(c, &c->d_tile0, B1)); A(dev_alloc(c, &c->d_samp0, B1));
    A(dev_alloc(c, &c->d_k, B1)); A(dev_alloc(c, &c->d_T, B1)); A(dev_alloc(c, &c->d_need, B1));
    A(dev_alloc(c, &c->d_par, B1)); A(dev_alloc(c, &c->d_wpar, B1)); A(dev_alloc(c, &c->d_fast, B1)); A(dev_alloc(c, &c->d_ftile0, B1));
    A(dev_alloc(c, &c->d_sel0, B1)); A(dev_alloc(c, &c->d_sh, B1)); A(dev_alloc(c, &c->d_why, B1)); A(dev_alloc(c, &c->d_margin, B1));
    A(dev_alloc(c, &c->d_tile_b, mt)); A(dev_alloc(c, &c->d_desc, mt));
    A(dev_alloc(c, &c->d_zero, zero_words(max_buckets)));
    A(dev_alloc(c, &c->d_ccnt, mt)); A(dev_alloc(c, &c->d_cG, mt)); A(dev_alloc(c, &c->d_cE, mt));
    /* k_select_count workgroups: every bucket can end with a short one */
    c->max_sel = (uint32_t)(mt / 16 + B1);
    A(dev_alloc(c, &c->d_selw, c->max_sel));
    A(dev_alloc(c, &c->d_part, c->max_sel));
    A(dev_alloc(c, &c->d_lkey, mt * LIST_PER_SEG + B1 * LCAP));
    A(dev_alloc(c, &c->d_cidx, c->max_cand)); A(dev_alloc(c, &c->d_cval, c->max_cand));
    {   /* survivor values in final order: ceil(ratio * n_b) per bucket, at most one more than
         * ratio * n_b each */
        uint64_t mv = (uint64_t)ceil(max_ratio * (double)max_n) + max_buckets;
        if (mv > max_n) mv = max_n;
        A(dev_alloc(c, &c->d_v, mv));
        /* chunks of the payload: every bucket can end with a short one */
        c->max_chunks = mv / chunk + max_buckets + 1;
        A(dev_alloc(c, &c->d_chunk_b, c->max_chunks)); A(dev_alloc(c, &c->d_chunk_seg, c->max_chunks));
    }
    A(dev_alloc(c, &c->d_ts, mt + B1 + 1));
    A(dev_alloc(c, &c->d_tile_sq, mt)); A(dev_alloc(c, &c->d_l2sq, B1));
    A(dev_alloc(c, &c->d_pmask, mt * (TILE / 32)));
    A(dev_alloc(c, &c->d_kw, B1)); A(dev_alloc(c, &c->d_Tw, B1)); A(dev_alloc(c, &c->d_needw, B1));
    A(dev_alloc(c, &c->d_wfast, B1));
    A(dev_alloc(c, &c->d_wprevT, B1)); A(dev_alloc(c, &c->d_wprevHw, B1)); A(dev_alloc(c, &c->d_wnband, B1));
    if (rc == NSML_OK) {
        hipError_t e = hipMemset(c->d_margin, 0, sizeof(uint32_t) * B1);
        if (e == hipSuccess) e = hipMemset(c->d_wprevT, 0xFF, sizeof(uint32_t) * B1);   /* nothing remembered */
        if (e != hipSuccess) { c->last_hip = (int)e; rc = NSML_EHIP; }
    }
    if (rc == NSML_OK) {
        c->pinned_bytes = B1 * 24;
        hipError_t e = hipHostMalloc(&c->pinned, c->pinned_bytes, hipHostMallocDefault);
        if (e != hipSuccess) { c->last_hip = (int)e; rc = NSML_EHIP; }
    }
    if (rc == NSML_OK) {
        /* two words the kernels write only when a consistency check fails; the host reads them
         * at the start of the next call, without waiting for anything */
        void *hp = nullptr, *dp = nullptr;
        hipError_t e = hipHostMalloc(&hp, 64, hipHostMallocMapped);
        if (e == hipSuccess) {
            c->h_flags = static_cast<uint32_t *>(hp);
            c->h_flags[0] = c->h_flags[1] = 0u;
            e = hipHostGetDevicePointer(&dp, hp, 0);
        }
        if (e != hipSuccess) { c->last_hip = (int)e; rc = NSML_EHIP; }
        else c->d_flags = static_cast<uint32_t *>(dp);
    }
    if (rc != NSML_OK) { nsml_destroy(c); return rc; }
    *out = c;
    return NSML_OK;
}

int nsml_destroy(nsml_ctx *c)
{
    if (!c) return NSML_EINVAL;
    DeviceGuard guard(c->device);
    (void)hipDeviceSynchronize();
    void *ptrs[] = {c->d_off, c->d_P, c->d_V, c->d_S, c->d_C, c->d_tile0, c->d_samp0,
                    c->d_tile_b, c->d_desc, c->d_k, c->d_T, c->d_need, c->d_par, c->d_wpar, c->d_fast, c->d_ftile0,
                    c->d_zero, c->d_ccnt, c->d_cG, c->d_cE, c->d_cidx,
                    c->d_cval, c->d_v, c->d_ts, c->d_tile_sq, c->d_l2sq, c->d_pmask, c->d_kw,
                    c->d_Tw, c->d_needw, c->d_wfast,
                    c->d_sel0, c->d_selw, c->d_chunk_b, c->d_chunk_seg, c->d_part, c->d_lkey, c->d_sh, c->d_why, c->d_margin, c->d_wprevT, c->d_wprevHw, c->d_wnband};
    for (void *p : ptrs) if (p) (void)hipFree(p);
    if (c->pinned) (void)hipHostFree(c->pinned);
    if (c->h_flags) (void)hipHostFree(c->h_flags);
    for (auto &r : c->recs) { (void)hipEventDestroy(r.a); (void)hipEventDestroy(r.b); }
    for (auto e : c->pool) (void)hipEventDestroy(e);
    delete c;
    return NSML_OK;
}

int nsml_last_hip_error(const nsml_ctx *c) { return c ? c->last_hip : 0; }
uint64_t nsml_workspace_bytes(const nsml_ctx *c) { return c ? c->ws_bytes : 0; }

/* Shared body of nsml_compress and nsml_compress_pruned (weights == NULL: no pruning). */
static int compress_impl(nsml_ctx *c, const float *grad, float *residual, const float *weights,
                         uint64_t n, const uint64_t *bucket_off, uint32_t B, double ratio, int bits,
                         uint32_t *idx, void *val, float *scales, void *stream)
{
    if (!c || !grad || !residual || !idx || !val) return NSML_EINVAL;
    if ((bits == 8 || bits == 4) && !scales) return NSML_EINVAL;
    if (!aligned(grad, 16) || !aligned(residual, 16) || !aligned(idx, 4) || !aligned(val, 4) ||
        !aligned(scales, 4) || !aligned(weights, 16))
        return NSML_EINVAL;
    if (ratio > c->max_ratio) return NSML_ECAP;
    if (pending_internal_error(c)) return NSML_EINTERNAL;
    hipStream_t st = static_cast<hipStream_t>(stream);
    DeviceGuard guard(c->device);
    if (!guard.ok) { c->last_hip = (int)hipErrorInvalidDevice; return NSML_EHIP; }
    int rc = ensure_layout(c, n, bucket_off, B, st);
    if (rc) return rc;
    bool stale;
    rc = plan_tables(c, ratio, bits, stale);
    if (rc) return rc;
    /* Sample and prediction by a workgroup per bucket, which also makes stale tables: up to four turns of a workgroup
     * on every compute unit, and no bucket that needs a larger sample (compress, us, this / k_sample and k_predict: 1024 buckets of
     * 45 elements 100 / 103, 1000 of 40000 204 / 243, one of 1 Mi 50.6 / 54.1; 16 of 4 M 195 / 202). */
    const bool presample = B <= 4u * (uint32_t)c->n_cu && c->max_nb < PRE_BIG && !c->force_dense;

    Tables t = tables_of(c);
    const Cand cd0 = cand_of(c);
    const Hists h = hists_of(c, B);
    const uint64_t zw = zero_words(B);
    const uint32_t clear_grid = (uint32_t)((zw + WG * 8 - 1) / (WG * 8));
    const dim3 sgrid = xcd_grid(c->n_tiles);         /* streaming passes: a workgroup per tile */
    const bool nt = c->nt_acc < 0 ? n > NT_ELEMS : c->nt_acc != 0;
    /* the window's bins by a kernel of their own: with many tiles, which may be those of many small buckets (and
     * whenever the accumulator goes past the caches, which it does with more elements than so many tiles have) */
    const bool bins = !c->force_dense && (nt || c->n_tiles >= HIST_MAX_TILES);
    /* floor(0.5 * (1 - ratio) * n_b) parameters are pruned: when that is none of any bucket (ratio 1, the
     * controller's cap), the weights decide nothing and are not read */
    const bool none_pruned = weights && floor(0.5 * (1.0 - ratio) * (double)c->max_nb) < 1.0;
    if (none_pruned) weights = nullptr;
    const bool full = c->K == n && !c->force_dense && (bits >= 16 || TILE % c->chunk == 0);
    const bool small = !weights && !c->force_dense && !c->force_rescan && c->max_nb <= SMALL_MAX && B < (1u << 22);      /* (2^32 threads cannot be launched) */
    if (stale && (full || small || weights || !presample)) {
        rc = make_tables(c, st);
        if (rc) return rc;
        stale = false;
    }
    if (full) {
        /* everything is sent: nothing to select (TILE % chunk: chunks nest in tiles) */
        const bool fnt = nt && c->off_mult4 && aligned(idx, 16) && aligned(val, 16);      /* (misaligned non-temporal stores leave partly written lines) */
#define NSML_FULL(BITS_)                                                                                                                      \
    do {                                                                                                                                       \
        if (fnt) LAUNCHB(c, KID_EF_EMIT, st, (k_full<BITS_, true>), sgrid, STH, grad, residual, t, cd0, c->d_tile_sq, idx, val, scales);        \
        else LAUNCHB(c, KID_EF_EMIT, st, (k_full<BITS_, false>), sgrid, STH, grad, residual, t, cd0, c->d_tile_sq, idx, val, scales);           \
    } while (0)
        switch (bits) {
        case 32: NSML_FULL(32); break;
        case 16: NSML_FULL(16); break;
        case 8:  NSML_FULL(8); break;
        default: NSML_FULL(4); break;
        }
#undef NSML_FULL
        if (c->max_nb > STATE_BIG) LAUNCHB(c, KID_PLAN, st, k_full_state<1024>, B, 1024, t, cd0, (const double *)c->d_tile_sq, c->d_l2sq);
        else LAUNCHB(c, KID_PLAN, st, k_full_state<256>, B, 256, t, cd0, (const double *)c->d_tile_sq, c->d_l2sq);
        c->have_l2 = true;
        c->have_prune = none_pruned; c->none_pruned = none_pruned;
        return NSML_OK;
    }

    /* Small buckets: the whole call in one launch.  A workgroup fills a compute unit, so its time goes in rounds of one
     * bucket for each of them, and it is ahead of the chain of kernels however many there are (us, 1 % sent as 8-bit codes, this /
     * the chain: 1 bucket of 32764 elements 31 / 34, 512 of them 89 / 115, 4000 of them 611 / 781; 1000 of 5000 50 / 94,
     * 20000 of them 878 / 1617; 17000 of 45 521 / 1105). */
    if (small) {
        switch (bits) {
        case 32: LAUNCHB(c, KID_EF_EMIT, st, k_small<32>, B, SMALL_T, grad, residual, t, c->d_l2sq, idx, val, scales); break;
        case 16: LAUNCHB(c, KID_EF_EMIT, st, k_small<16>, B, SMALL_T, grad, residual, t, c->d_l2sq, idx, val, scales); break;
        case 8:  LAUNCHB(c, KID_EF_EMIT, st, k_small<8>, B, SMALL_T, grad, residual, t, c->d_l2sq, idx, val, scales); break;
        default: LAUNCHB(c, KID_EF_EMIT, st, k_small<4>, B, SMALL_T, grad, residual, t, c->d_l2sq, idx, val, scales); break;
        }
        c->have_l2 = true;
        c->have_prune = none_pruned; c->none_pruned = none_pruned;
        return NSML_OK;
    }

    /* the kernels below zero what they have read of the per-call histograms and flags, so a fill
     * is only needed after something else used the area: another bucket count, a call that did not
     * get to its end */
    if (!c->zero_clean || c->zero_B != B)
        LAUNCH(c, KID_CLEAR, st, k_clear, clear_grid < 2048 ? clear_grid : 2048, c->d_zero, zw);
    c->zero_clean = false;

    if (weights) {
        /* Algorithm 2 Step 2: threshold and cut of |w| per bucket, on its own set of tables */
        Tables tw = t;
        tw.k = c->d_kw; tw.T = c->d_Tw; tw.need = c->d_needw; tw.fast = c->d_wfast;
        tw.par = c->d_wpar;                            /* the staged band of weight keys (never without an upper bound) */
        const uint32_t *known = c->whistory && !c->wband_miss ? c->d_wprevT : nullptr;      /* what the last call found */
        if (!c->force_dense)
            LAUNCH(c, KID_SAMPLE, st, k_sample<false>, c->n_samp, weights, (const float *)nullptr, tw, h.hs, known);
        LAUNCH(c, KID_WPLAN, st, k_wpredict, B, tw, h.hs, c->force_dense, c->wband_miss, known, (const uint32_t *)c->d_wprevHw);
        if (bins) LAUNCHB(c, KID_WHIST, st, k_whist<false>, sgrid, WTH, weights, tw, h.hw, cd0, c->d_pmask);
        else LAUNCHB(c, KID_WHIST, st, k_whist<true>, sgrid, WTH, weights, tw, h.hw, cd0, c->d_pmask);
        /* buckets decided from their band: undecided keys, threshold key and tie count, the pruned
         * band elements' bits; buckets on the dense passes (no band, or one that missed): by the last launch's first workgroups */
        if (c->force_dense) {
            LAUNCH(c, KID_WPLAN, st, k_wplan_dense, (B + WG - 1) / WG, tw, c->d_wprevT);
            LAUNCH(c, KID_WHARD, st, k_whard, (uint32_t)c->n_cu, weights, tw, cd0, h.f0, h.f1, h.f2, c->d_pmask, c->d_flags + 1);
        } else {
            if (bins) LAUNCH(c, KID_BINS, st, k_bins, c->n_sel, tw, cd0, (const uint4 *)c->d_selw, c->selSh, h.hw, weights);
            LAUNCH(c, KID_SELECT, st, k_select_count<false>, c->n_sel, tw, cd0, (const uint4 *)c->d_selw, (const uint32_t *)h.hw, h.cursor, c->d_part, c->d_lkey, c->d_flags + 1, weights, c->d_wnband);
            LAUNCHB(c, KID_FINISH, st, k_select_finish, B, SEL_THREADS, tw, cd0, (const uint32_t *)c->d_sel0, c->selSh, h.cursor,
                    (const uint2 *)c->d_part, (const uint32_t *)c->d_lkey, (uint32_t *)nullptr, c->d_flags + 1, c->force_rescan);
            const bool apart = c->wfix_apart < 0 ? c->n_tiles > 65536u : c->wfix_apart != 0;       /* see k_wfix */
            if (apart) LAUNCH(c, KID_WMASK, st, k_wfix, (c->n_tiles + 15) / 16, tw, cd0, c->d_pmask);
            LAUNCH(c, KID_WMASK, st, k_wrest, (uint32_t)c->n_cu + (apart ? 0u : (c->n_tiles + 15) / 16), weights, tw, cd0, h.f0, h.f1, h.f2, c->d_pmask, c->d_flags + 1, (uint32_t)c->n_cu, h.hw,
                   (const uint32_t *)c->d_wnband, c->d_wprevT, c->d_wprevHw);
        }
        t.pmask = c->d_pmask;
    }

    const bool pruned = weights != nullptr;
    if (presample) {
        uint64_t chunks = 0;
        const uint32_t extra = stale ? setup_grid(c, PRE_T, chunks) : 0u;
        LAUNCHB(c, KID_SAMPLE, st, k_presample, B + extra, PRE_T, grad, (const float *)residual, t, ratio, bits, c->max_nb < SAMPLE_ALL_BELOW, chunks, c->d_chunk_b);
        if (stale) { rc = chunk_map(c, st); if (rc) return rc; }
    } else {
        if (!c->force_dense)
            LAUNCH(c, KID_SAMPLE, st, k_sample<true>, c->n_samp, grad, (const float *)residual, t, h.hs, (const uint32_t *)nullptr);
        LAUNCH(c, KID_PREDICT, st, k_predict, B, t, h.hs, c->force_dense);
    }
#define NSML_EF(EMIT_, PRUNE_, NT_, HIST_) LAUNCHB(c, KID_EF_EMIT, st, (k_ef_emit<EMIT_, PRUNE_, NT_, HIST_>), sgrid, STH, grad, residual, t, h.hw, cd0, c->d_tile_sq)
    if (c->force_dense) { if (nt) NSML_EF(false, false, true, false); else NSML_EF(false, false, false, false); }
    else if (nt) { if (pruned) NSML_EF(true, true, true, false); else NSML_EF(true, false, true, false); }
    else if (bins) { if (pruned) NSML_EF(true, true, false, false); else NSML_EF(true, false, false, false); }
    else { if (pruned) NSML_EF(true, true, false, true); else NSML_EF(true, false, false, true); }
#undef NSML_EF
    if (bins) LAUNCH(c, KID_BINS, st, k_bins, c->n_sel, t, cd0, (const uint4 *)c->d_selw, c->selSh, h.hw, (const float *)residual);
    if (c->force_dense) LAUNCHB(c, KID_PLAN, st, k_plan_dense, B, 1024, t, (const double *)c->d_tile_sq, c->d_l2sq);
    /* the workgroups that meet at barriers on the dense passes: one per compute unit, so that the teams of two or
     * three contexts working at the same time still fit the device together */
    const bool big = c->chunk > DENC_SMALL_CHUNK;
    const uint32_t hgrid = (uint32_t)(c->hard_occ[big ? 1 : 0] * c->n_cu), team = std::min((uint32_t)c->n_cu, hgrid);
    if (!c->force_dense) {
        /* buckets decided from their staged elements: undecided keys set apart, threshold and
         * survivor order per bucket, then the payload of the candidate-path buckets */
        const uint4 *selw = c->d_selw;
        LAUNCH(c, KID_SELECT, st, k_select_count<true>, c->n_sel, t, cd0, selw, (const uint32_t *)h.hw, h.cursor, c->d_part, c->d_lkey, c->d_flags, (const float *)residual, (uint32_t *)nullptr);
        LAUNCHB(c, KID_FINISH, st, k_select_finish, B, SEL_THREADS, t, cd0, (const uint32_t *)c->d_sel0, c->selSh, h.cursor,
                (const uint2 *)c->d_part, (const uint32_t *)c->d_lkey, c->d_chunk_seg, c->d_flags, c->force_rescan);
        {
            const uint32_t *cb_ = c->d_chunk_b, *cs_ = c->d_chunk_seg;
            const uint64_t nc64e = c->NC;
            /* Threads per chunk: 256 once there are two workgroups for every compute unit, unless the chunks are long
             * (8-bit codes in chunks of 2048, 256 / 512 threads, us: 2000 buckets of 5000 elements at 0.001, five
             * survivors a chunk, 22 / 45; 600 of 30000 at 0.1, 1500 a chunk, 32 / 45; fewer workgroups: ResNet-50's
             * 165 chunks of 156 survivors 25 / 18, 279 of 940 22 / 20; full chunks: 3072 of 2048 190 / 182). */
            const bool narrow = c->NC >= 2u * (uint64_t)c->n_cu && c->K <= 1900u * c->NC;
            /* A workgroup per chunk that may be coded here (beyond a ratio of an eighth those of the smallest buckets: k_hard
             * codes the others), a few to look for them, and not very many (2^32 threads cannot be launched).  (A small grid as soon
             * as K * 8 > n codes all of it at a ratio of 1/8 and odd sizes: 4 buckets of 27370561 elements 677 us a round, so 663.) */
            const uint32_t first = bits >= 16 ? std::max(B, team) : B;
            const uint32_t egrid2 = (uint32_t)std::min<uint64_t>({c->NC, std::max<uint64_t>(c->NC_cand, (narrow ? 4u : 2u) * (uint64_t)c->n_cu), 16384u});
#define NSML_ENCODE1(BITS_, T_) LAUNCHB(c, KID_ENCODE, st, (k_encode<BITS_, T_>), first + egrid2, T_, t, cd0, cb_, cs_, residual, idx, val, scales, c->d_flags, nc64e, h.hw, \
                                        (const double *)c->d_tile_sq, c->d_l2sq, h.f0, h.f1, h.f2, first, team)
#define NSML_ENCODE(BITS_)                     \
    do {                                        \
        if (narrow) NSML_ENCODE1(BITS_, 256);    \
        else NSML_ENCODE1(BITS_, 512);           \
    } while (0)
            switch (bits) {
            case 32: NSML_ENCODE(32); break;
            case 16: NSML_ENCODE(16); break;
            case 8:  NSML_ENCODE(8); break;
            default: NSML_ENCODE(4); break;
            }
#undef NSML_ENCODE
#undef NSML_ENCODE1
        }
    }
    /* the buckets whose survivors come from the dense accumulator (up to an eighth sent usually none: the workgroups read one
     * word and leave): whole values tile by tile; codes by a fixed grid, resident at once, that streams the band and zero-threshold buckets (ordered write and coding in one pass) and then does all
     * the steps of the buckets on the dense passes with barriers between (force_dense: for all widths), and after it what that left uncoded */
    if (bits >= 16 && !c->force_dense) {
        const uint32_t fgrid = std::min(c->n_tiles, BAND_WG_PER_CU * (uint32_t)c->n_cu);
        if (c->K * 8u <= n && bits == 32) LAUNCHB(c, KID_HARD, st, k_band_few<32>, fgrid, BAND_T, residual, t, cd0, idx, val, c->d_flags);
        else if (c->K * 8u <= n) LAUNCHB(c, KID_HARD, st, k_band_few<16>, fgrid, BAND_T, residual, t, cd0, idx, val, c->d_flags);
        else if (bits == 32 && nt) LAUNCHB(c, KID_HARD, st, (k_band<32, true>), sgrid, BAND_T, residual, t, cd0, idx, val, c->d_flags);
        else if (bits == 32) LAUNCHB(c, KID_HARD, st, (k_band<32, false>), sgrid, BAND_T, residual, t, cd0, idx, val, c->d_flags);
        else if (nt) LAUNCHB(c, KID_HARD, st, (k_band<16, true>), sgrid, BAND_T, residual, t, cd0, idx, val, c->d_flags);
        else LAUNCHB(c, KID_HARD, st, (k_band<16, false>), sgrid, BAND_T, residual, t, cd0, idx, val, c->d_flags);
    } else {
        const uint32_t *cb_ = c->d_chunk_b, *cs_ = c->d_chunk_seg;
        const int stream_coding = c->chunk <= DENC_MAX_CHUNK ? 1 : 0;
#define NSML_HARD(BITS_, BIG_) LAUNCHB(c, KID_HARD, st, (k_hard<BITS_, BIG_>), hgrid, HTH, residual, t, cd0, h.f0, h.f1, h.f2, idx, c->d_v, val, scales, c->d_flags, stream_coding, team)
        switch (bits) {
        case 32: NSML_HARD(32, false); break;
        case 16: NSML_HARD(16, false); break;
        case 8:  if (big) NSML_HARD(8, true); else NSML_HARD(8, false); break;
        default: if (big) NSML_HARD(4, true); else NSML_HARD(4, false); break;
        }
#undef NSML_HARD
        const uint32_t qgrid = (uint32_t)c->NC, per_wg = (WG / 64) * QUANT_PER_WAVE;
        /* a chunk longer than a wavefront's per workgroup as long as that is not more than 16 for a compute unit (BERT-shaped gradient at 0.1,
         * 5496 chunks: 11.5 us, with eight 22.9), up to eight beyond (419 M elements at a half, 102400 of them: the round 2434 us,
         * with one each 2541) */
        const uint32_t big_per_wg = std::max(1u, std::min(QUANT_BIG_PER_WG, qgrid / (16u * (uint32_t)c->n_cu)));
        const uint32_t ngrid = c->chunk <= QUANT_WAVE_CHUNK ? (qgrid + per_wg - 1) / per_wg
                                                            : (qgrid + big_per_wg - 1) / big_per_wg;
        if (bits == 8) LAUNCH(c, KID_QUANT, st, k_quant<8>, ngrid, (const float *)c->d_v, (const uint32_t *)idx, t, cd0, residual, val, scales, cb_, cs_, c->NC, stream_coding);
        if (bits == 4) LAUNCH(c, KID_QUANT, st, k_quant<4>, ngrid, (const float *)c->d_v, (const uint32_t *)idx, t, cd0, residual, val, scales, cb_, cs_, c->NC, stream_coding);
    }
    c->have_l2 = true;
    c->have_prune = pruned || none_pruned;
    c->none_pruned = none_pruned;
    c->zero_clean = true;
    c->zero_B = B;
    return NSML_OK;
}

int nsml_compress(nsml_ctx *c, const float *grad, float *residual, uint64_t n,
                  const uint64_t *bucket_off, uint32_t B, double ratio, int bits,
                  uint32_t *idx, void *val, float *scales, void *stream)
{
    return compress_impl(c, grad, residual, nullptr, n, bucket_off, B, ratio, bits, idx, val, scales, stream);
}

int nsml_compress_pruned(nsml_ctx *c, const float *grad, float *residual, const float *weights,
                         uint64_t n, const uint64_t *bucket_off, uint32_t B, double ratio, int bits,
                         uint32_t *idx, void *val, float *scales, void *stream)
{
    if (!weights) return NSML_EINVAL;
    return compress_impl(c, grad, residual, weights, n, bucket_off, B, ratio, bits, idx, val, scales, stream);
}

}  // extern "C"

/* The launches of one decompress: tile-start table, then the dense output.  c may be NULL
 * (the entry point without a context): then nothing is profiled and no error code is kept. */
/* Up to one survivor in SCATTER_SHARE elements the dense output is zeroed and the survivors are stored
 * over the zeros. */
constexpr uint64_t SCATTER_SHARE = 512;
static bool decomp_by_scatter(int variant, uint64_t K, uint64_t n) { return variant > 0 || (variant < 0 && K * SCATTER_SHARE <= n); }
/* Workgroups of k_scatter for K survivors of n elements, and from which end.  Up to one survivor in eight
 * elements additions run from the last to the first, a block of 256 per workgroup: what a fill or the
 * addition before wrote last is still in the 256 MB cache (a fill and four payloads of 1.1 M into 110 M
 * elements, 8-bit codes: 57.2 us per payload, from the front 58.6; of 3.3 M: 96.9 and 98.5).  From there to one
 * in four from the front (84 M into 419 M: 778 us, from the back 805, in a loop 824).  Beyond that nearly every
 * line is touched and what counts is the order of the payload's reads: 8192 workgroups that walk it together
 * (all of 110 M: 448 us, a block per workgroup 594 from the front and 653 from the back, 32768 workgroups 468;
 * half of 34 M, 32-bit values: 89, 106, 129, 97). */
struct ScatterGrid { uint32_t grid; bool backward; };
static ScatterGrid scatter_grid(uint64_t K, uint64_t n, bool add)
{
    const uint64_t blocks = (K + WG - 1) / WG, most = add && K * 4u > n ? 8192u : 1u << 23;      /* (2^32 threads cannot be launched) */
    return {(uint32_t)std::min(blocks, most), add && K * 8u <= n};
}
/* Whether the decoder's workgroups look for their tile's survivors themselves (tilestart_wave), and no table is
 * made beforehand: its launch costs more than that as long as few tiles, or few survivors, are in the way of each other's
 * looks (a worker's round, us, with table / without: 60 Ki elements 22.6 / 18.4, ResNet-50 at 5 % 157 / 151, at 40 % 206 / 197; 110 M in
 * 250 buckets at 1 % 428 / 407, but at 10 % 646 / 656, the BERT-shaped gradient's rows at 10 % 647 / 675; 419 M at 1 % 1445 / 1535, at a half
 * 2453 / 2472). */
static bool decomp_searches(uint64_t K, uint64_t n, uint32_t n_tiles) { return n_tiles <= 16384u || (n_tiles <= 65536u && K * 64u <= n); }
static bool tilestart_by_search(uint64_t K, uint32_t n_tiles) { return K >= 32ull * n_tiles; }      /* many survivors per tile */
template <typename MAP>
static int launch_decompress(nsml_ctx *c, hipStream_t st, const Tables &t, uint64_t n, uint64_t K, const MAP *tile_b, uint32_t *d_ts,
                             const uint32_t *idx, const void *val, const float *scales, int bits, float *dense_out, int variant, int nt_zero, bool starts_done = false)
{
    const uint32_t n_tiles = t.n_tiles;
    if (decomp_by_scatter(variant, K, n)) {
        /* few survivors: zeros at the speed of a fill, then the survivors stored over them */
        const dim3 zgrid = xcd_grid((n + ZERO_T * 4 - 1) / (ZERO_T * 4));
        if (nt_zero < 0 ? n > NT_ELEMS : nt_zero != 0) LAUNCHB(c, KID_DECOMP, st, k_zero<true>, zgrid, ZERO_T, dense_out, n);
        else LAUNCHB(c, KID_DECOMP, st, k_zero<false>, zgrid, ZERO_T, dense_out, n);
        const ScatterGrid sg = scatter_grid(K, n, false);
        switch (bits) {
        case 32: LAUNCH(c, KID_DECOMP, st, (k_scatter<32, false, false>), sg.grid, idx, val, scales, t, K, dense_out); break;
        case 16: LAUNCH(c, KID_DECOMP, st, (k_scatter<16, false, false>), sg.grid, idx, val, scales, t, K, dense_out); break;
        case 8:  LAUNCH(c, KID_DECOMP, st, (k_scatter<8, false, false>),  sg.grid, idx, val, scales, t, K, dense_out); break;
        default: LAUNCH(c, KID_DECOMP, st, (k_scatter<4, false, false>),  sg.grid, idx, val, scales, t, K, dense_out); break;
        }
        return NSML_OK;
    }
    const uint32_t *ts = d_ts;
    if (K == n || starts_done) {
        /* everything was sent: no index list is read; or made with the other tables (25.5 us for ResNet-50 at 1 %, with searches 27.8) */
    } else if (decomp_searches(K, n, n_tiles)) {
        ts = nullptr;
    } else if (tilestart_by_search(K, n_tiles)) {
        LAUNCH(c, KID_TILESTART, st, k_tilestart_search, (n_tiles + WG - 1) / WG, idx, t, n_tiles, d_ts);
    } else if (K >= (4ull << 20)) {
        const uint64_t want = (K + (uint64_t)WG * 8 - 1) / ((uint64_t)WG * 8);
        LAUNCH(c, KID_TILESTART, st, k_tilestart<8>, (uint32_t)(want < 16384 ? want : 16384), idx, t, K, d_ts);
    } else {
        const uint64_t want = (K + (uint64_t)WG * 2 - 1) / ((uint64_t)WG * 2);
        LAUNCH(c, KID_TILESTART, st, k_tilestart<2>, (uint32_t)want, idx, t, K, d_ts);
    }
    const dim3 grid = xcd_grid(n_tiles);
    /* Threads per tile.  Everything sent is a plain decode without a chain of dependent loads: whole values in the
     * streaming kernels' shape (419 M elements: 537 us with 512 threads, 575 with 128), narrower ones with more of
     * them per thread (8 bits: 393 us with 128 threads, 474 with 512; 16: 415 and 450; 4: 540 and 591).  Few
     * survivors decode faster with 256 threads than with 128 (419 M elements, 8 bits: ratio 0.01 239 us and 280,
     * 0.05 266 and 296, 0.2 533 and 465), but the compress call that follows in a worker's round then takes longer:
     * 200 tensors of 110 M, a whole round at 0.003 426 us with 256 and 439 with 128, at 0.01 450 and 451, at 0.05
     * 592 and 575; a BERT-shaped one at 0.01 429 and 411.  So 256 up to one in 128, in 64 where no cache holds the
     * output (419 M at 0.01, 200 tensors: decode 300 and 376, round 1514 and 1503), and for a receiver without a
     * context, who compresses nothing, up to one in eight (25.6 M at 0.01: 25.4 and 26.5), in 32 for whole values
     * (419 M at 0.05: 365 and 336). */
    const bool receiver = c == nullptr;
    const bool sparse = receiver ? K * (bits == 32 ? 32u : 8u) <= n : K * (n > (1ull << 27) ? 64u : 128u) <= n;
#define NSML_DECOMP1(BITS_, NTH_) LAUNCHB(c, KID_DECOMP, st, (k_decomp<BITS_, MAP, NTH_>), grid, NTH_, idx, val, scales, t, tile_b, ts, dense_out)
#define NSML_DECOMP(BITS_)                                      \
    do {                                                         \
        if (K != n && sparse) NSML_DECOMP1(BITS_, 256);          \
        else NSML_DECOMP1(BITS_, 128);                           \
    } while (0)
    switch (bits) {
    case 32: if (K == n) NSML_DECOMP1(32, STH); else NSML_DECOMP(32); break;
    case 16: NSML_DECOMP(16); break;
    case 8:  NSML_DECOMP(8); break;
    default: NSML_DECOMP(4); break;
    }
#undef NSML_DECOMP
#undef NSML_DECOMP1
    return NSML_OK;
}

extern "C" {

int nsml_decompress(nsml_ctx *c, const uint32_t *idx, const void *val, const float *scales,
                    uint64_t n, const uint64_t *bucket_off, uint32_t B, double ratio, int bits,
                    float *dense_out, void *stream)
{
    if (!c || !idx || !val || !dense_out) return NSML_EINVAL;
    if ((bits == 8 || bits == 4) && !scales) return NSML_EINVAL;
    if (!aligned(dense_out, 16) || !aligned(idx, 4) || !aligned(val, 4) || !aligned(scales, 4))
        return NSML_EINVAL;
    if (pending_internal_error(c)) return NSML_EINTERNAL;
    hipStream_t st = static_cast<hipStream_t>(stream);
    DeviceGuard guard(c->device);
    if (!guard.ok) { c->last_hip = (int)hipErrorInvalidDevice; return NSML_EHIP; }
    int rc = ensure_layout(c, n, bucket_off, B, st);
    if (rc) return rc;
    rc = ensure_tables(c, ratio, bits, st);
    if (rc) return rc;
    return launch_decompress<uint32_t>(c, st, tables_of(c), c->n, c->K, c->d_tile_b, c->d_ts, idx, val, scales, bits, dense_out, c->decomp_variant, c->nt_dense);
}

/* ---------------------------------------------------------------- no-allocation decompress */

}  // extern "C"

/* Scratch of nsml_decompress_static: the layout tables and the tile-start table of one call.
 * One copy per GPU, at its own address on each; host code never uses this name as a pointer,
 * only what hipGetSymbolAddress returns for the current device. */
static __device__ __align__(256) unsigned char scratch[NSML_STATIC_SCRATCH_BYTES];

namespace {

constexpr int STATIC_MAX_DEVICES = 64;
void *g_scratch_ptr[STATIC_MAX_DEVICES];        /* per device, resolved on the first call there */

constexpr uint32_t STATIC_B1 = NSML_STATIC_MAX_BUCKETS + 1;
constexpr uint64_t STATIC_MAX_TILES = NSML_STATIC_MAX_N / TILE + 2ull * NSML_STATIC_MAX_BUCKETS + 2;

struct StaticOffsets { uint64_t off[STATIC_B1]; };      /* travels as a kernel argument */

/* where each table sits inside the scratch array */
struct StaticScratch {
    uint64_t *off, *P, *V, *S, *C;
    uint32_t *tile0, *k, *kw, *ts;
    uint16_t *tile_b;
};
StaticScratch carve(void *base)
{
    StaticScratch m;
    uint64_t *q = static_cast<uint64_t *>(base);
    m.off = q; q += STATIC_B1;
    m.P = q; q += STATIC_B1;
    m.V = q; q += STATIC_B1;
    m.S = q; q += STATIC_B1;
    m.C = q; q += STATIC_B1;
    uint32_t *w = reinterpret_cast<uint32_t *>(q);
    m.tile0 = w; w += STATIC_B1 + 1;
    m.k = w; w += STATIC_B1 + 1;
    m.kw = w; w += STATIC_B1 + 1;
    m.ts = w; w += STATIC_MAX_TILES + STATIC_B1 + 1;
    m.tile_b = reinterpret_cast<uint16_t *>(w);
    return m;
}
static_assert(5 * STATIC_B1 * 8 + 3 * (STATIC_B1 + 1) * 4 + (STATIC_MAX_TILES + STATIC_B1 + 1) * 4 + STATIC_MAX_TILES * 2
                  <= NSML_STATIC_SCRATCH_BYTES, "scratch array too small for its tables");
static_assert(sizeof(StaticOffsets) <= 3072, "bucket offsets must fit the kernel argument block");

/* Everything the dense output of one call needs beside its payload: bucket tables and the tiles' prefix from
 * the offsets (handed over by value), the bucket of every tile, and where each tile's survivors start.  Each
 * workgroup makes the tables for itself in LDS and the first one stores them: one launch of 8.9 us
 * where the chain took four (14.4 + 5.7 + 3.7 + 5.6 us, 161 buckets of 25.6 M elements, 1 % sent).  walk, find: make the tile starts by one or the other method. */
__global__ __launch_bounds__(WG) void k_static_setup(StaticOffsets so, Tables t, uint64_t *__restrict__ off, uint32_t *__restrict__ tile0,
                                                     double ratio, int bits, uint16_t *__restrict__ tile_b,
                                                     const uint32_t *__restrict__ idx, uint64_t K, uint32_t *__restrict__ ts, bool walk, bool find)
{
    __shared__ uint64_t sOff[STATIC_B1], sP[STATIC_B1];
    __shared__ uint32_t sT[STATIC_B1], sK[STATIC_B1];
    const bool first = blockIdx.x == 0;
    setup_body<WG>(t.B, t.chunk, ratio, bits, [&](uint32_t b) { return so.off[b]; },
               [&](uint32_t b, uint64_t nb, uint64_t k, uint64_t P, uint64_t V, uint64_t C, uint64_t tile) {
                   sOff[b] = so.off[b]; sP[b] = P; sT[b] = (uint32_t)tile; sK[b] = (uint32_t)k;
                   if (first) {
                       setup_store(t, ratio, bits, b, nb, k, P, V, C);
                       off[b] = so.off[b];
                       tile0[b] = (uint32_t)tile;
                   }
               });
    wg_sync();
    Tables own = t;
    own.off = sOff; own.P = sP; own.tile0 = sT; own.k = sK;
    for (uint32_t g = blockIdx.x * WG + threadIdx.x; g < t.n_tiles; g += gridDim.x * WG) {
        tile_b[g] = (uint16_t)find_bucket<uint32_t>(sT, t.B, g);
        if (find) tilestart_find(idx, own, g, ts);
    }
    if (walk) tilestart_walk<2>(idx, own, sP, K, ts);
}

}  // namespace

extern "C" {

int nsml_decompress_static(const uint32_t *idx, const void *val, const float *scales, uint64_t n,
                           const uint64_t *bucket_off, uint32_t B, double ratio, int bits,
                           uint32_t chunk, float *dense_out, void *stream)
{
    if (!idx || !val || !dense_out || !bucket_off || B == 0 || n == 0) return NSML_EINVAL;
    if ((bits == 8 || bits == 4) && !scales) return NSML_EINVAL;
    if (!aligned(dense_out, 16) || !aligned(idx, 4) || !aligned(val, 4) || !aligned(scales, 4))
        return NSML_EINVAL;
    if (B > NSML_STATIC_MAX_BUCKETS || n > NSML_STATIC_MAX_N) return NSML_ECAP;
    if (bucket_off[0] != 0 || bucket_off[B] != n) return NSML_EINVAL;
    uint64_t K = 0;
    int rc = nsml_payload_layout(bucket_off, B, ratio, bits, chunk, nullptr, &K, nullptr, nullptr);
    if (rc) return rc;                      /* also rejects descending offsets, bad ratio / bits / chunk */
    /* the same geometry a context would build, computed without any table on the host */
    uint64_t nt = 0;
    StaticOffsets so;
    for (uint32_t b = 0; b < B; ++b) {
        const uint64_t lo = bucket_off[b], hi = bucket_off[b + 1];
        if (hi > lo) nt += (hi - (lo & ~3ull) + TILE - 1) / TILE;
        so.off[b] = lo;
    }
    if (nt > STATIC_MAX_TILES) return NSML_ECAP;
    so.off[B] = n;
    for (uint32_t b = B + 1; b < STATIC_B1; ++b) so.off[b] = n;

    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= STATIC_MAX_DEVICES) return NSML_EHIP;
    void *base = __atomic_load_n(&g_scratch_ptr[dev], __ATOMIC_ACQUIRE);
    if (!base) {
        /* this GPU's copy of the array; the symbol's own name is no device address on the host */
        if (hipGetSymbolAddress(&base, HIP_SYMBOL(scratch)) != hipSuccess || !base) return NSML_EHIP;
        __atomic_store_n(&g_scratch_ptr[dev], base, __ATOMIC_RELEASE);
    }
    const StaticScratch m = carve(base);
    hipStream_t st = static_cast<hipStream_t>(stream);
    nsml_ctx *none = nullptr;

    Tables t;
    memset(&t, 0, sizeof t);
    t.off = m.off; t.tile0 = m.tile0;
    t.k = m.k; t.kw = m.kw; t.P = m.P; t.V = m.V; t.S = m.S; t.C = m.C;
    t.B = B; t.n_tiles = (uint32_t)nt; t.chunk = chunk; t.chunkSh = chunk_shift(chunk);
    const bool starts = K != n && !decomp_by_scatter(-1, K, n);
    const bool find = starts && tilestart_by_search(K, (uint32_t)nt), walk = starts && !find;
    const uint64_t tgrid = (nt + WG - 1) / WG, wgrid = walk ? (K + WG * 2 - 1) / (WG * 2) : 1u;
    LAUNCH(none, KID_SETUP, st, k_static_setup, (uint32_t)std::min<uint64_t>(1024, std::max(tgrid, wgrid)), so, t, m.off, m.tile0, ratio, bits, m.tile_b,
           idx, K, m.ts, walk, find);
    return launch_decompress<uint16_t>(none, st, t, n, K, m.tile_b, m.ts, idx, val, scales, bits, dense_out, -1, -1, true);
}

int nsml_decompress_accumulate(nsml_ctx *c, const uint32_t *idx, const void *val, const float *scales,
                               uint64_t n, const uint64_t *bucket_off, uint32_t B, double ratio,
                               int bits, float *dense_inout, void *stream)
{
    if (!c || !idx || !val || !dense_inout) return NSML_EINVAL;
    if ((bits == 8 || bits == 4) && !scales) return NSML_EINVAL;
    if (!aligned(dense_inout, 16) || !aligned(idx, 4) || !aligned(val, 4) || !aligned(scales, 4))
        return NSML_EINVAL;
    if (pending_internal_error(c)) return NSML_EINTERNAL;
    hipStream_t st = static_cast<hipStream_t>(stream);
    DeviceGuard guard(c->device);
    if (!guard.ok) { c->last_hip = (int)hipErrorInvalidDevice; return NSML_EHIP; }
    int rc = ensure_layout(c, n, bucket_off, B, st);
    if (rc) return rc;
    rc = ensure_tables(c, ratio, bits, st);
    if (rc) return rc;
    const Tables t = tables_of(c);
    const ScatterGrid sg = scatter_grid(c->K, c->n, true);
#define NSML_ACC(BITS_)                                                                                                                     \
    do {                                                                                                                                     \
        if (sg.backward) LAUNCH(c, KID_DECOMP_ACC, st, (k_scatter<BITS_, true, true>), sg.grid, idx, val, scales, t, c->K, dense_inout);      \
        else LAUNCH(c, KID_DECOMP_ACC, st, (k_scatter<BITS_, true, false>), sg.grid, idx, val, scales, t, c->K, dense_inout);                 \
    } while (0)
    switch (bits) {
    case 32: NSML_ACC(32); break;
    case 16: NSML_ACC(16); break;
    case 8:  NSML_ACC(8); break;
    default: NSML_ACC(4); break;
    }
#undef NSML_ACC
    return NSML_OK;
}

int nsml_last_l2norm(nsml_ctx *c, double *total, double *per_bucket)
{
    if (!c || !total) return NSML_EINVAL;
    *total = 0.0;
    if (!c->have_l2 || c->B == 0) return NSML_EINVAL;
    DeviceGuard guard(c->device);
    NSML_HIP(c, hipDeviceSynchronize());
    std::vector<double> sq(c->B);
    NSML_HIP(c, hipMemcpy(sq.data(), c->d_l2sq, sizeof(double) * c->B, hipMemcpyDeviceToHost));
    double sum = 0.0;
    for (uint32_t b = 0; b < c->B; ++b) {
        const double v = c->h_off[b + 1] > c->h_off[b] ? sq[b] : 0.0;
        sum += v;
        if (per_bucket) per_bucket[b] = sqrt(v);
    }
    *total = sqrt(sum);
    return NSML_OK;
}

int nsml_profile_enable(nsml_ctx *c, int on)
{
    if (!c) return NSML_EINVAL;
    c->prof = on != 0;
    return NSML_OK;
}

int nsml_profile_read(nsml_ctx *c, uint32_t *launches, double *total_ms)
{
    if (!c || !launches || !total_ms) return NSML_EINVAL;
    DeviceGuard guard(c->device);
    for (int i = 0; i < NSML_MAX_KERNELS; ++i) { launches[i] = 0; total_ms[i] = 0.0; }
    int rc = NSML_OK;
    for (auto &r : c->recs) {
        float ms = 0.f;
        hipError_t e = hipEventSynchronize(r.b);
        if (e == hipSuccess) e = hipEventElapsedTime(&ms, r.a, r.b);
        if (e != hipSuccess) { c->last_hip = (int)e; rc = NSML_EHIP; }
        else { launches[r.kid] += 1; total_ms[r.kid] += (double)ms; }
        c->pool.push_back(r.a); c->pool.push_back(r.b);
    }
    c->recs.clear();
    return rc;
}

int nsml_path_stats(nsml_ctx *c, uint32_t *fast_buckets, uint32_t *fallback_buckets)
{
    if (!c || !fast_buckets || !fallback_buckets) return NSML_EINVAL;
    *fast_buckets = *fallback_buckets = 0;
    if (c->B == 0) return NSML_OK;
    DeviceGuard guard(c->device);
    NSML_HIP(c, hipDeviceSynchronize());
    std::vector<uint32_t> f(c->B);
    NSML_HIP(c, hipMemcpy(f.data(), c->d_fast, sizeof(uint32_t) * c->B, hipMemcpyDeviceToHost));
    for (uint32_t b = 0; b < c->B; ++b) {
        if (c->h_off[b + 1] == c->h_off[b]) continue;
        if (f[b]) *fast_buckets += 1; else *fallback_buckets += 1;
    }
    return *(volatile uint32_t *)&c->h_flags[0] ? NSML_EINTERNAL : NSML_OK;
}

int nsml_bucket_state(nsml_ctx *c, uint32_t b, uint32_t *out8)
{
    if (!c || !out8 || b >= c->B) return NSML_EINVAL;
    DeviceGuard guard(c->device);
    NSML_HIP(c, hipDeviceSynchronize());
    const uint32_t *par = reinterpret_cast<const uint32_t *>(c->d_par + b);
    const uint32_t *src[8] = {c->d_fast + b, c->d_why + b, par, par + 1, c->d_T + b, c->d_need + b, c->d_sh + b, c->d_k + b};
    for (int i = 0; i < 8; ++i)
        NSML_HIP(c, hipMemcpy(out8 + i, src[i], sizeof(uint32_t), hipMemcpyDeviceToHost));
    return NSML_OK;
}

int nsml_prune_stats(nsml_ctx *c, uint32_t *band_buckets, uint32_t *dense_buckets)
{
    if (!c || !band_buckets || !dense_buckets) return NSML_EINVAL;
    *band_buckets = *dense_buckets = 0;
    if (c->B == 0 || !c->have_prune) return NSML_OK;
    DeviceGuard guard(c->device);
    NSML_HIP(c, hipDeviceSynchronize());
    std::vector<uint32_t> f(c->B);
    NSML_HIP(c, hipMemcpy(f.data(), c->d_wfast, sizeof(uint32_t) * c->B, hipMemcpyDeviceToHost));
    for (uint32_t b = 0; b < c->B; ++b) {
        if (c->h_off[b + 1] == c->h_off[b]) continue;
        if (c->none_pruned || f[b]) *band_buckets += 1; else *dense_buckets += 1;
    }
    return *(volatile uint32_t *)&c->h_flags[1] ? NSML_EINTERNAL : NSML_OK;
}

int nsml_calibration_copy(const void *src, void *dst, uint64_t bytes, void *stream)
{
    if (!src || !dst || bytes == 0 || bytes % 16 != 0 || !aligned(src, 16) || !aligned(dst, 16))
        return NSML_EINVAL;
    const uint64_t n16 = bytes / 16;
    const uint64_t want = (n16 + WG - 1) / WG;
    const uint32_t grid = (uint32_t)(want < 65536 ? want : 65536);
    hipLaunchKernelGGL(k_calib_copy, dim3(grid), dim3(WG), 0, static_cast<hipStream_t>(stream),
                       static_cast<const f4 *>(src), static_cast<f4 *>(dst), n16);
    return hipGetLastError() == hipSuccess ? NSML_OK : NSML_EHIP;
}

int nsml_set_option(nsml_ctx *c, const char *name, int value)
{
    if (!c || !name) return NSML_EINVAL;
    auto is = [&](const char *s) { return strcmp(name, s) == 0; };
    if (is("span_tiles")) {
        if (value < 0 || value > 16) return NSML_EINVAL;
        c->unit_tiles = value;
    } else if (is("seg_waves")) {
        if (value != 0 && value != 4 && value != 8 && value != 16) return NSML_EINVAL;
        c->sel_waves = value;
    } else if (is("nt")) {
        if (value != 1 && value != 3 && value != 5 && value != 7) return NSML_EINVAL;
        c->nt_acc = (value & 4) != 0;
    } else if (is("nt_dense")) {
        if (value < -1 || value > 1) return NSML_EINVAL;
        c->nt_dense = value;
    } else if (is("persist")) {                /* accepted, without effect: a workgroup takes one tile */
        if (value < 0 || value > 8) return NSML_EINVAL;
    } else if (is("decomp_variant")) {
        if (value < -1 || value > 1) return NSML_EINVAL;
        c->decomp_variant = value;
    } else if (is("force_dense")) {
        if (value != 0 && value != 1) return NSML_EINVAL;
        c->force_dense = value;
    } else if (is("rescan")) {
        if (value != 0 && value != 1) return NSML_EINVAL;
        c->force_rescan = value;
    } else if (is("whistory")) {
        if (value != 0 && value != 1) return NSML_EINVAL;
        c->whistory = value;
    } else if (is("wfix_apart")) {
        if (value < -1 || value > 1) return NSML_EINVAL;
        c->wfix_apart = value;
    } else if (is("wband_miss")) {
        if (value != 0 && value != 1) return NSML_EINVAL;
        c->wband_miss = value;
    } else if (is("trip_check")) {
        if (value != 1) return NSML_EINVAL;
        *(volatile uint32_t *)&c->h_flags[0] = 1u;
    } else {
        return NSML_EINVAL;
    }
    return NSML_OK;
}

int nsml_calibration_stream(int mode, const void *a, void *b, uint64_t bytes, int nontemporal, void *stream)
{
    constexpr uint64_t PER_WG = 16ull * 16384ull;      /* 16 wavefronts x 16 KiB */
    if (!a || !b || bytes == 0 || bytes % PER_WG != 0 || !aligned(a, 16) || !aligned(b, 16)) return NSML_EINVAL;
    if (mode < 0 || mode > 3) return NSML_EINVAL;
    const uint64_t wgs = bytes / PER_WG;
    if (wgs > 0x7FFFFFFFull) return NSML_ECAP;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const f4 *pa = static_cast<const f4 *>(a);
    f4 *pb = static_cast<f4 *>(b);
    const dim3 grid((uint32_t)wgs), block(1024);
    switch (mode * 2 + (nontemporal ? 1 : 0)) {
    case 0: hipLaunchKernelGGL((k_calib_read<false>), grid, block, 0, st, pa, pb); break;
    case 1: hipLaunchKernelGGL((k_calib_read<true>), grid, block, 0, st, pa, pb); break;
    case 2: hipLaunchKernelGGL((k_calib_fill<false>), grid, block, 0, st, pb); break;
    case 3: hipLaunchKernelGGL((k_calib_fill<true>), grid, block, 0, st, pb); break;
    case 4: hipLaunchKernelGGL((k_calib_add<false>), grid, block, 0, st, pa, pb); break;
    case 5: hipLaunchKernelGGL((k_calib_add<true>), grid, block, 0, st, pa, pb); break;
    case 6: hipLaunchKernelGGL((k_calib_copy2<false>), grid, block, 0, st, pa, pb); break;
    default: hipLaunchKernelGGL((k_calib_copy2<true>), grid, block, 0, st, pa, pb); break;
    }
    return hipGetLastError() == hipSuccess ? NSML_OK : NSML_EHIP;
}

const char *nsml_kernel_name(int id) { return (id >= 0 && id < KID_N) ? kKernelNames[id] : nullptr; }

}  // extern "C"
