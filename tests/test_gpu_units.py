"""Calls whose survivors are not all staged: buckets taken from the dense accumulator (by k_hard and k_quant, or as whole values tile by
tile) beside those that come from staged entries, bit for bit against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2506_16235_amd import workloads as W
from gpu_util import DEV, Case, compare_payload, say

pytestmark = pytest.mark.gpu

ELSEWHERE = 300_000      # elements of a second bucket that is decided from staged entries, and keeps the whole call below an eighth


def _signs(rng, n):
    return np.where(rng.random(n) < 0.5, -1.0, 1.0).astype(np.float32)


def _values(kind, n, rng):
    x = (rng.standard_normal(n) * 1e-5).astype(np.float32)
    if kind == "block":          # as many large values as survive, in one place: tiles of survivors only
        x[n // 3:n // 3 + n // 8] = (rng.standard_normal(n // 8) + 3.0).astype(np.float32)
    elif kind == "clusters":     # runs of large values: tiles of survivors only, others with none
        for at in range(0, n - 900, 9973):
            m = int(rng.integers(200, 900))
            x[at:at + m] = rng.standard_normal(m)
    elif kind == "zeros":        # fewer values than survivors: the first zeros survive as well
        keep = np.repeat(rng.random(-(-n // 768)) < 0.05, 768)[:n]
        x = (rng.standard_normal(n) * keep).astype(np.float32)
    elif kind == "ties":         # clusters of few magnitudes: ties begin and end inside a tile
        for at in range(0, n - 3000, 20011):
            x[at:at + 2500] = rng.integers(1, 3, 2500)
        x *= _signs(rng, n)
    else:                        # one magnitude: the dense passes
        x = _signs(rng, n)
    return x


@pytest.mark.parametrize("kind", ["block", "clusters", "zeros", "ties", "one"])
@pytest.mark.parametrize("bits,chunk", [(8, 2048), (4, 2048), (8, 256), (4, 8), (16, 64), (32, 1024)])
def test_units_of_survivors_not_staged(kind, bits, chunk):
    """Up to an eighth sent: tiles of survivors only, survivors in clusters and far apart, a last chunk of one survivor, chunks from
    8 to 2048; a bucket that starts beside a multiple of 4."""
    for seed, nb in ((1, 2048 * 128), (2, 300_007)):
        rng = np.random.default_rng([seed, bits, chunk])
        sizes = [ELSEWHERE + seed - 1, nb, ELSEWHERE]
        off = W.offsets_of(sizes)
        n = int(off[-1])
        g = (rng.standard_normal(n) * 1e-3).astype(np.float32)
        g[int(off[1]):int(off[2])] = _values(kind, nb, rng)
        for ratio in (0.125 if nb % 2048 == 0 else 0.12, (2048 * 9 + 0.5) / nb, 0.02):
            say(kind, bits, chunk, nb, ratio)
            c = Case(torch.from_numpy(g).to(DEV), off, chunk=chunk)
            c.step(ratio, bits)
            c.step(ratio, bits)


@pytest.mark.parametrize("kind", ["clusters", "ties", "one"])
def test_units_beside_pruned_parameters(kind):
    rng = np.random.default_rng(5)
    off = W.offsets_of([ELSEWHERE + 1, 250_003, ELSEWHERE])
    n = int(off[-1])
    g = (rng.standard_normal(n) * 1e-3).astype(np.float32)
    g[int(off[1]):int(off[2])] = _values(kind, 250_003, rng)
    w = rng.standard_normal(n).astype(np.float32)
    for bits in (8, 32):
        c = Case(torch.from_numpy(g).to(DEV), off)
        for ratio in (0.1, 0.03):
            say(kind, bits, ratio)
            idx, val, sc = c.ctx.compress_pruned(c.g, c.r, torch.from_numpy(w).to(DEV), off, ratio, bits)
            torch.cuda.synchronize()
            c.ctx.path_stats()
            want = oracle.compress_pruned(c.g_host, c.r_host, w, off, ratio, bits, 2048, nthreads=8)
            _, K, vb, ns = oracle.layout(off, ratio, bits, 2048)
            compare_payload(off, ratio, bits, 2048, (idx.cpu().numpy().view(np.uint32)[:K], val.cpu().numpy()[:vb], sc.cpu().numpy()[:ns]), want)
            assert np.array_equal(c.r.cpu().numpy().view(np.uint32), c.r_host.view(np.uint32))


@pytest.mark.parametrize("kind", ["normal", "block", "clusters", "zeros", "ties", "one"])
@pytest.mark.parametrize("bits,nt", [(32, 3), (16, 3), (32, 7), (16, 7)])
def test_whole_values_tile_by_tile(monkeypatch, kind, bits, nt):
    """16- and 32-bit values beyond an eighth: tiles without survivors, of survivors only, with fewer of them than lines are
    written whole for, ties that end inside a tile, a bucket's first and last tile; into the caches and past them."""
    from paper_2506_16235_amd import binding as nsml
    monkeypatch.setitem(nsml.Context.default_options, "nt", nt)
    for seed, lead in ((1, 40_000), (2, 40_003)):
        rng = np.random.default_rng([seed, bits])
        off = W.offsets_of([lead, 2048 * 40 + seed - 1, 5, 2049, 100_000])
        n = int(off[-1])
        g = (rng.standard_normal(n) * 1e-3).astype(np.float32)
        if kind != "normal":
            for b in (1, 3, 4):
                g[int(off[b]):int(off[b + 1])] = _values(kind, int(off[b + 1] - off[b]), rng)
        w = rng.standard_normal(n).astype(np.float32)
        for ratio in (0.126, 0.4, 0.93):
            say(kind, bits, nt, lead, ratio)
            c = Case(torch.from_numpy(g).to(DEV), off, chunk=24)
            c.step(ratio, bits)
            c.step(ratio, bits)
            idx, val, sc = c.ctx.compress_pruned(c.g, c.r, torch.from_numpy(w).to(DEV), off, ratio, bits)
            torch.cuda.synchronize()
            c.ctx.path_stats()
            want = oracle.compress_pruned(c.g_host, c.r_host, w, off, ratio, bits, 24, nthreads=8)
            _, K, vb, ns = oracle.layout(off, ratio, bits, 24)
            compare_payload(off, ratio, bits, 24, (idx.cpu().numpy().view(np.uint32)[:K], val.cpu().numpy()[:vb], sc.cpu().numpy()[:ns]), want)
            assert np.array_equal(c.r.cpu().numpy().view(np.uint32), c.r_host.view(np.uint32))
