"""GPU parity at the edges of the rules that choose a launch by size: bit for bit against the oracle,
or against torch's own indexed store where only the decoder is asked."""
import numpy as np
import pytest
import torch

import oracle
from paper_2506_16235_amd import binding as nsml
from paper_2506_16235_amd import workloads as W
from gpu_util import DEV, Case, compare_payload, say

pytestmark = pytest.mark.gpu


def _rand(n, seed, sigma=1e-3):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return torch.randn(n, generator=g, device=DEV) * sigma


PER_CU = torch.cuda.get_device_properties(0).multi_processor_count if torch.cuda.is_available() else 256


@pytest.mark.parametrize("sizes", [
    [8191, 1, 8192, 8193, 0, 16383, 16385, 2, 32765, 5, 65537],
    [262143, 3, 262144, 262145],
    [(1 << 22) - 1], [1 << 22], [1, (1 << 22) + 1],
    [40_001] + [90] * (4 * PER_CU - 1), [40_001] + [90] * (4 * PER_CU),
], ids=["sample", "stride", "below", "limit", "above", "buckets", "buckets+1"])
def test_sample_and_prediction_in_one_launch(sizes):
    """Buckets around the elements a workgroup samples, odd starts, the largest bucket and the most buckets that
    are sampled and predicted in one launch and the next size up; three ratios in turn, so that the tables are made
    anew by that launch too, then a pruned call and one at the first ratio."""
    off = W.offsets_of(sizes)
    n = int(off[-1])
    say("sample", n, len(sizes))
    c = Case(_rand(n, n & 1023), off, chunk=256)
    c.g[: n // 5] = 0.0
    c.set_grad(c.g)
    c.step(0.02, 8)
    c.step(0.2, 4)
    w = _rand(n, 7)
    idx, val, sc = c.ctx.compress_pruned(c.g, c.r, w, off, 0.003, 8)
    torch.cuda.synchronize()
    want = oracle.compress_pruned(c.g_host, c.r_host, w.cpu().numpy(), off, 0.003, 8, 256, nthreads=8)
    _, K, vb, ns = oracle.layout(off, 0.003, 8, 256)
    compare_payload(off, 0.003, 8, 256, (idx.cpu().numpy().view(np.uint32)[:K], val.cpu().numpy()[:vb], sc.cpu().numpy()[:ns]), want)
    assert np.array_equal(c.r.cpu().numpy().view(np.uint32), c.r_host.view(np.uint32))
    c.step(0.02, 16)


@pytest.mark.parametrize("pruned", [False, True])
@pytest.mark.parametrize("ratio", [0.1, 0.2, 0.3, 0.5])
def test_one_magnitude_in_small_buckets_of_the_chain(ratio, pruned):
    """Buckets of under 16384 elements beside one that is too large for a single launch, whose last wavefront has
    1, 2, 5, 10 or 15 runs of 16 to sample: one magnitude (or zeros) and 16 to 240 larger values at the end, so that more
    elements share a digit than can be staged and the dense passes go on from the sample's counts."""
    sizes = [40_000, 8208, 7840, 4112, 8192 + 80, 16 * 175, 16_368, 32, 12_304]
    larger = [16, 16, 32, 16, 80, 240, 160, 16, 16]
    off = W.offsets_of(sizes)
    n = int(off[-1])
    rng = np.random.default_rng(int(ratio * 10) + pruned)
    g_h = np.where(rng.random(n) < 0.5, -1e-3, 1e-3).astype(np.float32)
    for b, m in enumerate(larger):
        g_h[int(off[b + 1]) - m:int(off[b + 1])] *= 2
    g_h[int(off[8]):int(off[9]) - 16] = 0.0
    c = Case(torch.from_numpy(g_h).to(DEV), off, chunk=256)
    if not pruned:
        for bits in (4, 8, 16, 32):
            c.set_residual(np.zeros(n))
            c.step(ratio, bits)
        return
    w = _rand(n, 5)
    for bits in (4, 8, 16, 32):
        c.set_residual(np.zeros(n))
        idx, val, sc = c.ctx.compress_pruned(c.g, c.r, w, off, ratio, bits)
        torch.cuda.synchronize()
        c.ctx.path_stats()
        want = oracle.compress_pruned(c.g_host, c.r_host, w.cpu().numpy(), off, ratio, bits, 256, nthreads=8)
        _, K, vb, ns = oracle.layout(off, ratio, bits, 256)
        compare_payload(off, ratio, bits, 256, (idx.cpu().numpy().view(np.uint32)[:K], val.cpu().numpy()[:vb], sc.cpu().numpy()[:ns]), want)
        assert np.array_equal(c.r.cpu().numpy().view(np.uint32), c.r_host.view(np.uint32))


@pytest.mark.parametrize("sizes", [[16_384, 40_003, 100_001], [262_143, 1], [262_144, 16_385], [1_000_003, 60_001], [(1 << 22) - 1]],
                         ids=lambda s: str(max(s)))
@pytest.mark.parametrize("values", ["clipped", "two"])
def test_buckets_sampled_a_second_time(sizes, values):
    """Large groups of equal values near the threshold, of which the small sample leaves nothing to stage: the whole
    bucket is sampled then (up to 262143 elements), or as much of a larger one as when buckets are many.  Plain rounds with
    error feedback, then a pruned call."""
    off = W.offsets_of(sizes)
    n = int(off[-1])
    say("again", n, len(sizes), values)
    g = _rand(n, n & 1023)
    g = g.clamp(-1e-3, 1e-3) if values == "clipped" else torch.where(g.abs() < 6e-4, 1e-3, 2e-3) * torch.sign(g)
    c = Case(g, off, chunk=2048)
    for ratio, bits in ((0.4, 32), (0.38, 8), (0.5, 4), (0.1, 8)):
        c.step(ratio, bits)
    w = _rand(n, 9)
    idx, val, sc = c.ctx.compress_pruned(c.g, c.r, w, off, 0.4, 16)
    torch.cuda.synchronize()
    c.ctx.path_stats()
    want = oracle.compress_pruned(c.g_host, c.r_host, w.cpu().numpy(), off, 0.4, 16, 2048, nthreads=8)
    _, K, vb, ns = oracle.layout(off, 0.4, 16, 2048)
    compare_payload(off, 0.4, 16, 2048, (idx.cpu().numpy().view(np.uint32)[:K], val.cpu().numpy()[:vb], sc.cpu().numpy()[:ns]), want)
    assert np.array_equal(c.r.cpu().numpy().view(np.uint32), c.r_host.view(np.uint32))


@pytest.mark.parametrize("bits", [4, 8, 32])
@pytest.mark.parametrize("ratio", [0.09, 0.12, 0.125, 0.13, 0.3])
def test_more_chunks_than_workgroups_that_code_them(ratio, bits):
    """More chunks than the launch that codes staged survivors has workgroups, below and above a ratio of an eighth:
    chunks of other paths between them (a bucket of mostly zeros), buckets of a few survivors, a last short chunk."""
    sizes = [1_500_001, 300_000, 40_000] + [37] * 3000
    off = W.offsets_of(sizes)
    n = int(off[-1])
    g = _rand(n, 11)
    g[1_500_001:1_800_001].mul_((torch.arange(300_000, device=DEV) % 4096 < 300).float())
    c = Case(g, off, chunk=8)
    c.step(ratio, bits)
    c.step(ratio, bits)


@pytest.mark.parametrize("dense", [0, 1])
@pytest.mark.parametrize("n", [4_200_003, 4_400_003, 9_000_001])
def test_long_chunks_left_to_a_second_pass(monkeypatch, n, dense):
    """Chunks longer than a wavefront codes that the ordered pass leaves uncoded (those across its units, or all of them):
    about as many as make the second pass give a workgroup one (below 32 for every compute unit), two, and four."""
    monkeypatch.setitem(nsml.Context.default_options, "force_dense", dense)
    off = W.offsets_of([n - 70_001, 70_001])
    g = _rand(n, 13)
    g[: n // 3].mul_((torch.arange(n // 3, device=DEV) % 2048 < 700).float())
    c = Case(g, off, chunk=264)
    c.step(0.5, 8)
    c.step(0.499, 4)


@pytest.mark.parametrize("digits", [1, 2])
@pytest.mark.parametrize("close", [4095, 4096, 4097, 9000])
def test_undecided_keys_of_a_small_bucket(close, digits):
    """As many keys as the list of a bucket in one launch holds, one less and one more, that share the first digit of
    12 bits, or the second as well; the threshold among them, at their first, at their last, and at a group of equal ones."""
    n = 20_000
    rng = np.random.default_rng(close + digits)
    g_h = (rng.standard_normal(n) * 1e-3).astype(np.float32)
    at = rng.permutation(n)[:close]
    low = 19 if digits == 1 else 7                    # bits of a key below the digits that are the same
    keys = np.uint32(0x3F800000) + rng.integers(0, 1 << low, size=close).astype(np.uint32)
    g_h[at] = keys.view(np.float32) * np.where(rng.random(close) < 0.5, -1, 1).astype(np.float32)
    g_h[at[: close // 8]] = g_h[at[0]]                # a group of equal ones
    off = W.offsets_of([n])
    for k in (1, close // 3, close, close + 1):
        c = Case(torch.from_numpy(g_h).to(DEV), off, chunk=64)
        c.step((k - 0.5) / n, 8)


@pytest.mark.parametrize("share", [100, 50])
@pytest.mark.parametrize("tiles", [16384, 16385, 65536, 65537])
def test_tiles_that_look_for_their_survivors(tiles, share):
    """The decoder's tiles look for their survivors themselves up to a number of tiles and of survivors, and read a
    table beyond: both sides of each limit, two odd bucket starts, against an indexed store."""
    n = tiles * 2048 - 1
    off = W.offsets_of([1, n // 2, n - 1 - n // 2])
    ratio = 1.0 / share
    k_b, K, vb, ns = nsml.payload_layout(off, ratio, 32)
    say("decode", n, K)
    ctx = nsml.Context(n, len(off) - 1, 2048)
    ctx.set_option("decomp_variant", 0)
    lo = torch.zeros(K, dtype=torch.int64, device=DEV)
    idx = torch.zeros(K, dtype=torch.int64, device=DEV)
    p = 0
    for b, k in enumerate(int(k) for k in k_b):
        nb = int(off[b + 1] - off[b])
        idx[p:p + k] = (torch.arange(k, device=DEV, dtype=torch.int64) * nb) // k + (_rand(k, b).abs() * 1e3).long() % max(1, nb // k)
        lo[p:p + k] = int(off[b])
        p += k
    v = _rand(K, 3)
    out = torch.full((n,), 7.0, device=DEV)
    ctx.decompress(idx.to(torch.int32), v.view(torch.uint8), torch.zeros(1, device=DEV), n, off, ratio, 32, out)
    want = torch.zeros(n, device=DEV)
    want[idx + lo] = v
    assert torch.equal(out.view(torch.int32), want.view(torch.int32))
