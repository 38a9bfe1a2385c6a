"""Small buckets in one launch, where a lower bound of the threshold leaves a list of candidates: the sizes at which the
list is made another way, and values that make the bound or the bins miss; bit for bit against the oracle."""
import numpy as np
import pytest
import torch

from paper_2506_16235_amd import workloads as W
from gpu_util import DEV, Case, say

pytestmark = pytest.mark.gpu


def _values(kind, n, rng):
    x = rng.standard_normal(n).astype(np.float32)
    if kind == "tail":           # a few values far above the others: the bins above the bound are open
        x *= 1e-6
        m = max(1, n // 700)
        x[rng.choice(n, m, replace=False)] = (10.0 ** rng.uniform(-3, 30, m)).astype(np.float32)
    elif kind == "ties":         # more equal keys in a bin than are searched bit by bit
        x = np.round(x * 4).astype(np.float32) / 4
    elif kind == "close":        # keys that differ in their last bits
        x = ((0x3F800000 + rng.integers(0, 5000, n)).astype(np.uint32).view(np.float32) * np.sign(x)).astype(np.float32)
    elif kind == "rows":         # runs of values among zeros: as many as survive, more, fewer
        x *= np.repeat(rng.random(-(-n // 300)) < 0.15, 300)[:n]
    elif kind == "pairs":        # what is sampled (every fourth) is no sample
        x[::4] *= 1e-4
    elif kind == "nan":
        x[rng.choice(n, max(1, n // 300), replace=False)] = rng.choice(np.array([np.inf, -np.inf, np.nan], np.float32))
    return x


@pytest.mark.parametrize("kind", ["normal", "tail", "ties", "close", "rows", "pairs", "nan"])
@pytest.mark.parametrize("bits,chunk", [(4, 8), (4, 2048), (8, 8), (8, 2048), (16, 24), (32, 2048)])
def test_candidates_of_small_buckets(kind, bits, chunk):
    if kind == "nan" and bits <= 8:
        pytest.skip("the scale of a chunk with an infinity is not a number that codes can be made with")
    sizes = [4096, 4097, 1, 4093, 8184, 8188, 8189, 8193, 32764, 0, 16_411, 32_763, 20_000, 63, 5]
    off = W.offsets_of(sizes)
    n = int(off[-1])
    rng = np.random.default_rng([len(kind), bits, chunk])
    g = np.concatenate([_values(kind, s, rng) for s in sizes if s])
    for ratio in (0.001, 0.03, 0.125, 0.25, 0.26):
        say(kind, bits, chunk, ratio)
        c = Case(torch.from_numpy(g).to(DEV), off, chunk=chunk)
        c.step(ratio, bits)
        if kind != "nan":
            c.step(ratio, bits)


@pytest.mark.parametrize("bits,chunk", [(4, 64), (8, 2048), (16, 2048), (32, 2048)])
def test_a_digit_too_full_for_the_list(bits, chunk):
    """More keys share a digit than the list of candidates holds: the k-th key's digit, few and many keys in it, and one that only the sample
    takes for it; keys of one magnitude."""
    sizes = [32_000, 20_001, 32_764, 9_000, 4097]
    off = W.offsets_of(sizes)
    for kind in ("crowd", "off", "one", "two"):
        rng = np.random.default_rng([len(kind), bits])
        parts = []
        for nb in sizes:
            x = (rng.standard_normal(nb) * 1e-6).astype(np.float32)
            if kind == "one":
                x[:] = 0.25
            elif kind == "two":
                x = rng.choice(np.array([0.25, 0.5], np.float32), nb)
            else:
                above = rng.permutation(nb)[:int(0.12 * nb)]
                if kind == "off":        # not among every fourth element, which are what is sampled
                    above = np.flatnonzero(np.arange(nb) % 4)[:int(0.14 * nb)]
                rest = np.setdiff1d(np.arange(nb), above)
                if kind == "off":
                    x[rest] = rng.uniform(1.0, 1.03, len(rest))
                else:
                    x[rng.permutation(rest)[:int(0.1125 * nb)]] = rng.uniform(1.0, 1.03, int(0.1125 * nb))
                x[above] = 2.0 + np.abs(rng.standard_normal(len(above)))
            parts.append((x * np.where(rng.random(nb) < 0.5, -1, 1)).astype(np.float32))
        g = np.concatenate(parts)
        for ratio in (0.125, 0.01, 0.06):
            say(kind, bits, chunk, ratio)
            c = Case(torch.from_numpy(g).to(DEV), off, chunk=chunk)
            c.step(ratio, bits)
            c.step(ratio, bits)
