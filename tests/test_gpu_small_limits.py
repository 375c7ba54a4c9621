"""What happens at limits that only large calls meet, in a library built with
them set small: a node stack of 64 entries in the waves of pre-subdivision
(nodes without room are walked by their lane alone, which decides by the whole
search what a wave decides by bounds, samples and shared searches), and three
candidates of a list in a launch (further launches go on from the nearest hit).
Every output has to equal the usual library's bit for bit.
"""
import os

import numpy as np
import pytest
import torch

from paper_1811_03374_amd import binding, build_lib
from paper_1811_03374_amd import workloads as W

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module")
def both():
    """both(call): the call's result from the usual and the small library."""
    if not os.path.exists(build_lib.LIB_SMALL):
        build_lib.build_small()
    usual, usual_path = binding.lib(), build_lib.LIB
    try:
        binding._lib, build_lib.LIB = None, build_lib.LIB_SMALL
        small = binding.lib()
    finally:
        binding._lib, build_lib.LIB = usual, usual_path

    def run(call):
        a = call()
        torch.cuda.synchronize()
        try:
            binding._lib = small
            b = call()
            torch.cuda.synchronize()
        finally:
            binding._lib = usual
        return a, b
    return run


def equal(a, b):
    bits = {torch.float32: torch.int32, torch.float64: torch.int64}
    return len(a) == len(b) and all(
        x.shape == y.shape and torch.equal(x.contiguous().view(bits.get(x.dtype, x.dtype)),
                                           y.contiguous().view(bits.get(y.dtype, y.dtype))) for x, y in zip(a, b))


def deep(n):
    """Degenerate and bent curves in turn: cusps and thick ends, whose trees
    go down to the level limit."""
    d, m = W.degenerate_geometry(-(-n // 4) * 4).fibers, W.straight_and_curved(2 * n).fibers[:, 1::2]
    return np.stack([d[:, :n], m[:, :n]], 2).reshape(16, -1)[:, :n].copy()


@pytest.mark.parametrize("level", [1, 6, 10])
@pytest.mark.parametrize("n", [1, 16, 64, 3001, (1 << 15) + 65])        # 16 and 64 fibers a wave
def test_full_node_stack(both, n, level):
    f = deep(n)
    f[3::4, ::7] *= 20.0                                               # thick
    f = torch.from_numpy(f).to(DEV)
    a, b = both(lambda: binding.presplit(f, level))
    if n > 1 << 15:
        # a wave takes 64 roots at once and has room for the halves of 32 of
        # them: more break an inequality, so that the rest are walked alone
        halved = ((binding.validate(f) & 31) != 0)[:n // 64 * 64].view(-1, 64).sum(1)
        assert int((halved > 32).sum()) > 100
    assert equal(a, b)


@pytest.mark.parametrize("most", [0, 1, 2, 3, 4, 6, 7, 40])
@pytest.mark.parametrize("refine", [False, True])
def test_lists_over_several_launches(both, most, refine):
    w = W.straight_and_curved(1 << 13)
    rng = np.random.default_rng(most)
    n = 5001
    length = np.where(rng.random(n) < 0.1, 31, rng.integers(0, 9, n))
    off = np.concatenate([[0], np.cumsum(length)])
    own = np.repeat(np.arange(n), length)
    cand = np.where(rng.random(own.size) < 0.4, own, rng.integers(0, 1 << 13, own.size)).astype(np.int32)
    R, F = torch.from_numpy(w.rays[:, :n].copy()).to(DEV), torch.from_numpy(w.fibers).to(DEV)
    off, cand = torch.from_numpy(off).to(DEV), torch.from_numpy(cand).to(DEV)
    a, b = both(lambda: binding.intersect_candidates(R, F, off, cand, 22, max_candidates=most, refine=refine,
                                                     normal=True))
    assert equal(a, b)
    assert most == 0 or int(a[2].sum()) > 100
