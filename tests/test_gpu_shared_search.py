"""Searches shared by the lanes of a wave.

Once a wave has no pair left to start, its free lanes take pending siblings of
the searches that go on. The counting call visits the same nodes one after
another and never shares, so every result of a plain call has to equal the
counting call's bit for bit: searches of hundreds of nodes (random walks and
degenerate curves at depth 22), every edge of a wave's share, batches and
candidate lists.
"""
import numpy as np
import pytest
import torch

from paper_1811_03374_amd import binding
from paper_1811_03374_amd import workloads as W

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def g(a):
    return None if a is None else torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


def same(a, b):
    return all(torch.equal(x.view(torch.int32) if x.dtype == torch.float32 else x,
                           y.view(torch.int32) if y.dtype == torch.float32 else y) for x, y in zip(a, b))


@pytest.fixture(scope="module")
def long_searches():
    """Pairs of both recipes whose searches visit more than 32 nodes, in turn
    with short ones."""
    m, d = W.straight_and_curved(1 << 18), W.degenerate_geometry(1 << 18)
    R, F = np.concatenate([m.rays, d.rays], 1), np.concatenate([m.fibers, d.fibers], 1)
    tests = binding.intersect_pairs(g(R), g(F), 22, counts=True)[3][:, 0].cpu().numpy()
    long, short = np.nonzero(tests > 32)[0], np.nonzero(tests < 16)[0]
    assert long.size > 200 and tests.max() > 100
    n = min(long.size, 2000)
    i = np.empty(2 * n, np.int64)
    i[0::2], i[1::2] = long[:n], short[:n]
    return R[:, i], F[:, i]


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 129, 400])
@pytest.mark.parametrize("depth", [0, 9, 22])
def test_plain_equals_counting(long_searches, n, depth):
    R, F = (g(x)[:, :n] for x in long_searches)
    a = binding.intersect_pairs(R, F, depth)
    b = binding.intersect_pairs(R, F, depth, counts=True)
    assert same(a, b[:3])


def test_whole_recipes_equal_counting():
    for w in (W.straight_and_curved(1 << 17), W.degenerate_geometry(1 << 17)):
        R, F, pd = g(w.rays), g(w.fibers), g(w.pair_depth)
        assert same(binding.intersect_pairs(R, F, 22, pair_depth=pd),
                    binding.intersect_pairs(R, F, 22, pair_depth=pd, counts=True)[:3])
    w = W.quadratic_fibers(1 << 17)
    R, F = g(w.rays), g(w.fibers)
    assert same(binding.intersect_pairs(R, F, 22, quadratic=True),
                binding.intersect_pairs(R, F, 22, quadratic=True, counts=True)[:3])


def test_normals_batches_and_lists(long_searches):
    """The normal, the scene and the candidate of a shared search: batched
    scenes and one-candidate lists against the plain call, and the plain
    call's normals against those of the same pairs in another order (other
    waves, other helpers)."""
    R, F = (g(x) for x in long_searches)
    n = R.shape[1]
    t, u, h, nrm = binding.intersect_pairs(R, F, 22, normal=True)
    assert same((t, u, h), binding.intersect_pairs(R, F, 22, counts=True)[:3])
    back = torch.arange(n - 1, -1, -1, device=DEV, dtype=torch.int32)
    other = binding.intersect_pairs(R, F, 22, back, back, normal=True)
    assert same((t, u, h), [x.flip(0) for x in other[:3]]) and same([nrm], [other[3].flip(1).contiguous()])
    cuts = [0, 1, 64, 190, 191, 500, n]
    probs = [binding.Problem(R[:, a:b].contiguous(), F[:, a:b].contiguous(), 22, normal=True)
             for a, b in zip(cuts, cuts[1:])]
    binding.intersect_batched(probs)
    for p, a, b in zip(probs, cuts, cuts[1:]):
        assert same((p.t, p.u, p.hit, p.normal), (t[a:b], u[a:b], h[a:b], nrm[:, a:b].contiguous()))
    off = torch.arange(n + 1, device=DEV)
    c = binding.intersect_candidates(R, F, off, torch.arange(n, device=DEV, dtype=torch.int32), 22,
                                     max_candidates=1, normal=True)
    assert same((c[0], c[1], c[2], c[4]), (t, u, h, nrm))


@pytest.mark.parametrize("n", [1 << 16, (1 << 16) + 1, 1 << 19, (1 << 19) + 1])
def test_limits_of_call_sizes(n):
    """Either side of the sizes at which waves wait longer before they share."""
    w = W.straight_and_curved(n + (n & 1))
    R, F = g(w.rays)[:, :n], g(w.fibers)[:, :n]
    assert same(binding.intersect_pairs(R, F, 22), binding.intersect_pairs(R, F, 22, counts=True)[:3])
