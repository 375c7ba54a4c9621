"""Searches that meet the trip limit.

Fibers of an extent near 1e-6 and below are searched in FP32 products that
underflow, and some of their pairs visit more than 65,536 nodes: such a pair is
a miss, in whatever call, and whether its search is shared by a wave's lanes or
not. The counting call never shares, so plain calls (alone, in another order,
batched, refined against itself) have to equal it bit for bit.
"""
import numpy as np
import pytest
import torch

from paper_1811_03374_amd import binding
from paper_1811_03374_amd import workloads as W

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
LIMIT = 1 << 16


def g(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


def pairs(n, scale, seed):
    """Circular arcs of radius `scale`, as thick as 1e-3 to 1 of it, half of
    them with a vanishing end tangent, and rays aimed at them."""
    rng = np.random.default_rng(seed)
    a = rng.uniform(0.05, 2.5, n)
    k = 4.0 / 3.0 * np.tan(a / 4.0)
    P = np.zeros((n, 4, 4))
    P[:, 0, 0] = P[:, 1, 0] = 1.0
    P[:, 1, 1] = k
    c, s = np.cos(a), np.sin(a)
    P[:, 2, 0], P[:, 2, 1], P[:, 3, 0], P[:, 3, 1] = c + k * s, s - k * c, c, s
    P[::2, 1] = P[::2, 0]
    P[:, :, 3] = (10.0 ** rng.uniform(-3.0, 0.0, n))[:, None]
    C, d = W.bernstein_point(P, rng.uniform(0.0, 1.0, n))[:, :3], W.unit_vectors(rng, n)
    t = C + (rng.standard_normal(n) * P[:, 0, 3])[:, None] * W.unit_vectors(rng, n)
    rays = W.pack_rays((t - 3.0 * d) * scale, d, np.full(n, 100.0))
    return g(rays), g(W.pack_fibers(P * scale))


def same(a, b):
    return all(torch.equal(x.contiguous().view(torch.int32) if x.dtype == torch.float32 else x,
                           y.contiguous().view(torch.int32) if y.dtype == torch.float32 else y) for x, y in zip(a, b))


@pytest.mark.parametrize("scale", [2.0 ** -24, 2.0 ** -20, 2.0 ** -16])
@pytest.mark.parametrize("n", [64, 4001, 70000])
def test_plain_equals_counting(n, scale):
    R, F = pairs(n, scale, 5)
    *want, counts = binding.intersect_pairs(R, F, 23, counts=True)
    if scale < 2.0 ** -18 and n > 4000:
        assert int((counts[:, 0] > LIMIT).sum()) > 2
    assert not bool(want[2][counts[:, 0] > LIMIT].any())
    assert same(binding.intersect_pairs(R, F, 23), want)


def test_other_neighbours_and_batches():
    n = 9000
    R, F = pairs(n, 2.0 ** -22, 6)
    t, u, h, nrm = binding.intersect_pairs(R, F, 23, normal=True)
    assert same((t, u, h), binding.intersect_pairs(R, F, 23, counts=True)[:3])
    order = torch.randperm(n, generator=torch.Generator().manual_seed(1)).to(DEV)
    i = order.to(torch.int32)
    b = binding.intersect_pairs(R, F, 23, i, i, normal=True)
    assert same((t[order], u[order], h[order], nrm[:, order]), b)
    cuts = [0, 1, 65, 4000, n]
    probs = [binding.Problem(R[:, a:b].contiguous(), F[:, a:b].contiguous(), 23, normal=True)
             for a, b in zip(cuts, cuts[1:])]
    binding.intersect_batched(probs)
    for p, a, b in zip(probs, cuts, cuts[1:]):
        assert same((p.t, p.u, p.hit, p.normal), (t[a:b], u[a:b], h[a:b], nrm[:, a:b]))


def test_refined_calls_do_not_depend_on_the_order():
    n = 9000
    R, F = pairs(n, 2.0 ** -22, 7)
    a = binding.intersect_pairs(R, F, 23, refine=True)
    order = torch.randperm(n, generator=torch.Generator().manual_seed(2)).to(DEV)
    i = order.to(torch.int32)
    b = binding.intersect_pairs(R, F, 23, i, i, refine=True)
    assert same([x[order].view(torch.int64) if x.dtype == torch.float64 else x[order] for x in a],
                [x.view(torch.int64) if x.dtype == torch.float64 else x for x in b])
