"""Refined pairs where the FP64 decision changes its way.

A pair is decided from the one closest point of a short, nearly straight piece
where the taper is mild, the piece bends little and the ray is not nearly in
the plane of the discs, and by the sampled search elsewhere. The families here
straddle those lines: tapers from none to steep, arcs from straight to strongly
bent, rays from 1e-3 rad off the curve to 1e-3 rad off its normal plane, hits
next to the ends. All against the exact swept-disc oracle.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_1811_03374_amd import binding
from paper_1811_03374_amd import workloads as W

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
# FP64 evaluation rounds at 2^-52 of coordinates of about 3; a ray 1e-3 rad off
# the curve turns an error across it into 1e3 times as much along it
# (relative to t about 3: 2^-52 * 1e3 * a few)
T_TOL = 5e-12


def curves(n, seed, taper, bend):
    """Curves of length 0.4 with r from 0.004 to 0.004 (1 - taper) and inner
    points `bend` off the chord (of its length), in random positions."""
    rng = np.random.default_rng(seed)
    a, s = rng.uniform(0, 1, (n, 3)), W.unit_vectors(rng, n)
    o = np.cross(s, W.unit_vectors(rng, n))
    o /= np.linalg.norm(o, axis=1, keepdims=True)
    P = np.empty((n, 4, 4))
    k = np.arange(4) / 3.0
    P[:, :, :3] = a[:, None] + 0.4 * k[None, :, None] * s[:, None]
    P[:, 1:3, :3] += 0.4 * bend * o[:, None]
    r = np.full(n, 0.004 * 10.0 ** rng.uniform(0, 1))
    P[:, :, 3] = W.linear_taper(r, r * (1.0 - taper))
    return rng, W.unpack_fibers(W.pack_fibers(P))


def rays(rng, P, angle, u0):
    """Rays at `angle` to the tangent at u0, 3 units away, offset sideways."""
    C, T = W.bernstein_point(P, u0), W.bernstein_tangent(P, u0)[:, :3]
    T /= np.linalg.norm(T, axis=1, keepdims=True)
    x = np.cross(T, W.unit_vectors(rng, len(T)))
    x /= np.linalg.norm(x, axis=1, keepdims=True)
    d = np.cos(angle)[:, None] * T + np.sin(angle)[:, None] * x
    side = np.cross(T, x)
    t = C[:, :3] + (rng.uniform(-1.2, 1.2, len(T)) * C[:, 3])[:, None] * side
    O = (t - 3.0 * d).astype(np.float32).astype(np.float64)
    return W.pack_rays(O, t - O, np.full(len(T), 100.0))


@pytest.mark.parametrize("bend", [0.0, 0.01, 0.1])
@pytest.mark.parametrize("taper", [0.0, 1e-3, 0.5, 1.0 - 1e-3])
def test_decision_against_exact(taper, bend):
    n = 4096
    rng, P = curves(n, 77, taper, bend)
    u0 = np.where(np.arange(n) % 4 == 0, rng.choice([0.0, 1.0, 1e-4, 1 - 1e-4], n), rng.uniform(0, 1, n))
    off = 10.0 ** rng.uniform(-3, 0, n)                      # of the tangent, or of its normal plane
    R = rays(rng, P, np.where(np.arange(n) % 2 == 0, off, np.pi / 2 - off), u0)
    F = W.pack_fibers(P)
    out = binding.intersect_pairs(torch.from_numpy(R).to(DEV), torch.from_numpy(F).to(DEV), 22, refine=True)
    h, t = out[2].cpu().numpy().astype(bool), out[3].cpu().numpy()
    tx, _, hx, _ = oracle.intersect_exact(R, F)
    band = np.zeros(n, bool)
    for s in (1 - 1e-4, 1 + 1e-4):
        band |= oracle.intersect_exact(R, F, radius_scale=s)[2] != hx
    valid = np.array([oracle.cubic_constraints(P[i].reshape(16)) == 31 for i in range(n)]) & ~band
    hx = hx.astype(bool)
    assert np.array_equal(h[valid], hx[valid])
    both = valid & h
    assert both.sum() > n // 4
    assert (np.abs(t[both] - tx[both]) / tx[both]).max() <= T_TOL


@pytest.mark.parametrize("n", [1, 63, 64, 65, 1023, 4097])
def test_results_do_not_depend_on_the_call(n):
    """The first n pairs of a call alone and within a larger call, with shallow
    and deep pairs, normals and every family: the same bits."""
    w = W.degenerate_geometry(20000)
    m = W.straight_and_curved(20000)
    F = np.where(np.arange(20000) % 2, w.fibers, m.fibers)
    R = np.where(np.arange(20000) % 2, w.rays, m.rays)
    pd = np.where(np.arange(20000) % 5 == 0, 12, w.pair_depth).astype(np.uint8)
    g = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(DEV)
    big = binding.intersect_pairs(g(R), g(F), 22, pair_depth=g(pd), refine=True, normal=True)
    small = binding.intersect_pairs(g(R[:, :n]), g(F[:, :n]), 22, pair_depth=g(pd[:n]), refine=True, normal=True)
    assert big[2].max() <= 1
    for x, y in zip(small, big):
        x, y = x.contiguous(), y[..., :n].contiguous()
        if x.is_floating_point():
            i = torch.int64 if x.dtype == torch.float64 else torch.int32
            x, y = x.view(i), y.view(i)
        assert torch.equal(x, y)
