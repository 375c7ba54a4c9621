"""Candidate lists, tested by one wave from a ray's first candidate to its last.

Reference: one per-pair call for each position of the lists, on rays shortened
to their nearest hit so far. It runs the same search on the same pairs, so the
plain results have to be the same bit for bit. Refined lists are held to the
nearest of their pairs.
"""
import numpy as np
import pytest
import torch

from paper_1811_03374_amd import binding
from paper_1811_03374_amd import workloads as W

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def g(a):
    return torch.from_numpy(np.array(a, order="C")).to(DEV)


def lists(n, kind, n_fibers, seed):
    """Offsets and fibers of n lists around each ray's own fiber."""
    rng = np.random.default_rng(seed)
    length = {"short": rng.integers(0, 4, n), "ragged": np.where(rng.random(n) < 0.02, 150, rng.integers(0, 9, n)),
              "one": np.ones(n, np.int64), "sparse": np.where(rng.random(n) < 0.1, 12, 0),
              "empty": np.zeros(n, np.int64)}[kind]
    off = np.concatenate([[0], np.cumsum(length)]).astype(np.int64)
    own = np.repeat(np.arange(n), length) % n_fibers
    other = rng.integers(0, n_fibers, off[-1])
    return off, np.where(rng.random(off[-1]) < 0.4, own, other).astype(np.int32)


def one_position_at_a_time(R, F, off, cand, depth, most, normal):
    n = R.shape[1]
    t = torch.full((n,), float("inf"), device=DEV)
    u, nrm = torch.full((n,), float("nan"), device=DEV), torch.full((3, n), float("nan"), device=DEV)
    hit = torch.zeros(n, dtype=torch.uint8, device=DEV)
    fiber = torch.full((n,), -1, dtype=torch.int32, device=DEV)
    length = np.minimum(np.diff(off), most)
    for k in range(int(length.max(initial=0))):
        i = np.nonzero(length > k)[0]
        f, gi = g(cand[off[i] + k]), g(i)
        S = R[:, gi].contiguous()
        S[6] = torch.minimum(S[6], t[gi])
        out = binding.intersect_pairs(S, F, depth, None, f, normal=normal)
        h = out[2] != 0
        j = gi[h]
        t[j], u[j], hit[j], fiber[j] = out[0][h], out[1][h], out[2][h], f[h]
        if normal:
            nrm[:, j] = out[3][:, h]
    return (t, u, hit, fiber) + ((nrm,) if normal else ())


@pytest.mark.parametrize("kind,n,most", [
    ("short", 1, 3), ("ragged", 63, 200), ("ragged", 64, 200), ("ragged", 65, 7), ("ragged", 129, 200),
    ("one", 1000, 1), ("empty", 200, 5), ("sparse", 5000, 12), ("ragged", 20001, 200), ("short", 300001, 3),
    ("sparse", 300001, 12), ("short", 64, 0)])
@pytest.mark.parametrize("depth,normal", [(9, False), (22, True)])
def test_lists_equal_one_position_at_a_time(kind, n, most, depth, normal):
    m, d = W.straight_and_curved(1 << 13), W.degenerate_geometry(1 << 13)
    fibers = np.concatenate([m.fibers, d.fibers], 1)
    rays = np.concatenate([m.rays, d.rays], 1)
    R, F = g(rays[:, np.arange(n) % rays.shape[1]]), g(fibers)
    off, cand = lists(n, kind, fibers.shape[1], n + depth)
    a = binding.intersect_candidates(R, F, g(off), g(cand), depth, max_candidates=most, normal=normal)
    b = one_position_at_a_time(R, F, off, cand, depth, most, normal)
    for x, y in zip(a, b):
        v = torch.int32 if x.dtype == torch.float32 else x.dtype
        assert torch.equal(x.view(v), y.view(v))


@pytest.mark.parametrize("n", [65, 4001])
def test_refined_lists_find_the_pairs_nearest(n):
    """The nearest of all refined pairs of a list, by the per-pair call: t64 to
    1e-9 relative (both come from the same FP64 search, whose range depends on
    where the ray was shortened to)."""
    w = W.straight_and_curved(1 << 13)
    rays, fibers = w.rays[:, :n], w.fibers
    off, cand = lists(n, "ragged", fibers.shape[1], n)
    most = int(np.diff(off).max())
    c = binding.intersect_candidates(g(rays), g(fibers), g(off), g(cand), 22, max_candidates=most, refine=True)
    own = np.repeat(np.arange(n), np.diff(off)).astype(np.int32)
    p = binding.intersect_pairs(g(rays), g(fibers), 22, g(own), g(cand), refine=True)
    t = np.full(n, np.inf)
    np.minimum.at(t, own, p[3].cpu().numpy())
    got = c[4].cpu().numpy()
    hit = np.isfinite(t)
    assert np.array_equal(hit, np.isfinite(got)) and np.array_equal(hit, c[2].cpu().numpy() != 0)
    assert (np.abs(got[hit] - t[hit]) <= 1e-9 * np.abs(t[hit])).all()
