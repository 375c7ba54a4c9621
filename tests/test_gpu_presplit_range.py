"""Validation and pre-subdivision of very small and very large fibers.

The bounds that settle most ends compare products of eighth degree in the
coordinates. The mask alone has to be the mask that comes with the excesses
(every end searched, no bounds) at every scale of finite float32, subnormals
and coordinates near the largest value included, and pre-subdivision has to
split what that mask calls invalid. Whole numbers, so comparisons are exact.
"""
import numpy as np
import pytest
import torch

from paper_1811_03374_amd import binding

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
LARGEST = float(np.finfo(np.float32).max)


def bent_arcs(n, seed):
    """Arcs of extent about 1 (rows as in a fiber table, FP64) with radii up
    to their extent: thick ends among them, and clear ones."""
    g = np.random.default_rng(seed)
    p = np.array([[0, 0, 0], [0.55, 0, 0], [1, 0.45, 0], [1, 1, 0]], float)
    P = p[None] + g.uniform(-0.15, 0.15, (n, 4, 3))
    r = g.uniform(0.0, 1.0, (n, 1)) ** 3 * np.ones((n, 4))
    r[0] = 3.0                                  # the bent arc itself, thick at both ends
    P[0] = p
    return np.concatenate([P, r[:, :, None]], 2).reshape(n, 16).T.copy()


def scaled(x, scale):
    with np.errstate(over="raise"):
        return torch.from_numpy((x * scale).astype(np.float32)).to(DEV)


# the smallest subnormals, their upper end, the normal range, the largest values
SCALES = [2.0 ** -142, 1e-41, 2e-41, 1e-40, 1e-38, 1e-30, 2.0 ** -64, 2.0 ** -63, 1.0, 2.0 ** 63, 2.0 ** 64, 1e30,
          1e37, 0.3 * LARGEST]


@pytest.mark.parametrize("scale", SCALES)
def test_mask_alone_equals_searched_mask(scale):
    f = scaled(bent_arcs(4099, 1), scale)
    searched, excess = binding.validate(f, excess=True)
    assert torch.equal(binding.validate(f), searched)
    if scale in (1e-41, 2e-41, 1.0, 0.3 * LARGEST):           # the arc is thick whatever its size
        assert int(searched[0]) == 96 and float(excess[0].min()) > 0.1


def test_largest_coordinates():
    """Random control polygons over the whole range, no two points alike."""
    g = np.random.default_rng(2)
    f = g.uniform(-1.0, 1.0, (16, 20011)) * 0.97 * LARGEST * 2.0 ** -g.integers(0, 6, 20011)
    P = f.reshape(4, 4, -1)
    P[:, 3] = np.abs(P[:, 3])
    P[:, 0] = np.sort(P[:, 0], axis=0)          # forwards along x: inequalities hold more often
    f = scaled(f, 1.0)
    searched, _ = binding.validate(f, excess=True)
    assert int((searched & 96 != 0).sum()) > 1000
    assert torch.equal(binding.validate(f), searched)


@pytest.mark.parametrize("scale", [1e-41, 2e-41, 1e-38, 1.0, 1e37, 0.3 * LARGEST])
@pytest.mark.parametrize("n", [65, (1 << 15) + 3])            # 16 and 64 fibers a wave
def test_presplit_splits_what_the_search_calls_invalid(scale, n):
    f = scaled(bent_arcs(n, 3), scale)
    searched, _ = binding.validate(f, excess=True)
    count = torch.diff(binding.presplit(f, 2)[5])
    assert torch.equal(count > 1, searched != 0)
    # at the level limit the pieces' masks are those of the search
    _, _, _, _, mask, off = binding.presplit(f, 0)
    assert torch.equal(mask, searched) and int(off[-1]) == n
