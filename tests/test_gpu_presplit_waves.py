"""Validation and pre-subdivision where the work is shared between lanes.

The mask alone (settled by bounds where they suffice) against the mask that
comes with the excesses (every end searched), and pre-subdivision at the edges
of its waves: the pieces of a table's first n fibers are the first pieces of a
larger table's, whichever kernel variant n selects. Whole numbers and exact
halvings, so every comparison is bitwise.
"""
import numpy as np
import pytest
import torch

from paper_1811_03374_amd import binding
from paper_1811_03374_amd import workloads as W

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def awkward(n):
    """Degenerate, bent and hair fibers in turn; hooks far from the origin,
    single points, a NaN and an infinity among them."""
    k = -(-n // 4)
    parts = [W.degenerate_geometry(4 * k).fibers[:, :k], W.straight_and_curved(4 * k).fibers[:, 1:2 * k:2],
             W.pack_fibers(W.hair_strands(max(1, -(-k // 8))))[:, :k],
             W.pack_fibers(W.hair_strands(max(1, -(-k // 8))))[:, :k].copy()]
    hook = parts[3]
    hook[4:7] = 2 * hook[0:3] - hook[4:7]                     # p1 turned back behind p0
    f = np.stack(parts, axis=2).reshape(16, -1)[:, :n].copy()
    f[:, 5::97] = np.tile(f[:4, 5::97], (4, 1))               # all four points equal
    f[9, 11::193] = np.nan
    f[2, 13::211] = np.inf
    return f


@pytest.mark.parametrize("n", [1, 7, 255, 256, 257, 20000])
def test_mask_alone_equals_mask_with_excesses(n):
    f = torch.from_numpy(awkward(n)).to(DEV)
    with_excess, _ = binding.validate(f, excess=True)
    assert torch.equal(binding.validate(f), with_excess)
    wide = torch.empty(16, n + 13, device=DEV)[:, 5:5 + n]    # rows further apart, not aligned
    wide.copy_(f)
    assert torch.equal(binding.validate(wide), with_excess)


@pytest.fixture(scope="module")
def large():
    f = torch.from_numpy(awkward(40000)).to(DEV)              # above 2^15: 64 fibers a wave
    return f, {level: binding.presplit(f, level) for level in (0, 3, 10)}


@pytest.mark.parametrize("level", [0, 3, 10])
@pytest.mark.parametrize("n", [1, 15, 16, 17, 63, 64, 65, 1000, 1 << 15, (1 << 15) + 1])
def test_pieces_of_a_prefix(large, n, level):
    f, whole = large
    part = binding.presplit(f[:, :n].contiguous(), level)
    k = part[1].shape[0]
    assert torch.equal(part[5], whole[level][5][:n + 1]) and k == int(part[5][-1])
    for x, y in zip(part[:5], whole[level][:5]):
        x, y = x.contiguous(), y[..., :k].contiguous()
        if x.dtype == torch.float32:                          # NaN pieces compare by their bits
            x, y = x.view(torch.int32), y.view(torch.int32)
        assert torch.equal(x, y)
