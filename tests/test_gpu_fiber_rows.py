"""Gathered calls of few pairs read the fiber rows, larger ones records of them:
both load the same floats, so a gathered call equals the identity-paired call
on the gathered columns bit for bit, on either side of the limit."""
import numpy as np
import pytest
import torch

from paper_1811_03374_amd import binding
from paper_1811_03374_amd import workloads as W

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("n", [1, 65, (1 << 16) - 1, 1 << 16, (1 << 16) + 1])
@pytest.mark.parametrize("refine,noalloc", [(False, False), (True, False), (False, True)])
def test_gathered_equals_identity(n, refine, noalloc):
    w = W.straight_and_curved(1 << 17)
    pick = torch.from_numpy(np.random.default_rng(n).integers(0, 1000, n).astype(np.int32)).to(DEV)
    R = torch.from_numpy(np.array(w.rays, order="C")).to(DEV)[:, pick.long()].contiguous()
    F = torch.from_numpy(np.array(w.fibers[:, :1000], order="C")).to(DEV)
    call = binding.intersect_pairs_noalloc if noalloc else binding.intersect_pairs
    a = call(R, F, 20, None, pick, refine=refine)
    b = binding.intersect_pairs(R, F[:, pick.long()].contiguous(), 20, refine=refine)
    assert int(b[2].sum()) > n // 8 or n < 64
    for x, y in zip(a, b):
        v = {torch.float32: torch.int32, torch.float64: torch.int64}.get(x.dtype, x.dtype)
        assert torch.equal(x.view(v), y.view(v))
