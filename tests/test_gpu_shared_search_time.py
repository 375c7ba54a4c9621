"""Sharing the long searches of a call must not make it slower.

The counting call visits the same nodes one after another, never shares and
writes 16 bytes a pair more: over inputs as they come, most of them without
a search of hundreds of nodes, the plain call may take no longer than it. 5 %
allow for the timing and for inputs whose longest search ends just after
sharing starts (not shared, the plain call takes 0.98 of the counting call's
time).
"""
import pytest
import torch

from paper_1811_03374_amd import binding
from paper_1811_03374_amd import workloads as W

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def best_us(call, calls=10, runs=6):
    for _ in range(3):
        call()
    best = float("inf")
    for _ in range(runs):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(calls):
            call()
        b.record()
        b.synchronize()
        best = min(best, a.elapsed_time(b) / calls * 1e3)
    return best


@pytest.mark.parametrize("n", [13039, 40000])
def test_plain_call_no_slower_than_counting(n):
    plain = counting = 0.0
    for seed in range(8):
        w = W.straight_and_curved(n, seed=seed)
        R, F = torch.from_numpy(w.rays).to(DEV), torch.from_numpy(w.fibers).to(DEV)
        n_pairs = R.shape[1]
        out = (torch.empty(n_pairs, device=DEV), torch.empty(n_pairs, device=DEV),
               torch.empty(n_pairs, dtype=torch.uint8, device=DEV))
        plain += best_us(lambda: binding.intersect_pairs(R, F, 22, out=out))
        counting += best_us(lambda: binding.intersect_pairs(R, F, 22, out=out, counts=True))
    print(f"[shared] {n} pairs, 8 inputs: plain {plain / 8:.1f} us, counting {counting / 8:.1f} us", flush=True)
    assert plain <= 1.05 * counting
