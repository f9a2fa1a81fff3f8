"""The lanes past the last row of a block of 256 hold a row of zeros, whose logits are the bias or the shift alone.  They cost nothing,
also where those grow with the id, so that every token would be the best one so far."""
import pytest
import torch

from paper_2604_06483_amd import binding as LL
from tests.conftest import say

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def inputs(N, d, V, seed=71):
    """Rows whose logits fall with the id by some 5 ramp(id), and the ramp, from 0 to 1: a bias or shift that grows with it."""
    g = torch.Generator(device=DEV).manual_seed(seed)
    ramp = torch.arange(V, device=DEV, dtype=torch.float32) / V
    W = (0.001 * torch.randn((V, d), generator=g, device=DEV)).to(torch.bfloat16)
    W[:, 0] = -ramp.to(torch.bfloat16)
    W[:, 1] = ramp.to(torch.bfloat16)
    h = torch.randn((N, d), generator=g, device=DEV).to(torch.bfloat16)
    h[:, 0], h[:, 1] = 8.0, 0.0
    return h, torch.ones((d,), dtype=torch.bfloat16, device=DEV), W, ramp


def call_time(call, reps=9, inner=8):
    for _ in range(2):
        call()
    times = []
    for _ in range(reps):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(inner):
            call()
        b.record()
        b.synchronize()
        times.append(a.elapsed_time(b) / inner * 1e3)
    return sorted(times)[reps // 2]


@pytest.mark.parametrize("N,d,V,k", [
    (130, 64, 60000, 10),    # classes of splits, half tiles
    (130, 200, 200000, 10),  # the same, ragged
    (130, 64, 60000, 20),    # a list with a bias that has no classes
    (130, 64, 60000, 32),    # the longest, which shares no bounds
    (2049, 64, 120000, 10),  # the last block of nine: one row, 17 tiles a split
])
def test_projection_with_a_bias(N, d, V, k):
    h, gamma, W, ramp = inputs(N, d, V)
    flat = torch.zeros_like(ramp)
    ws = torch.empty(LL.ll_workspace_bytes(N, d, V, k), dtype=torch.uint8, device=DEV)
    grows, zero = (call_time(lambda: LL.ll_project(h, gamma, W, 1e-5, k, None, workspace=ws, bias=b)) for b in (4.0 * ramp, flat))
    say(f"padded rows, bias N={N} d={d} V={V} k={k}: {grows:.1f} us, without {zero:.1f}")
    assert grows < 1.3 * zero   # (the rows' own lists: up to 1.2; with such lanes' as well 1.4 to 2.6)


@pytest.mark.parametrize("N,V,n_alpha,k", [(3, 60000, 2, 2), (3, 60000, 3, 3), (3, 60000, 9, None), (3, 60000, 9, 4), (1025, 60000, 9, 3)])
def test_sweep(N, V, n_alpha, k):
    """v picks the column that the rows do not have: u is the ramp."""
    h, gamma, W, ramp = inputs(N, 64, V)
    v = torch.zeros((64,), device=DEV)
    v[1] = 1.0
    alphas = [4.0 - 0.25 * a for a in range(n_alpha)]
    ws = torch.empty(LL.ll_steer_sweep_workspace_bytes(N, 64, V, n_alpha, k or 1), dtype=torch.uint8, device=DEV)
    grows, falls = (call_time(lambda: LL.ll_steer_sweep(h, gamma, W, 1e-5, s * v, alphas, None, k=k, workspace=ws)) for s in (1.0, -1.0))
    say(f"padded rows, sweep N={N} V={V} A={n_alpha} k={k}: {grows:.1f} us, {falls:.1f} with shifts that fall")
    assert grows < 1.3 * falls   # (likewise; 1.9 to 4.5)
