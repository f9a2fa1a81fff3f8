"""The direct-to-LDS kernel of calls of few tiles a workgroup: vocabulary splits that end in half a tile, and bounds shared between
k classes of splits, against the CPU oracle and, where the oracle's fp64 says nothing, the register-staged kernel."""
import numpy as np
import pytest
import torch

from paper_2604_06483_amd import binding as LL
from paper_2604_06483_amd import workloads as WL
from tests import parity as P
from tests.conftest import say

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def inputs(N, d, V, k):
    return WL.make_workload(WL.LensConfig("short", L=1, T=N, d=d, V=V, k=k, n_outliers=2 if d > 100 else 0, outlier_scale=20.0),
                            DEV, seed=61)


def a_bias(V, seed=3):
    return 0.5 * torch.randn((V,), generator=torch.Generator(device=DEV).manual_seed(seed), device=DEV)


@pytest.mark.parametrize("N,d,V,k,with_bias,gamma", [
    (129, 64, 700, 4, False, True),       # six half tiles, a split each, the last of 60 ids; one stage
    (129, 64, 700, 20, False, True),      # the same, fewer splits than k
    (300, 128, 10000, 12, False, True),   # 79 splits of half a tile
    (300, 64, 40000, 10, False, True),    # 105 splits of three half tiles
    (300, 192, 40000, 1, True, False),    # the same with a bias; rows read in place
    (257, 128, 33000, 20, False, False),  # rows read in place, 20 classes
    (1000, 72, 50257, 3, True, True),     # 57 splits of six or seven half tiles, two stages, the second with one chunk
    (1000, 136, 50257, 12, True, True),   # the same, three stages
    (800, 200, 33000, 20, False, True),   # four stages, the last with one chunk
    (520, 64, 66000, 2, False, True),     # whole tiles, classes only
    (9000, 64, 4000, 5, False, True),     # two passes: fewer splits than k in the first, more in the second
    (9000, 64, 4000, 5, False, False),    # the same, rows read in place
])
def test_short_call(N, d, V, k, with_bias, gamma):
    say(f"short N={N} d={d} V={V} k={k} bias={with_bias} gamma={gamma}")
    w = inputs(N, d, V, k)
    bias = a_bias(V) if with_bias else None
    got = P.to_numpy(LL.ll_project(w.hidden, w.gamma if gamma else None, w.W_U, w.cfg.eps, k, w.target_ids, bias=bias))
    rows = np.arange(N) if N <= 1000 else np.unique(np.r_[0:300, 8150:8250, N - 200:N])
    ref = P.oracle_rows(WL.bf16_bits(w.hidden.reshape(-1, d))[rows], WL.bf16_bits(w.gamma) if gamma else None, WL.bf16_bits(w.W_U),
                        w.cfg.eps, k, w.target_ids.cpu().numpy()[rows], bias=None if bias is None else bias.cpu().numpy())
    P.compare({n: x[rows] for n, x in got.items()}, ref, k, label="short")


@pytest.mark.parametrize("N,d,V,k", [(300, 64, 40000, 10), (300, 72, 10000, 4), (1000, 64, 50257, 20)])
def test_equal_logits_are_listed_by_id(N, d, V, k):
    """Rows of zeros: every split's best is the shared bound."""
    say(f"short, equal logits N={N} d={d} V={V} k={k}")
    w = inputs(N, d, V, k)
    w.hidden.reshape(N, d)[::7] = 0
    w.W_U[V // 2:] = w.W_U[:V - V // 2].clone()      # and two of every other token
    ids, p, _, _ = LL.ll_project(w.hidden, w.gamma, w.W_U, w.cfg.eps, k, w.target_ids)
    assert torch.equal(ids[::7], torch.arange(k, device=DEV, dtype=torch.int32).expand_as(ids[::7]))
    b, q, _, _ = LL.ll_project(w.hidden, w.gamma, w.W_U, w.cfg.eps, k, w.target_ids, register_staged=True)
    assert (ids != b).float().mean() < 1e-3          # near-ties that the order of the sums decides
    torch.testing.assert_close(p, q, rtol=2e-5, atol=2e-5)


@pytest.mark.parametrize("N,d,V,k,gamma", [(300, 128, 10000, 12, True), (1000, 200, 50257, 3, True), (8500, 64, 20000, 5, True),
                                           (8500, 64, 20000, 5, False), (520, 64, 65000, 20, False)])
def test_a_workspace_without_room_for_the_classes_gives_the_same_bits(N, d, V, k, gamma):
    """The least workspace that is accepted holds neither the bounds of the classes nor the row of zeros behind the panel."""
    say(f"short, least workspace N={N} d={d} V={V} k={k} gamma={gamma}")
    w = inputs(N, d, V, k)
    g = w.gamma if gamma else None
    want = LL.ll_project(w.hidden, g, w.W_U, w.cfg.eps, k, w.target_ids)
    full = LL.ll_workspace_bytes(N, d, V, k)
    ws = torch.empty((full,), dtype=torch.uint8, device=DEV)
    lo, hi = 0, full // 256                                         # refused, accepted
    while hi - lo > 1:
        mid = (lo + hi) // 2
        try:
            LL.ll_project(w.hidden, g, w.W_U, w.cfg.eps, k, w.target_ids, workspace=ws[:256 * mid])
            hi = mid
        except LL.LLError as e:
            assert e.code == LL.LL_EWORKSPACE
            lo = mid
    ws.fill_(0xA5)                                                  # stale contents of another call
    got = LL.ll_project(w.hidden, g, w.W_U, w.cfg.eps, k, w.target_ids, workspace=ws[:256 * hi])
    assert full - 256 * hi >= (4 * min(N, 3000) * k if gamma else 0) and (ws[256 * hi:] == 0xA5).all()
    for a, b in zip(got, want):
        assert torch.equal(a, b)


@pytest.mark.parametrize("d", [64, 72])
def test_masked_and_infinite_logits(d):
    say(f"short, masks and infinities d={d}")
    N, V, k = 300, 40000, 5
    w = inputs(N, d, V, k)
    bias = torch.full((V,), torch.finfo(torch.float32).min, device=DEV)
    bias[[17, 20000, 39999]] = 0.0                   # fewer than k that count
    ids = LL.ll_project(w.hidden, w.gamma, w.W_U, w.cfg.eps, k, w.target_ids, bias=bias)[0]
    ref = LL.ll_project(w.hidden, w.gamma, w.W_U, w.cfg.eps, k, w.target_ids, bias=bias, register_staged=True)[0]
    assert torch.equal(ids, ref) and set(ids[:, :3].unique().tolist()) == {17, 20000, 39999}
    w.W_U[3, -1] = float("-inf")
    w.W_U[39999, 0] = float("inf")
    a = LL.ll_project(w.hidden, w.gamma, w.W_U, w.cfg.eps, k, w.target_ids)
    b = LL.ll_project(w.hidden, w.gamma, w.W_U, w.cfg.eps, k, w.target_ids, register_staged=True)
    fine = torch.isfinite(b[1]).all(1)
    assert 0 < int(fine.sum()) < N and (a[0][fine] != b[0][fine]).float().mean() < 1e-3
    for x, y in zip(a[1:], b[1:]):                   # fp32 sums in another order
        torch.testing.assert_close(x, y, rtol=2e-5, atol=2e-5, equal_nan=True)
