"""The direct-to-LDS kernel of calls of few tiles a workgroup: vocabulary splits that end in half a tile, and bounds shared between
k classes of splits, against the CPU oracle and, where the oracle's fp64 says nothing, the register-staged kernel."""
import numpy as np
import pytest
import torch

from paper_2604_06483_amd import binding as LL
from paper_2604_06483_amd import workloads as WL
from tests import parity as P
from tests.conftest import kernels_of, say

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def inputs(N, d, V, k):
    return WL.make_workload(WL.LensConfig("short", L=1, T=N, d=d, V=V, k=k, n_outliers=2 if d > 100 else 0, outlier_scale=20.0),
                            DEV, seed=61)


def runs(call, *kernels):
    """Asserts which projection kernel each pass of the call takes."""
    names = [n.split("<")[0] for n in kernels_of(call) if n.startswith("ll_lens_")]
    assert names == list(kernels), names


SHORT, LONG = "ll_lens_gemm_short_kernel", "ll_lens_gemm_dma_kernel"


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
    (520, 64, 65000, 2, False, True),     # whole tiles, classes only
    (9000, 64, 4000, 5, False, True),     # two passes, 8 and 32 splits: classes in both
    (9000, 64, 4000, 12, False, True),    # fewer splits than k in the first (the long kernel, one bound a row), more in the second
    (9000, 64, 4000, 12, False, False),   # the same, rows read in place
])
def test_short_call(N, d, V, k, with_bias, gamma):
    say(f"short N={N} d={d} V={V} k={k} bias={with_bias} gamma={gamma}")
    w = inputs(N, d, V, k)
    bias = a_bias(V) if with_bias else None
    call = lambda: LL.ll_project(w.hidden, w.gamma if gamma else None, w.W_U, w.cfg.eps, k, w.target_ids, bias=bias)
    got = P.to_numpy(call())
    runs(call, *([LONG, SHORT] if N > 8192 and k == 12 else [SHORT] * (1 + N // 8192)))
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
    call = lambda: LL.ll_project(w.hidden, w.gamma, w.W_U, w.cfg.eps, k, w.target_ids)
    runs(call, SHORT)
    ids, p, _, _ = call()
    assert torch.equal(ids[::7], torch.arange(k, device=DEV, dtype=torch.int32).expand_as(ids[::7]))
    b, q, _, _ = LL.ll_project(w.hidden, w.gamma, w.W_U, w.cfg.eps, k, w.target_ids, register_staged=True)
    assert (ids != b).float().mean() < 1e-3          # near-ties that the order of the sums decides
    torch.testing.assert_close(p, q, rtol=2e-5, atol=2e-5)


@pytest.mark.parametrize("N,d,V,k,static", [
    (1422, 21376, 3000, 10, SHORT),                         # half tiles, without classes
    (1700, 16320, 18000, 20, LONG),                         # whole ones
    (1700, 16264, 18000, 20, "ll_lens_gemm_dma_tail_kernel"),
])
def test_a_pass_that_fills_the_static_buffer_gives_the_same_bits(N, d, V, k, static):
    """Its panel ends where the buffer does: neither the bounds of the classes nor the row of zeros behind it have room."""
    say(f"short, a pass that fills the static buffer N={N} d={d} V={V} k={k}")
    w = inputs(N, d, V, k)
    workspace = lambda: LL.ll_project(w.hidden, w.gamma, w.W_U, w.cfg.eps, k, w.target_ids)
    buffer = lambda: LL.ll_project_static(w.hidden, w.gamma, w.W_U, w.cfg.eps, k, w.target_ids)
    runs(workspace, SHORT)
    runs(buffer, static)
    for a, b in zip(workspace(), buffer()):
        assert torch.equal(a, b)


@pytest.mark.parametrize("N,gamma", [(300, True), (9000, True), (9000, False)])
def test_stale_contents_of_the_workspace(N, gamma):
    say(f"short, stale workspace N={N} gamma={gamma}")
    d, V, k = 64, 4000, 12
    w = inputs(N, d, V, k)
    ws = torch.full((LL.ll_workspace_bytes(N, d, V, k),), 0xA5, dtype=torch.uint8, device=DEV)
    call = lambda **kw: LL.ll_project(w.hidden, w.gamma if gamma else None, w.W_U, w.cfg.eps, k, w.target_ids, **kw)
    for a, b in zip(call(workspace=ws), call()):
        assert torch.equal(a, b)


@pytest.mark.parametrize("d", [64, 72, 200])
def test_masked_and_infinite_logits(d):
    say(f"short, masks and infinities d={d}")
    N, V, k = 300, 40000, 5
    w = inputs(N, d, V, k)
    bias = torch.full((V,), torch.finfo(torch.float32).min, device=DEV)
    bias[[17, 20000, 39999]] = 0.0                   # fewer than k that count
    runs(lambda: LL.ll_project(w.hidden, w.gamma, w.W_U, w.cfg.eps, k, w.target_ids, bias=bias), SHORT)
    runs(lambda: LL.ll_project(w.hidden, w.gamma, w.W_U, w.cfg.eps, k, w.target_ids), SHORT)
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


@pytest.mark.parametrize("d,V", [(200, 40000), (392, 30000)])
def test_an_infinity_at_a_row_end_stays_in_its_own_logit(d, V):
    """The last chunk of vocabulary rows that lie in the half tile behind a split's whole one (105 splits of three half tiles of 128, then
    118 of two; the end of the vocabulary in a half one): the padding of the last stage, which that chunk fills first, is zero again
    before it is multiplied."""
    say(f"short, infinities at the rows' ends d={d} V={V}")
    N, k = 300, 5
    w = inputs(N, d, V, k)
    halves, splits = -(-V // 128), 105 if V == 40000 else 118
    ends = [(s + 1) * halves // splits * 128 - 1 - 7 * s % 120 for s in range(0, splits, 9)]      # ids of splits' last half tiles
    odd = [i for i in ends if 0 < i < V]
    assert len(odd) >= 10
    w.W_U[odd, -1] = float("-inf")
    call = lambda: LL.ll_project(w.hidden, w.gamma, w.W_U, w.cfg.eps, k, w.target_ids)
    runs(call, SHORT)
    a, b = call(), LL.ll_project(w.hidden, w.gamma, w.W_U, w.cfg.eps, k, w.target_ids, register_staged=True)
    fine = torch.isfinite(b[1]).all(1)               # rows whose last entry is positive: those tokens are at -inf
    assert N // 4 < int(fine.sum()) < N and (a[0][fine] != b[0][fine]).float().mean() < 1e-3
    for x, y in zip(a[1:], b[1:]):                   # fp32 sums in another order
        torch.testing.assert_close(x, y, rtol=2e-5, atol=2e-5, equal_nan=True)
