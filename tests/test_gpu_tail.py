"""The direct-to-LDS kernels at hidden sizes that are not a multiple of 64 (more than 128 rows: fewer have a kernel of
their own; the one of short calls in most cases, the long one where a case says so), against the CPU oracle and, where the oracle's fp64 says nothing (infinities), the register-staged kernel."""
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
    return WL.make_workload(WL.LensConfig("tail", L=1, T=N, d=d, V=V, k=k, n_outliers=2 if d > 100 else 0, outlier_scale=20.0),
                            DEV, seed=31)


@pytest.mark.parametrize("N,d,V,k,with_bias,gamma", [
    (129, 8, 700, 1, False, True),        # one stage, one chunk of it real
    (300, 56, 257, 20, True, False),      # one stage, seven chunks, rows used as they are: register-staged
    (257, 72, 3000, 32, True, True),      # the longest list with a bias: register-staged
    (520, 120, 5001, 12, False, True),    # two stages, seven chunks
    (777, 1608, 2050, 3, True, True),     # many stages
    (9000, 136, 600, 5, False, True),     # two row passes
    (8200, 8, 5001, 1, False, True),      # one stage, three tiles a workgroup
    (8200, 56, 8000, 20, True, False),    # one stage, four tiles, a long list with a bias: register-staged
    (8200, 8, 12801, 1, False, True),     # one stage, seven tiles a workgroup
    (8200, 56, 12801, 20, True, True),    # the same, seven chunks of the stage real: the long kernel
    (1000, 72, 41000, 12, False, True),   # two stages, three tiles, the second stage with one chunk
    (300, 328, 700, 32, False, True),     # six stages, one tile: the long kernel
    (300, 648, 700, 3, True, False),      # eleven stages, rows only padded
])
def test_ragged_hidden_size(N, d, V, k, with_bias, gamma):
    say(f"tail N={N} d={d} V={V} k={k} bias={with_bias} gamma={gamma}")
    w = inputs(N, d, V, k)
    bias = 0.5 * torch.randn((V,), generator=torch.Generator(device=DEV).manual_seed(3), device=DEV) if with_bias else None
    got = P.to_numpy(LL.ll_project(w.hidden, w.gamma if gamma else None, w.W_U, w.cfg.eps, k, w.target_ids, bias=bias))
    ref = P.oracle_rows(WL.bf16_bits(w.hidden.reshape(-1, d)), WL.bf16_bits(w.gamma) if gamma else None, WL.bf16_bits(w.W_U),
                        w.cfg.eps, k, w.target_ids.cpu().numpy(), bias=None if bias is None else bias.cpu().numpy())
    P.compare(got, ref, k, label="tail")


@pytest.mark.parametrize("N,d", [(200, 200), (100, 200), (200, 392)])     # the kernel of short calls, half tiles alone; the few-rows kernel
def test_infinite_weights_stay_in_their_own_logit(N, d):
    say(f"tail, infinite weights N={N} d={d}")
    w = inputs(N, d, 1000, 6)
    w.W_U[3, -1] = float("-inf")     # the last chunk of a row, which lanes past the end fetch
    w.W_U[700, 0] = float("inf")     # the first chunk of a row, which is what follows the end of the row before
    a = LL.ll_project(w.hidden, w.gamma, w.W_U, w.cfg.eps, 6, w.target_ids)
    b = LL.ll_project(w.hidden, w.gamma, w.W_U, w.cfg.eps, 6, w.target_ids, register_staged=True)
    fine = torch.isfinite(b[1]).all(1)
    assert 0 < int(fine.sum()) < N                               # rows where both infinities give -inf, and rows where one does not
    assert torch.equal(a[0][fine], b[0][fine])
    for x, y in zip(a[1:], b[1:]):                               # fp32 sums in another order, as in ll_project_static's test
        torch.testing.assert_close(x, y, rtol=2e-5, atol=2e-5, equal_nan=True)
