"""Which kernel a call takes, and its results against the CPU oracle there: shapes on either side of the lines of the dispatch, so that
a line that moves cannot leave a kernel without a case of its own unnoticed."""
import numpy as np
import pytest
import torch

from paper_2604_06483_amd import binding as LL
from paper_2604_06483_amd import workloads as WL
from tests import parity as P
from tests.conftest import kernels_of, say
from tests.test_gpu_sweep import ALPHAS9, direction
from tests.test_gpu_sweep_forms import check

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

LONG, TAIL, SHORT = "ll_lens_gemm_dma_kernel", "ll_lens_gemm_dma_tail_kernel", "ll_lens_gemm_short_kernel"
STAGED, FEW = "ll_lens_gemm_kernel", "ll_lens_few_kernel"


def main_kernels(call):
    return [n.split("(")[0] for n in kernels_of(call) if n.startswith(("ll_lens_", "ll_sweep_table"))]


def projection(N, d, V, k, with_bias, gamma, expected, zero_rows=False):
    """Runs the call, asserts its kernels (one name a pass) and compares up to 600 of its rows with the oracle."""
    w = WL.make_workload(WL.LensConfig("route", L=1, T=N, d=d, V=V, k=k, n_outliers=2 if d > 100 else 0, outlier_scale=20.0), DEV, seed=67)
    bias = 0.5 * torch.randn((V,), generator=torch.Generator(device=DEV).manual_seed(3), device=DEV) if with_bias else None
    if zero_rows:
        w.hidden.reshape(N, d)[::7] = 0
        w.W_U[V // 2:] = w.W_U[:V - V // 2].clone()      # and two of every token
    call = lambda: LL.ll_project(w.hidden, w.gamma if gamma else None, w.W_U, w.cfg.eps, k, w.target_ids, bias=bias)
    out = call()
    if zero_rows and not with_bias:
        assert torch.equal(out[0][::7], torch.arange(k, device=DEV, dtype=torch.int32).expand_as(out[0][::7]))
    got = P.to_numpy(out)
    names = main_kernels(call)
    assert [n.split("<")[0] for n in names] == expected, names
    rows = np.arange(N) if N <= 600 else np.unique(np.r_[0:200, N // 2:N // 2 + 200, N - 200:N])
    ref = P.oracle_rows(WL.bf16_bits(w.hidden.reshape(-1, d))[rows], WL.bf16_bits(w.gamma) if gamma else None, WL.bf16_bits(w.W_U),
                        w.cfg.eps, k, w.target_ids.cpu().numpy()[rows], bias=None if bias is None else bias.cpu().numpy())
    P.compare({n: x[rows] for n, x in got.items()}, ref, k, label="route")
    return names


@pytest.mark.parametrize("N,d,V,k,with_bias,gamma,expected", [
    (300, 56, 10000, 4, False, True, [SHORT]),     # one stage: classes of splits always pay for the padded rows
    (300, 72, 40000, 20, False, False, [SHORT]),   # no norm either
    (1000, 56, 5000, 3, True, False, [SHORT]),     # a bias and half tiles
    (700, 56, 15000, 3, True, True, [STAGED]),     # a bias, whole tiles: one stage
    (700, 200, 15000, 3, True, True, [SHORT]),     # four
    (700, 200, 15000, 3, True, False, [STAGED]),
    (700, 264, 15000, 10, True, False, [SHORT]),   # five
    (9000, 72, 2000, 20, False, True, [STAGED, STAGED]),   # fewer splits than k: two stages
    (300, 584, 128256, 1, True, True, [TAIL]), (300, 584, 128256, 3, True, True, [SHORT]),   # the shortest list with a bias: four tiles
    (700, 584, 50257, 1, True, True, [SHORT]),     # half a tile less
    (4000, 584, 60000, 3, True, True, [TAIL]), (4000, 584, 60000, 5, True, True, [SHORT]),   # fifteen
    (4000, 200, 60000, 1, True, True, [SHORT]),    # fewer stages
    (300, 200, 10000, 24, False, True, [STAGED]),  # the longest list: four stages, then six
    (300, 328, 10000, 24, False, True, [TAIL]),
])
def test_ragged_hidden_sizes(N, d, V, k, with_bias, gamma, expected):
    say(f"route N={N} d={d} V={V} k={k} bias={with_bias} gamma={gamma}")
    projection(N, d, V, k, with_bias, gamma, expected)


@pytest.mark.parametrize("k,with_bias", [(3, False), (10, False), (20, False), (32, False), (3, True), (10, True), (20, True), (32, True)])
@pytest.mark.parametrize("d", [64, 72])
def test_long_calls(d, k, with_bias):
    """A full pass of 35 tiles a workgroup, with rows of zeros and two of every token: ties across the splits."""
    say(f"route, 8192 rows, 35 tiles a workgroup d={d} k={k} bias={with_bias}")
    projection(8192, d, 70000, k, with_bias, True, [LONG if d == 64 else STAGED if k == 32 and with_bias else TAIL], zero_rows=True)


@pytest.mark.parametrize("N,d,V,k,with_bias,expected", [
    (128, 64, 128256, 12, True, [SHORT]), (97, 64, 128256, 20, False, [SHORT]),
    (128, 64, 128256, 13, True, [FEW]), (128, 64, 128256, 21, False, [FEW]),
    (128, 72, 128256, 4, False, [SHORT]), (128, 72, 128256, 5, False, [FEW]),
    (96, 64, 128256, 1, False, [FEW]), (128, 64, 98000, 1, False, [FEW]),      # one round of workgroups
])
def test_few_rows_in_two_rounds(N, d, V, k, with_bias, expected):
    say(f"route N={N} d={d} V={V} k={k} bias={with_bias}")
    projection(N, d, V, k, with_bias, True, expected)


@pytest.mark.parametrize("N,d,V,A,k,expected", [
    (300, 128, 20000, 1, 2, ["projection"]), (300, 72, 20000, 1, 4, ["projection"]), (300, 128, 20000, 1, None, ["own general"]),
    (1500, 64, 50257, 1, None, ["projection"]),
    (300, 128, 50257, 6, None, ["own general"]), (300, 128, 50257, 7, None, ["table", "general", "factored"]),     # two tiles a split
    (300, 512, 50257, 5, None, ["own general"]), (300, 512, 50257, 6, None, ["table", "general", "factored"]),
    (70, 128, 5000, 8, None, ["own general"]), (70, 128, 5000, 9, None, ["table", "general", "factored"]),         # one
    (2100, 64, 60000, 4, None, ["own general"]), (2100, 320, 60000, 4, None, ["table", "general", "factored"]),    # nine
    (70, 64, 5000, 4, 4, ["own general"]), (70, 64, 5000, 5, 4, ["table", "general", "factored"]),                 # lists
    (10, 128, 70000, 3, 3, ["own general"]), (10, 128, 70000, 4, 3, ["table", "general", "factored"]),
])
def test_sweeps(N, d, V, A, k, expected):
    say(f"route sweep N={N} d={d} V={V} A={A} k={k}")
    w = WL.make_workload(WL.LensConfig("route", L=1, T=N, d=d, V=V, k=1), DEV, seed=41)
    names = main_kernels(lambda: LL.ll_steer_sweep(w.hidden.reshape(N, d), w.gamma, w.W_U, w.cfg.eps, direction(d), ALPHAS9[:A], w.target_ids, k=k))
    kinds = ["table" if n.startswith("ll_sweep_table") else "projection" if "TopKEpilogue" in n else
             ("own " if "WholeSweep" in n else "") + ("general" if "true> >" in n or "true>>" in n else "factored") for n in names]
    assert kinds == expected, names
    check(N, d, V, ALPHAS9[:A], k, 1.0, "route", rows=np.unique(np.r_[0:40, N // 2:N // 2 + 40, N - 40:N]) if N > 100 else None)
