"""The projection of few lens rows (at most 128: its own kernel, vocabulary dealt in groups of 16 rows, unordered
candidate lists merged by counting), at the sizes where it can go wrong, against the CPU oracle."""
import numpy as np
import pytest
import torch

import oracle.lens_oracle as O
from paper_2604_06483_amd import binding as LL
from paper_2604_06483_amd import workloads as WL
from tests import parity as P
from tests.conftest import kernels_of, say

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

CASES = [
    # N,   d,    V,   k, bias
    (1,    64,   33,  1, False),     # one stage (filled up to two), three groups of 16, the last with one row
    (16,   192,  300, 32, False),    # three stages; longest list
    (17,   72,   129, 5, True),      # d not a whole number of stages: one chunk in the last
    (33,   120,  2000, 20, False),   # seven chunks in the last stage
    (48,   8,    4096, 7, False),    # one chunk in all
    (64,   1096, 5001, 3, True),     # odd number of stages and a ragged last one
    (65,   320,  40000, 20, False),  # 16-row blocks rounded up to six
    (96,   128,  70000, 10, False),  # parts of 17 and 18 groups
    (97,   256,  33000, 32, True),   # eight 16-row blocks
    (128,  64,   140000, 20, False),  # two rounds of workgroups
    (128,  64,   100000, 5, False),  # the same, two groups a wavefront
    (113,  64,   100000, 4, False),  # the same with a short list: the 256-row kernel
    (37,   64,   151936, 10, False),  # five groups per wavefront
    (20,   64,   300000, 12, False),  # two rounds of five
    (5,    64,   400000, 4, False),  # a vocabulary past the kernel's parts: the 256-row kernel
]


def inputs(N, d, V, seed=21):
    cfg = WL.LensConfig("few", L=1, T=N, d=d, V=V, k=1, n_outliers=2 if d > 100 else 0, outlier_scale=20.0)
    return WL.make_workload(cfg, DEV, seed=seed)


def reference(w, k, bias=None):
    return P.oracle_rows(WL.bf16_bits(w.hidden.reshape(-1, w.cfg.d)), WL.bf16_bits(w.gamma), WL.bf16_bits(w.W_U), w.cfg.eps, k,
                         w.target_ids.cpu().numpy(), bias=None if bias is None else bias.cpu().numpy())


@pytest.mark.parametrize("N,d,V,k,with_bias", CASES)
def test_few_rows(N, d, V, k, with_bias):
    say(f"few rows N={N} d={d} V={V} k={k} bias={with_bias}")
    w = inputs(N, d, V)
    bias = 0.5 * torch.randn((V,), generator=torch.Generator(device=DEV).manual_seed(3), device=DEV) if with_bias else None
    ws = torch.full((LL.ll_workspace_bytes(N, d, V, k),), 0xFF, dtype=torch.uint8, device=DEV)
    res = LL.ll_project(w.hidden, w.gamma, w.W_U, w.cfg.eps, k, w.target_ids, workspace=ws, bias=bias)
    torch.cuda.synchronize()
    got = P.to_numpy(res)
    P.compare(got, reference(w, k, bias), k, label="few")
    P.check_invariants(got, V, k, label="few")
    if bias is None:
        static = LL.ll_project_static(w.hidden, w.gamma, w.W_U, w.cfg.eps, k, w.target_ids)
        for a, b in zip(res, static):
            assert torch.equal(a, b)


def test_a_workspace_sized_for_more_rows():
    N, d, V, k = 81, 128, 128256, 10
    say(f"few rows in the workspace of a longer call N={N} d={d} V={V} k={k}")
    assert LL.ll_workspace_bytes(1500, d, V, k) < LL.ll_workspace_bytes(N, d, V, k)
    w = inputs(N, d, V)
    ws = torch.full((LL.ll_workspace_bytes(1500, d, V, k),), 0xFF, dtype=torch.uint8, device=DEV)
    got = P.to_numpy(LL.ll_project(w.hidden, w.gamma, w.W_U, w.cfg.eps, k, w.target_ids, workspace=ws))
    P.compare(got, reference(w, k), k, label="longer call's workspace")


@pytest.mark.parametrize("N,d,V,k", [(100, 256, 9000, 20), (128, 320, 3000, 32)])
def test_same_logits_as_the_256_row_kernel(N, d, V, k):
    """K order and matrix instruction are the same, so ids and their order are; the softmax sums run over other
    parts: a relative 2^-24 for each of the at most log2(V) + 16 additions in sequence, under 1e-5."""
    say(f"few rows against many N={N} d={d} V={V} k={k}")
    w = inputs(N + 200, d, V)
    few = LL.ll_project(w.hidden[:, :N].contiguous(), w.gamma, w.W_U, w.cfg.eps, k, w.target_ids[:N].contiguous())
    many = LL.ll_project(w.hidden, w.gamma, w.W_U, w.cfg.eps, k, w.target_ids)
    assert torch.equal(few[0], many[0][:N])
    for a, b in zip(few[1:], many[1:]):
        torch.testing.assert_close(a, b[:N], rtol=1e-5, atol=1e-5)


@pytest.mark.parametrize("N,V,k", [(70, 9000, 20), (128, 70000, 32), (11, 40000, 5)])
def test_lists_that_overflow(N, V, k):
    """Many equal logits (all-zero rows, one repeated vocabulary row) and best entries that sit in one lane: more entries
    reach a part's threshold than its list holds."""
    say(f"few rows, overflowing lists N={N} V={V} k={k}")
    w = inputs(N, 128, V)
    w.hidden[0, 1] = 0
    w.W_U[V // 3:V // 3 + 2000] = 8.0 * w.W_U[V // 3]       # the best 2000 of about half the rows
    w.W_U[V // 2:V // 2 + 4] *= 3.0
    got = P.to_numpy(LL.ll_project(w.hidden, w.gamma, w.W_U, w.cfg.eps, k, w.target_ids))
    ref = reference(w, k)
    P.compare(got, ref, k, label="overflow")
    assert list(got["topk_ids"][1]) == list(range(k))
    ids = got["topk_ids"].astype(np.int64)                  # equal logits in ascending id
    tie = ref["topk_logits"][:, 1:] == ref["topk_logits"][:, :-1]
    assert tie.sum() > k and np.all(ids[:, 1:][tie] > ids[:, :-1][tie])


@pytest.mark.parametrize("low", [torch.finfo(torch.float32).min, -3.2e38])
@pytest.mark.parametrize("N,V,k", [(40, 5000, 5), (100, 40000, 20)])
def test_tokens_masked_by_the_lowest_bias_are_listed_last(N, V, k, low):
    """A bias that leaves fewer than k tokens: the others have probability zero, but they are tokens, equal ones."""
    say(f"few rows, masked N={N} V={V} k={k} low={low}")
    w = inputs(N, 128, V)
    allowed = np.array([17, V // 2, V - 1])
    bias = torch.full((V,), low, device=DEV)
    bias[allowed.tolist()] = 0.25
    ids, p, logp, ent = (x.cpu().numpy() for x in LL.ll_project(w.hidden, w.gamma, w.W_U, w.cfg.eps, k, w.target_ids, bias=bias))
    z = reference(w, 1)["z"][:, allowed]
    order = np.argsort(-z, axis=1)
    want = np.exp(np.take_along_axis(z, order, 1) - z.max(1, keepdims=True))
    want /= want.sum(1, keepdims=True)
    assert np.array_equal(ids[:, :3], allowed[order])
    assert np.array_equal(ids[:, 3:], np.tile(np.setdiff1d(np.arange(k), allowed)[:k - 3], (N, 1)))
    assert np.abs(p[:, :3] - want).max() < 1e-4 and np.all(p[:, 3:] == 0)     # (the logits' fp32 sums: some 1e-6 of their size)
    assert np.abs(ent + (want * np.log(want)).sum(1)).max() < 1e-3
    masked = ~np.isin(w.target_ids.cpu().numpy(), allowed)
    assert np.all(logp[masked] < -1e38)


def like_tokens(w, n):
    """The last n tokens are near copies of one with long logits: every row's best (or worst) entries sit together."""
    V = w.cfg.V
    w.W_U[V - n:] = (4.0 * w.W_U[V - n].float() + 0.25 * w.W_U[V - n:].float()).to(torch.bfloat16)


@pytest.mark.parametrize("N,d,V,k", [
    (3, 128, 1000, 32),        # eight parts of 128 ids
    (16, 192, 50257, 32),      # longest list: the threshold is the least of the partial maxima
    (81, 128, 128256, 32),
    (128, 64, 40000, 21),
    (37, 128, 151936, 10),     # five groups a wavefront
])
def test_best_entries_that_sit_together(N, d, V, k):
    say(f"few rows, like tokens N={N} d={d} V={V} k={k}")
    w = inputs(N, d, V, seed=23)
    w.hidden[0, N // 2] = 0
    like_tokens(w, 300)
    got = P.to_numpy(LL.ll_project(w.hidden, w.gamma, w.W_U, w.cfg.eps, k, w.target_ids))
    P.compare(got, reference(w, k), k, label="together")
    assert list(got["topk_ids"][N // 2]) == list(range(k))


def call_time(w, rows, k):
    hidden, target = w.hidden[:, :rows].contiguous(), w.target_ids[:rows].contiguous()
    ws = torch.empty(LL.ll_workspace_bytes(rows, w.cfg.d, w.cfg.V, k), dtype=torch.uint8, device=DEV)
    out = LL.ll_project(hidden, w.gamma, w.W_U, w.cfg.eps, k, target, workspace=ws)
    times = []
    for _ in range(9):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(10):
            LL.ll_project(hidden, w.gamma, w.W_U, w.cfg.eps, k, target, workspace=ws, out=out)
        b.record()
        b.synchronize()
        times.append(a.elapsed_time(b) / 10)
    return sorted(times)[4]


@pytest.mark.parametrize("rows,V,k,what", [(96, 50257, 32, "longest list"), (96, 128256, 32, "longest list"), (96, 50257, 10, "zero rows"),
                                           (96, 50257, 10, "like tokens")])
def test_full_lists_cost_no_more_than_the_256_row_kernel(rows, V, k, what):
    """(One row more than this kernel takes.  Half as much again is allowed for the clock's moods.)"""
    say(f"few rows, time of {what}, {rows} rows, V={V} k={k}")
    w = inputs(129, 256, V)
    if what == "zero rows":
        w.hidden[0, ::16] = 0
    if what == "like tokens":
        like_tokens(w, 256)
    few, many = call_time(w, rows, k), call_time(w, 129, k)
    say(f"few rows, time of {what}: {1e3 * few:.1f} us, 129 rows {1e3 * many:.1f} us")
    assert few < 1.5 * many


@pytest.mark.parametrize("d,V,shift,past_the_caches", [
    (2048, 30000, 0, True),    # 123 MB, which the Infinity Cache could hold, but not beside twice its bytes
    (2048, 21846, 0, True),    # 3 KB more than a third of the Infinity Cache
    (2048, 21845, 0, False),
    (256, 5000, 0, False),
    (2048, 30000, 8, False),   # the first's rows, from 16 bytes into a line on
    (1608, 30000, 0, False),   # rows that are not whole lines
])
def test_how_w_is_read_depends_on_its_lines_and_size(d, V, shift, past_the_caches):
    say(f"few rows, loads of W_U d={d} V={V} shift={shift}")
    w = inputs(16, d, V)
    W = torch.empty((V * d + shift,), dtype=torch.bfloat16, device=DEV)[shift:].view(V, d)
    W.copy_(w.W_U)
    names = kernels_of(lambda: LL.ll_project(w.hidden, w.gamma, W, w.cfg.eps, 5, w.target_ids))
    assert len(names) == 3 and names[0].startswith("ll_norm_panel_kernel") and names[1].startswith("ll_lens_few_kernel")
    assert names[1].split(">")[0].endswith("true" if past_the_caches else "false")


@pytest.mark.parametrize("V,past_the_caches", [(3000, True), (20000, False), (60000, True)])
def test_a_sweep_of_one_strength_reads_w_where_it_has_just_left_it(V, past_the_caches):
    """12 MB stay in the L2s and 246 MB are more than the Infinity Cache keeps beside the rest; 82 MB are there."""
    say(f"few rows, sweep of one strength V={V}")
    w = inputs(16, 2048, V)
    v = torch.randn((2048,), generator=torch.Generator(device=DEV).manual_seed(5), device=DEV)
    names = kernels_of(lambda: LL.ll_steer_sweep(w.hidden.reshape(16, -1), w.gamma, w.W_U, w.cfg.eps, v / v.norm(), [2.0], w.target_ids))
    assert names[0].startswith("ll_unembed_direction_kernel") and names[2].startswith("ll_lens_few_kernel")
    assert names[2].split(">")[0].endswith("true" if past_the_caches else "false")


@pytest.mark.parametrize("V", [777, 4096, 8000, 16384, 16400])
@pytest.mark.parametrize("N", [17, 48, 81, 128])
def test_rows_dealt_to_several_workgroups_are_those_of_calls_of_sixteen(N, V):
    """A small vocabulary's parts go to several workgroups, some rows each: the same bits as from calls of 16 rows, which have one a part."""
    say(f"few rows, dealt N={N} V={V}")
    d, k = 328, 7
    w = WL.make_workload(WL.LensConfig("dealt", L=1, T=N, d=d, V=V, k=k), DEV, seed=29)
    bias = 0.5 * torch.randn((V,), generator=torch.Generator(device=DEV).manual_seed(8), device=DEV)
    h = w.hidden.reshape(N, d)
    whole = LL.ll_project(h, w.gamma, w.W_U, w.cfg.eps, k, w.target_ids, bias=bias)
    for r in range(0, N, 16):
        part = LL.ll_project(h[r:r + 16].contiguous(), w.gamma, w.W_U, w.cfg.eps, k, w.target_ids[r:r + 16].contiguous(), bias=bias)
        for a, b in zip(whole, part):
            assert torch.equal(a[r:r + 16], b)
