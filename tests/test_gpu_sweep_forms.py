"""The two forms of the steering sweep's epilogue (e^(alpha u) as a table factor; every shifted logit exponentiated, for
shifts past 20) and its splits of the vocabulary, against the CPU oracle."""
import numpy as np
import pytest
import torch

import oracle.lens_oracle as O
from paper_2604_06483_amd import binding as LL
from paper_2604_06483_amd import workloads as WL
from tests.conftest import say
from tests.test_gpu_sweep import ALPHAS9, compare_sweep, direction

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def check(N, d, V, alphas, k, length, label, rows=None):
    cfg = WL.LensConfig("form", L=1, T=N, d=d, V=V, k=1, n_outliers=2 if d > 100 else 0, outlier_scale=20.0)
    w = WL.make_workload(cfg, DEV, seed=41)
    v = direction(d) * length
    hidden = w.hidden.reshape(N, d)
    got = LL.ll_steer_sweep(hidden, w.gamma, w.W_U, cfg.eps, v, alphas, w.target_ids, k=k)
    torch.cuda.synchronize()
    rows = np.arange(N) if rows is None else rows
    inputs = (WL.bf16_bits(hidden)[rows], WL.bf16_bits(w.gamma), WL.bf16_bits(w.W_U), cfg.eps, v.cpu().numpy(), alphas)
    u = O.bf16_bits_to_f64(inputs[2]) @ inputs[4].astype(np.float64)
    want = O.steer_sweep(*inputs, w.target_ids.cpu().numpy()[rows], k=k or 1)
    compare_sweep(got, want, rows, label, inputs)
    return max(abs(a) for a in alphas) * np.abs(u).max()


# (u is Gaussian with sigma 0.02 times v's length: its largest entry of some thousand is about four sigma)
@pytest.mark.parametrize("k", [None, 2, 4])
@pytest.mark.parametrize("length,general", [(50.0, False), (400.0, True)])
@pytest.mark.parametrize("d", [256, 200])
def test_both_forms(k, length, general, d):
    say(f"sweep form general={general} d={d} k={k}")
    # a logit of some 20 is held to 2^-24 of itself and of its shift: the tolerances stand
    assert (check(300, d, 3001, ALPHAS9, k, length, f"form {length}") > 20.0) == general


@pytest.mark.parametrize("N,d,V,n_alpha,k", [
    (40, 64, 40000, 9, 3),       # 157 splits of one tile
    (10, 128, 70000, 2, None),   # 137 splits of two tiles: bounds are exchanged
    (300, 64, 66000, 9, 4),      # two row blocks, 86 splits of three tiles
    (1000, 64, 20000, 7, None),  # four row blocks
    (260, 192, 263, 9, 3),       # a last tile of seven ids
    (70, 128, 5000, 4, None), (70, 128, 5000, 5, None),   # one tile a split, the form without tables
    (70, 128, 5000, 3, 4), (70, 128, 5000, 4, 4), (70, 128, 5000, 1, 2),   # the same; with tables; few rows of one strength: a projection
    (129, 72, 5000, 1, None), (300, 64, 140000, 1, 3), (300, 72, 140000, 1, None),   # one strength: the sweep's own kernel; projections
    (70, 128, 5000, 6, None), (70, 128, 5000, 7, None), (70, 128, 5000, 5, 4), (70, 128, 5000, 6, 4),   # without tables; with
    (10, 128, 70000, 5, None), (10, 128, 70000, 6, None), (10, 128, 70000, 4, 3), (10, 128, 70000, 5, 3),   # the same, two tiles
    (260, 64, 140000, 3, 3), (260, 64, 140000, 4, 3),   # five tiles, without tables (test_gpu_routes.py has either side of each line)
])
def test_splits(N, d, V, n_alpha, k):
    say(f"sweep splits N={N} d={d} V={V} A={n_alpha} k={k}")
    check(N, d, V, ALPHAS9[:n_alpha], k, 1.0, "splits")


@pytest.mark.parametrize("k", [None, 3])
@pytest.mark.parametrize("alphas", [
    [-4.0, -3.0, -2.0, -1.0, 0.5, 1.0, 2.0, 3.0, 4.0],    # none is zero: a second table
    [0.0, -3.0, -2.0, -1.0, 0.5, 1.0, 2.0, 3.0, 4.0],     # one is: its sums apart from the products; at either end, and beside another
    [-4.0, -3.0, -2.0, -1.0, 0.5, 1.0, 2.0, 3.0, 0.0],
    [-4.0, -3.0, 0.0, -1.0, 0.5, 1.0, -0.0, 3.0, 4.0],
    [-4.0, -3.0, 0.0, -1.0, 0.5, 1.0, 2.0, 3.0],          # eight: as any other
])
def test_nine_strengths_with_and_without_zero(alphas, k):
    say(f"sweep strengths {alphas} k={k}")
    check(300, 128, 7000, alphas, k, 1.0, "strengths")
    check(300, 72, 5003, alphas, k, 30.0, "strengths, ragged")


@pytest.mark.parametrize("N,d,V,n_alpha,k", [
    (4200, 64, 100000, 9, 3),     # 17 row blocks, 15 splits of 27 tiles: 432 groups of 16 ids a sum
    (1500, 128, 50257, 8, None),  # 40 splits of five tiles
    (300, 200, 3001, 9, 4),       # one tile a split
])
def test_sums_have_the_error_of_single_roundings(N, d, V, n_alpha, k):
    """The softmax sums against 64 bits, rows given as bf16 so that only the logits and the sums round.  A sum of the G groups of
    a split rounds G times, to nearest: a relative sqrt(G) 2^-24 at most in the root mean square, and no bias to speak of.  The
    entropy is that of the sums' quotient, weighed logits of up to 30 or so, and a logit's own sum rounds d times."""
    say(f"sweep sums N={N} d={d} V={V} A={n_alpha} k={k}")
    g = torch.Generator(device=DEV).manual_seed(51)
    hidden = torch.randn((N, d), generator=g, device=DEV).to(torch.bfloat16)
    W = (torch.randn((V, d), generator=g, device=DEV) * (5.0 / d ** 0.5)).to(torch.bfloat16)
    v, alphas = direction(d), ALPHAS9[:n_alpha]
    target = torch.randint(0, V, (N,), generator=g, device=DEV, dtype=torch.int32)
    _, _, logp, ent = LL.ll_steer_sweep(hidden, None, W, 1e-5, v, alphas, target, k=k)
    rows = torch.randint(0, N, (256,), generator=g, device=DEV)
    Wt = W.double().t().contiguous()
    z = hidden[rows].double() @ Wt
    u = v.double() @ Wt
    splits = max(1, 256 // ((N + 255) // 256))
    groups = -(-(-(-V // 256)) // splits) * 16
    for a, alpha in enumerate(alphas):
        w = z + alpha * u
        lse = torch.logsumexp(w, -1)
        lp = w - lse[:, None]
        p = lp.exp()
        of_logits = 2.0 ** -24 * d ** 0.5 * 5.0 + 2.0 ** -23 * float(w.abs().max())   # of a logit and of its shift
        of_sums = 2.0 ** -24 * groups ** 0.5
        err = logp[a, rows].double() - lp.gather(1, target[rows].long()[:, None])[:, 0]
        assert float(err.square().mean().sqrt()) <= of_logits + of_sums
        weighed = float((p * w).sum(-1).abs().max())
        err = ent[a, rows].double() + (p * lp).sum(-1)
        assert float(err.square().mean().sqrt()) <= of_logits + of_sums * weighed, (alpha, float(err.mean()))


@pytest.mark.parametrize("k", [None, 3, 4])
@pytest.mark.parametrize("N,d,V", [
    (300, 128, 66000),   # two row blocks, 86 splits of three tiles
    (300, 200, 66000),   # the same on the kernel for ragged hidden sizes
    (40, 64, 40000),     # one tile a split: what a list loses depends on which split came first
    (10, 128, 70000),    # two tiles a split
])
def test_equal_logits_are_listed_in_id_order(N, d, V, k):
    """Rows whose shifted logits are all zero (an all-zero row at strength 0, any row of zeros with no direction) and tokens
    that tie across splits: the k-th best equals the bound that the splits share."""
    say(f"sweep ties N={N} d={d} V={V} k={k}")
    w = WL.make_workload(WL.LensConfig("ties", L=1, T=N, d=d, V=V, k=1), DEV, seed=42)
    hidden = w.hidden.reshape(N, d)
    hidden[[0, 7, N - 1]] = 0
    listed = k or 1

    def uniform(got, a, row):
        ids, p, _, ent = (None if x is None else x[a, row].cpu().numpy() for x in got)
        assert np.array_equal(np.atleast_1d(ids), np.arange(listed)), ids
        # one rounding each of the sum, its logarithm and the probability's exponent (log V of magnitude 11)
        assert np.abs(p * V - 1.0).max() < 1e-5 and abs(ent - np.log(V)) < 1e-5

    got = LL.ll_steer_sweep(hidden, w.gamma, w.W_U, w.cfg.eps, direction(d), ALPHAS9, None, k=k)
    still = LL.ll_steer_sweep(hidden, w.gamma, w.W_U, w.cfg.eps, torch.zeros((d,), device=DEV), ALPHAS9, None, k=k)
    torch.cuda.synchronize()
    for row in (0, 7, N - 1):
        uniform(got, ALPHAS9.index(0.0), row)
        for a in range(len(ALPHAS9)):
            uniform(still, a, row)
    # every token three times, thousands of ids apart: lists of repeated logits, smaller id first
    w.W_U[V // 3:2 * (V // 3)] = w.W_U[:V // 3]
    w.W_U[2 * (V // 3):3 * (V // 3)] = w.W_U[:V // 3]
    w.W_U[3 * (V // 3):] = w.W_U[0]
    ids = LL.ll_steer_sweep(hidden, w.gamma, w.W_U, w.cfg.eps, direction(d), ALPHAS9, None, k=k)[0].cpu().numpy().reshape(9, N, listed)
    some = np.setdiff1d(np.arange(N), [0, 7, N - 1])
    assert ids.min() >= 0 and np.all(ids[:, some, 0] < V // 3)
    if listed > 1:
        assert np.all(ids[:, some, 1] == ids[:, some, 0] + V // 3) and np.all(ids[:, some, 2] == ids[:, some, 0] + 2 * (V // 3))


@pytest.mark.parametrize("k,limit", [(None, 1.33), (3, 1.67)])
def test_rows_of_zeros_cost_little_more_than_others(k, limit):
    """Equal logits are no candidates for a full list.  (Lists meet more groups that do hold one, whose sixteen equal logits then
    are looked at together.  The rest is for the clock's moods.)"""
    say(f"sweep, time with zero rows k={k}")
    N, d, V = 500, 256, 50257
    w = WL.make_workload(WL.LensConfig("zeros", L=1, T=N, d=d, V=V, k=1), DEV, seed=43)
    hidden, v = w.hidden.reshape(N, d), direction(d)
    ws = torch.empty(LL.ll_steer_sweep_workspace_bytes(N, d, V, 9, k or 1), dtype=torch.uint8, device=DEV)

    def call_time():
        times = []
        for _ in range(9):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            LL.ll_steer_sweep(hidden, w.gamma, w.W_U, w.cfg.eps, v, ALPHAS9, None, k=k, workspace=ws)
            a.record()
            for _ in range(5):
                LL.ll_steer_sweep(hidden, w.gamma, w.W_U, w.cfg.eps, v, ALPHAS9, None, k=k, workspace=ws)
            b.record()
            b.synchronize()
            times.append(a.elapsed_time(b) / 5)
        return sorted(times)[4]

    without = call_time()
    hidden[::64] = 0
    some = call_time()
    say(f"sweep k={k}: {1e3 * without:.1f} us, with zero rows {1e3 * some:.1f} us")
    assert some < limit * without


@pytest.mark.parametrize("k", [None, 3])
def test_a_logit_that_is_no_number_leaves_the_others_listed(k):
    """Token V / 2 overflows to +inf and back in rows 0, 2, ..: its logit there is NaN, and its shift is the largest of its group, far
    above every shifted logit of the row.  The rows' lists are those of the other tokens; rows 1, 3, .. are sound."""
    say(f"sweep, one NaN logit k={k}")
    N, d, V, odd = 300, 64, 7000, 3500
    g = torch.Generator(device=DEV).manual_seed(47)
    W = (0.05 * torch.randn((V, d), generator=g, device=DEV)).to(torch.bfloat16)
    h = torch.randn((N, d), generator=g, device=DEV).to(torch.bfloat16)
    v = torch.zeros(d, device=DEV)
    v[5] = 1.0
    W[:, 5] *= 0.2
    W[:, [0, 40]] = 0.0                              # columns of the two K halves
    h[:, 5] = 0.0
    h[::2, [0, 40]], h[1::2, [0, 40]] = 4.0, 1e-30
    W[odd, 0], W[odd, 40], W[odd, 5] = 3e38, -3e38, 4.5
    ids, p, logp, ent = LL.ll_steer_sweep(h, None, W, 1e-5, v, ALPHAS9, None, k=k)
    n = 1 if k is None else k
    ids, p = ids.reshape(len(ALPHAS9), N, n), p.reshape(len(ALPHAS9), N, n)
    z = h.double() @ W.double().t()
    z[::2, odd] = -float("inf")
    for a, alpha in enumerate(ALPHAS9):
        shifted = z + alpha * W[:, 5].double()
        best = shifted.topk(n).values
        assert 0 <= int(ids[a].min()) and int(ids[a].max()) < V
        # fp32 sums of 64 products and one shift, all below 1
        torch.testing.assert_close(shifted.gather(1, ids[a].long()), best, rtol=0, atol=64 * 2.0 ** -24)
        assert torch.isfinite(p[a, 1::2]).all() and torch.isfinite(ent[a, 1::2]).all()
        assert torch.isnan(ent[a, ::2]).all()


@pytest.mark.parametrize("k", [None, 3])
@pytest.mark.parametrize("n_alpha", [3, 9])
@pytest.mark.parametrize("d", [64, 72])
def test_rows_that_are_not_finite_leave_the_others_alone(d, n_alpha, k):
    """A NaN and an infinity in two rows of a block, in both forms: the sound rows are the bits of a call that has the row of zeros there."""
    say(f"sweep, rows that are not finite d={d} A={n_alpha} k={k}")
    N, V = 300, 9000
    cfg = WL.LensConfig("odd rows", L=1, T=N, d=d, V=V, k=1)
    w = WL.make_workload(cfg, DEV, seed=41)
    h, v = w.hidden.reshape(N, d), direction(d)
    odd = [5, 70, 299]
    h[odd] = 0
    call = lambda: LL.ll_steer_sweep(h, w.gamma, w.W_U, cfg.eps, v, ALPHAS9[:n_alpha], w.target_ids, k=k)
    want = [t.clone() for t in call()]
    h[5, 3], h[70, 0], h[299, -1] = float("nan"), float("inf"), float("-inf")
    sound = torch.ones(N, dtype=torch.bool, device=DEV)
    sound[odd] = False
    got = call()
    for a, b in zip(got, want):
        assert torch.equal(a[:, sound], b[:, sound])
    assert torch.isnan(got[3][:, odd]).all()
