"""Sweeps whose contraction forms u = W_U v itself, from three bf16 rows behind the lens rows of every block, in both forms: against
the CPU oracle, and against the kernels that take u from a pass of its own."""
import numpy as np
import pytest
import torch

from paper_2604_06483_amd import binding as LL
from paper_2604_06483_amd import workloads as WL
from tests.conftest import kernels_of, say
from tests.test_gpu_sweep import ALPHAS9, direction
from tests.test_gpu_sweep_forms import check

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def is_whole(call):
    names = [n for n in kernels_of(call) if n.startswith("ll_lens_gemm")]
    assert len({"WholeSweep" in n for n in names}) == 1, names
    return "WholeSweep" in names[0]


def workload(N, d, V, seed=61):
    w = WL.make_workload(WL.LensConfig("whole", L=1, T=N, d=d, V=V, k=1), DEV, seed=seed)
    return w, w.hidden.reshape(N, d)


@pytest.mark.parametrize("N,d,V,n_alpha,k", [
    (253, 64, 777, 3, None),      # a full block; one K stage, a vocabulary that ends within a tile
    (507, 72, 20000, 2, 3),       # three blocks, the last of one row; a ragged hidden size
    (1, 128, 300, 2, None),       # one row
    (1500, 64, 50257, 1, None), (300, 128, 20000, 1, None),   # one strength: a projection; a sweep
    (2000, 128, 33000, 3, 2),     # eight blocks
])
def test_general_form_matches_oracle(N, d, V, n_alpha, k):
    say(f"whole sweep, general N={N} d={d} V={V} A={n_alpha} k={k}")
    check(N, d, V, ALPHAS9[:n_alpha], k, 1.0, "whole, general", rows=np.unique(np.r_[0:min(N, 260), N - 1]))
    if n_alpha > 1 or N == 300:
        w, h = workload(N, d, V)
        assert is_whole(lambda: LL.ll_steer_sweep(h, w.gamma, w.W_U, w.cfg.eps, direction(d), ALPHAS9[:n_alpha], None, k=k))


@pytest.mark.parametrize("k", [None, 3])
@pytest.mark.parametrize("N,d,V,alphas,length", [
    (253, 704, 50000, ALPHAS9, 1.0),              # one block, one tile a split
    (300, 712, 50257, ALPHAS9[:8], 1.0),          # ragged hidden size; two blocks, two tiles; no zero strength of nine
    (1012, 704, 50257, ALPHAS9, 20.0),            # four full blocks
    (200, 704, 50257, [4.0, -3.0, -2.0, -1.0, 0.5, 1.0, 2.0, 3.0, 0.0], 50.0),   # shifts up to 17: the sample leaves it open
    (200, 704, 50257, ALPHAS9, 120.0),            # shifts of 40: the sample has it
])
def test_factored_form_matches_oracle(N, d, V, alphas, length, k):
    say(f"whole sweep N={N} d={d} V={V} A={len(alphas)} k={k} length={length}")
    check(N, d, V, alphas, k, length, "whole", rows=np.unique(np.r_[0:8, N // 2:N // 2 + 8, min(N, 256) - 8:min(N, 256), N - 8:N]))
    w, h = workload(N, d, V)
    assert is_whole(lambda: LL.ll_steer_sweep(h, w.gamma, w.W_U, w.cfg.eps, direction(d), alphas, None, k=k))


def u_of(n, h, gamma, W, v, alphas):
    """The u that a call of n rows leaves at the start of its workspace, as bits."""
    ws = torch.empty(LL.ll_steer_sweep_workspace_bytes(n, h.shape[1], W.shape[0], len(alphas), 1), dtype=torch.uint8, device=DEV)
    LL.ll_steer_sweep(h[:n].contiguous(), gamma, W, 1e-5, v, alphas, None, workspace=ws)
    return ws[:4 * W.shape[0]].view(torch.int32).clone()


def both(h, gamma, W, v, alphas, target, k):
    """Of the first 253 rows: from a call of just these (u within), and from one of 256 (a block more otherwise: u before)."""
    one = lambda n: LL.ll_steer_sweep(h[:n].contiguous(), gamma, W, 1e-5, v, alphas, target[:n].contiguous(), k=k)
    assert is_whole(lambda: one(253)) and not is_whole(lambda: one(256))
    return one(253), tuple(t[:, :253] for t in one(256))


@pytest.mark.parametrize("k", [None, 3])
@pytest.mark.parametrize("what", ["plain", "one large shift", "one large shift, sampled", "large shifts", "infinite W", "NaN in W", "infinite v", "NaN in v", "no direction"])
def test_as_with_u_from_a_pass_of_its_own(what, k):
    """The forms agree to fp32 sums in another order, and to the places of what is no number.  "One large shift" is one token that the
    sample does not meet: the factored form leaves it out; sampled, the general form runs, on u of its own."""
    say(f"whole sweep, both ways: {what} k={k}")
    d, V = 704, 50257
    w, h = workload(256, d, V)
    v, W = direction(d), w.W_U
    if what.startswith("one large shift"):
        v = v * 0.5                               # (short enough for u of the contraction)
        W[0 if "sampled" in what else -30] = (24.0 * v).to(torch.bfloat16)    # 6, times 4
    if what == "large shifts":
        v = v * 400.0
    if what == "infinite W":
        W[40000, 5] = float("inf")
        v[5] = 0.25            # its second and third rows are zero
    if what == "NaN in W":
        W[40000, 5] = float("nan")
    if what == "infinite v":
        v[5] = -float("inf")
    if what == "NaN in v":
        v[5] = float("nan")
    if what == "no direction":
        v = torch.zeros_like(v)
    a, b = both(h, w.gamma, W, v, ALPHAS9, w.target_ids, k)
    finite = torch.isfinite(b[3]) & torch.isfinite(a[3])
    assert torch.equal(torch.isnan(a[3]), torch.isnan(b[3])) and torch.equal(torch.isnan(a[2]), torch.isnan(b[2]))
    if finite.any():
        assert (a[0] != b[0])[finite].float().mean() < 1e-3        # near-ties
        scale = float(b[3][finite].abs().max()) + 20.0             # sums of logits and shifts of this size round in the last place
        for x, y in zip(a[1:], b[1:]):
            torch.testing.assert_close(x[finite], y[finite], rtol=4e-5, atol=2e-6 * scale)
    assert int(a[0].min()) >= 0 and torch.equal(a[0][~finite] < V, b[0][~finite] < V)


def test_captured_and_replayed():
    """One graph of it, replayed on other inputs in the same buffers: the results of a call."""
    say("whole sweep, captured")
    N, d, V = 300, 704, 50257
    w, h = workload(N, d, V)
    v, ws = direction(d), torch.empty(LL.ll_steer_sweep_workspace_bytes(N, d, V, 9, 1), dtype=torch.uint8, device=DEV)
    call = lambda: LL.ll_steer_sweep(h, w.gamma, w.W_U, w.cfg.eps, v, ALPHAS9, w.target_ids, workspace=ws)
    call()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        out = call()
    for length in (1.0, 400.0, 30.0):     # the factored form, the general one, the factored one
        v.copy_(direction(d) * length)
        h.copy_(h.roll(1, 0))
        want = [t.clone() for t in call()]
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(x, y) for x, y in zip(out, want))


@pytest.mark.parametrize("d,n_alpha,length,own", [
    (4096, 3, 34.0, False),   # the general form, u from the direction kernel
    (1024, 9, 17.0, False),   # the factored one
    (1024, 9, 0.72, True), (4096, 3, 1.4, True),   # 0.09 of the rows' length: u of the contraction, in both forms
    (4096, 9, 1.0, True),
])
def test_a_long_direction_adds_no_error(d, n_alpha, length, own):
    """Against 64 bits, rows given as bf16: the target's log-probability is no further off than with u from a pass of its own but
    for what the bound below allows for chance), whichever u it is."""
    say(f"whole sweep, error d={d} A={n_alpha} length={length}")
    N, V = 256, 50257
    g = torch.Generator(device=DEV).manual_seed(9)
    h = torch.randn((N, d), generator=g, device=DEV).to(torch.bfloat16)
    W = (0.02 * torch.randn((V, d), generator=g, device=DEV)).to(torch.bfloat16)
    v = direction(d) * length
    alphas = [4.0 * (2.0 * a / (n_alpha - 1) - 1.0) for a in range(n_alpha)]
    target = torch.randint(0, V, (N,), generator=g, device=DEV, dtype=torch.int32)
    within, before = both(h, None, W, v, alphas, target, None)
    assert own != torch.equal(*(u_of(n, h, None, W, v, alphas) for n in (253, 256)))
    Wt = W.double().t().contiguous()
    z, u = h[:253].double() @ Wt, v.double() @ Wt
    off = [[], []]
    for a, alpha in enumerate(alphas):
        q = torch.log_softmax(z + alpha * u, -1).gather(1, target[:253].long()[:, None])[:, 0]
        for o, got in zip(off, (within, before)):
            o.append(got[2][a].double() - q)
    rms = [float(torch.stack(o).square().mean().sqrt()) for o in off]
    # u of the contraction has an error of its own, as large beside the logits' as alpha v is beside the rows (r): it adds r^2 / 2, and by chance,
    # over 253 rows with a token each, up to 3 r / sqrt(253).  A u that is the same: sums in another order.
    r = 4.0 * length / d ** 0.5
    assert rms[0] <= (1.0 + r * r / 2 + 3.0 * r / 253 ** 0.5 if own else 1.01) * rms[1], rms


@pytest.mark.parametrize("d,n_alpha,shift", [(2048, 9, 13.0), (2056, 9, 12.0), (4096, 9, 13.0), (4096, 3, 13.0),
                                             (2048, 9, 21.0), (4096, 9, 30.0)])      # (left out of the factored form)
def test_a_token_along_the_direction_adds_no_error(d, n_alpha, shift):
    """Against 64 bits, eight tokens that the sample misses and whose unembedding rows lie along the direction, in a vocabulary whose u are
    small: what is off in their log-probabilities and in the entropy is no more than with u from a pass of its own."""
    say(f"whole sweep, along the direction d={d} A={n_alpha} shift={shift}")
    N, V = 256, 50257
    g = torch.Generator(device=DEV).manual_seed(19)
    h = torch.randn((N, d), generator=g, device=DEV).to(torch.bfloat16)
    W = (0.02 * torch.randn((V, d), generator=g, device=DEV)).to(torch.bfloat16)
    v = direction(d) * (0.015 * d ** 0.5)
    tokens = torch.arange(8, device=DEV) * 32 * 190 + 1000        # (the sample is one row in 32, from 0 on)
    W[tokens] += (v * (shift / 4.0 / float(v.square().sum()))).to(torch.bfloat16)
    alphas = [4.0 * (2.0 * a / (n_alpha - 1) - 1.0) for a in range(n_alpha)]
    target = tokens[torch.arange(N, device=DEV) % 8].to(torch.int32)
    within, before = both(h, None, W, v, alphas, target, None)
    Wt = W.double().t().contiguous()
    z, u = h[:253].double() @ Wt, v.double() @ Wt
    off = [[], []]
    for a, alpha in enumerate(alphas):
        q = torch.log_softmax(z + alpha * u, -1)
        entropy, q = -(q.exp() * q).sum(-1), q.gather(1, target[:253].long()[:, None])[:, 0]
        for o, got in zip(off, (within, before)):
            o.append(torch.stack([got[2][a].double() - q, got[3][a].double() - entropy]))
    rms = [torch.stack(o, 1).square().mean((1, 2)).sqrt().tolist() for o in off]
    # (two sums of the same logits in fp32, 253 rows and eight tokens: a tenth for chance)
    assert all(x <= 1.1 * y for x, y in zip(*rms)), rms


@pytest.mark.parametrize("n_alpha", [3, 9])
@pytest.mark.parametrize("length,rows,own", [
    (0.09, "all", True), (0.11, "all", False),
    (0.09, "one short", False), (0.09, "one zero", False), (0.09, "short", False), (0.0045, "short", True),
    (0.09, "gamma", True), (0.18, "gamma", True), (0.22, "gamma", False), (0.09, "eps", False), (0.0, "one zero", True),
])
def test_where_u_comes_from(length, rows, own, n_alpha):
    """The contraction's u only beside rows that are ten times as long as alpha v, by the rows themselves: else the direction kernel's, to the bit."""
    say(f"whole sweep, source of u length={length} rows={rows} A={n_alpha}")
    N, d, V = 256, 1024, 50257
    g = torch.Generator(device=DEV).manual_seed(29)
    h = torch.randn((N, d), generator=g, device=DEV)
    h /= h.square().mean(-1, keepdim=True).sqrt()
    gamma = None
    if rows in ("gamma", "eps"):
        gamma = torch.full((d,), 2.0, device=DEV, dtype=torch.bfloat16)
    if rows == "eps":
        h[17] *= 1e-4                     # beside eps = 1e-5 next to nothing after the norm too
    if rows == "short":
        h *= 0.05
    if rows.startswith("one"):
        h[252] *= 0.5 if rows == "one short" else 0.0
    h = h.to(torch.bfloat16)
    W = (0.02 * torch.randn((V, d), generator=g, device=DEV)).to(torch.bfloat16)
    v = direction(d) * (length * d ** 0.5 / 4.0)
    alphas = [4.0 * (2.0 * a / (n_alpha - 1) - 1.0) for a in range(n_alpha)]
    both(h, gamma, W, v, alphas, torch.zeros((N,), device=DEV, dtype=torch.int32), None)     # (which is which)
    within, before = (u_of(n, h, gamma, W, v, alphas) for n in (253, 256))
    assert torch.equal(within, before) == (not own or length == 0.0)


@pytest.mark.parametrize("N,d,V,n_alpha,expected", [
    (256, 4096, 131072, 2, False),    # a second block for three rows: four tiles a workgroup instead of two
    (253, 4096, 131072, 2, True), (1000, 704, 50257, 9, True),
    (256, 704, 20000, 2, True),       # a second block, and still one tile
])
def test_never_a_tile_more(N, d, V, n_alpha, expected):
    say(f"whole sweep, which N={N} d={d} V={V} A={n_alpha}")
    w, h = workload(N, d, V)
    assert is_whole(lambda: LL.ll_steer_sweep(h, w.gamma, w.W_U, w.cfg.eps, direction(d), ALPHAS9[:n_alpha], None)) == expected


def unsampled(V, tile, at):
    """An id of the tile that the sample (one row in 32) passes by, the one at `at` or just behind."""
    sampled = {s * V // ((V + 31) // 32) for s in range((V + 31) // 32)}
    i = tile * 256 + at
    return i + 1 if i in sampled else i


def with_large_shifts(N, d, V, tiles, seed=37):
    """A sweep with a token of a large shift, unmet by the sample, in each of these tiles."""
    w, h = workload(N, d, V, seed)
    v, W = direction(d) * (0.015 * d ** 0.5), w.W_U
    ids = [min(unsampled(V, t, 67 * i % 250), V - 1) for i, t in enumerate(tiles)]
    assert len(set(ids)) == len(ids)
    for i, t in enumerate(ids):
        W[t] = (v * ((-8.0 if i % 3 == 1 else 6.5) / float(v.square().sum()))).to(torch.bfloat16)    # times 4: beyond 20
    return w, h, v, ids


EIGHT = [a for a in ALPHAS9 if a != 0.0]


@pytest.mark.parametrize("k", [None, 1, 3, 4])
@pytest.mark.parametrize("N,d,tiles,n_alpha", [
    (1012, 704, [0], 8), (1012, 704, [3], 8), (1012, 712, [196], 8),      # a split's first tile, its last, the vocabulary's last (a part of one)
    (1012, 704, [0, 2, 3, 40, 41, 77], 8), (1012, 704, [0, 2, 3, 40, 41, 77], 9),
    (1012, 704, [0, 1, 2, 3] * 4, 9),                                     # as many as a split has place for
    (1012, 704, [0, 1, 2, 3] * 5, 9),                                     # more: the general form for all
    (253, 704, [5, 100, 196], 9), (300, 704, [0, 1, 195, 196], 6),        # one tile a split; a second block of few rows
    (1012, 704, range(197), 9),                                           # one in every tile
])
def test_tokens_that_are_left_out(N, d, tiles, n_alpha, k):
    """Tokens of large shifts that the sample misses: the factored form leaves them out, the merge adds them.  Against nine strengths none of which is
    zero, which take u and its largest from a pass of its own and so the general form for all."""
    say(f"whole sweep, left out N={N} d={d} tokens={len(tiles)} A={n_alpha} k={k}")
    V = 50257
    w, h, v, ids = with_large_shifts(N, d, V, tiles)
    target = w.target_ids.clone()
    target[::3] = torch.tensor(ids, device=DEV, dtype=torch.int32)[torch.arange(len(target[::3]), device=DEV) % len(ids)]
    target[1::3] = torch.tensor([t // 256 * 256 + 7 for t in ids], device=DEV, dtype=torch.int32)[torch.arange(len(target[1::3]), device=DEV) % len(ids)]
    target[4] = V
    call = lambda alphas: LL.ll_steer_sweep(h, w.gamma, w.W_U, w.cfg.eps, v, alphas, target, k=k)
    alphas = {6: EIGHT[2:], 8: EIGHT, 9: ALPHAS9}[n_alpha]
    nonzero = [x for x in alphas if x != 0.0]
    others = (nonzero + [0.125] * 9)[:9]
    assert is_whole(lambda: call(alphas)) and not is_whole(lambda: call(others))
    a, b = call(alphas), [t[:len(nonzero)] for t in call(others)]
    if n_alpha == 9:   # strength 0: the projection
        plain = LL.ll_project(h, w.gamma, w.W_U, w.cfg.eps, k or 1, target)
        plain = [plain[0] if k else plain[0][:, 0], plain[1] if k else plain[1][:, 0], *plain[2:]]
        b = [torch.cat([x[:4], y[None], x[4:]]) for x, y in zip(b, plain)]
    assert (a[0] != b[0]).float().mean() < 1e-3        # near-ties
    scale = float(b[3].abs().max()) + 20.0             # sums of logits and shifts of this size round in the last place
    for x, y in zip(a[1:], b[1:]):
        torch.testing.assert_close(x, y, rtol=4e-5, atol=2e-6 * scale, equal_nan=True)
    assert torch.equal(torch.isnan(a[2]), torch.isnan(b[2])) and int(torch.isnan(a[2]).sum()) == n_alpha


def test_equal_logits_of_tokens_left_out_keep_their_order():
    """The same unembedding row several times, of a large shift, in one tile and in several splits: listed by id."""
    say("whole sweep, equal logits of tokens left out")
    N, d, V = 1012, 704, 50257
    g = torch.Generator(device=DEV).manual_seed(3)
    W = 0.02 * torch.randn((V, d), generator=g, device=DEV)
    v = direction(d) * (0.015 * d ** 0.5)
    same = [unsampled(V, 4, 9), unsampled(V, 5, 190), unsampled(V, 5, 252), unsampled(V, 70, 3)]
    W[same] = 3.0 * torch.randn((d,), generator=g, device=DEV) / d ** 0.5 + v * (6.5 / float(v.square().sum()))
    h = 20.0 * W[same[0]] + 0.1 * torch.randn((N, d), generator=g, device=DEV)
    h = (h - (h @ v)[:, None] * v / v.square().sum()).to(torch.bfloat16)
    W = W.to(torch.bfloat16)
    ids4, p, _, _ = LL.ll_steer_sweep(h, None, W, 1e-5, v, EIGHT, None, k=4)
    assert (ids4 == torch.tensor(same, device=DEV)).all() and torch.equal(p[..., 0], p[..., 3])


def durations_of(call):
    """Of this library's kernels that call() launches, in order: name and microseconds."""
    from torch.profiler import ProfilerActivity, profile
    with profile(activities=[ProfilerActivity.CUDA]) as prof:
        call()
        torch.cuda.synchronize()
    return [(e.name, e.device_time) for e in sorted(prof.events(), key=lambda e: e.time_range.start) if "::ll_" in e.name]


@pytest.mark.parametrize("k", [None, 3])
def test_tokens_of_large_shifts_cost_no_second_pass(k):
    """What is launched behind the factored form returns at once, though there are such tokens."""
    say(f"whole sweep, the cost of tokens left out k={k}")
    w, h, v, _ = with_large_shifts(1012, 704, 50257, [17, 130])
    call = lambda: LL.ll_steer_sweep(h, w.gamma, w.W_U, w.cfg.eps, v, EIGHT, None, k=k)
    call()
    factored, general = (t for name, t in durations_of(call) if "ll_lens_gemm" in name)
    assert general < 0.3 * factored, (factored, general)
