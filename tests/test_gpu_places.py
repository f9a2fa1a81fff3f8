"""How the workgroups of the direct-to-LDS kernels are dealt to row blocks and vocabulary splits (groups of row blocks that share W_U's
tiles in an XCD's L2): every pair has to come up once, whatever the two numbers."""
import pytest
import torch

from paper_2604_06483_amd import binding as LL
from paper_2604_06483_amd import workloads as WL
from tests.conftest import say

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("N,V", [
    (300, 20000),     # 2 row blocks, one group
    (1537, 9000),     # 7, one group
    (1793, 9000),     # 8: two groups of four
    (2100, 7000),     # 9: three of three
    (4100, 4000),     # 17: four of four, and one
    (7900, 2300),     # 31 by 8 (and fewer) splits: each by itself
    (5400, 3000),     # 22, eleven splits: five of four, and two
])
def test_every_row_block_meets_every_split(N, V):
    say(f"places N={N} V={V}")
    d, k = 64, 4
    w = WL.make_workload(WL.LensConfig("places", L=1, T=N, d=d, V=V, k=k), DEV, seed=71)
    a = LL.ll_project(w.hidden, w.gamma, w.W_U, w.cfg.eps, k, w.target_ids)
    b = LL.ll_project(w.hidden, w.gamma, w.W_U, w.cfg.eps, k, w.target_ids, register_staged=True)   # one row block after the other
    assert (a[0] != b[0]).float().mean() < 1e-3       # near-ties that the order of the sums decides
    for x, y in zip(a[1:], b[1:]):                    # fp32 sums in another order
        torch.testing.assert_close(x, y, rtol=2e-5, atol=2e-5)
    v = torch.randn((d,), generator=torch.Generator(device=DEV).manual_seed(3), device=DEV)
    alphas = [-2.0, -1.0, -0.5, 0.0, 0.5, 1.0, 2.0]
    ids, p, logp, ent = LL.ll_steer_sweep(w.hidden.reshape(N, d), w.gamma, w.W_U, w.cfg.eps, v / v.norm(), alphas, w.target_ids)
    assert (ids[3] != a[0][:, 0]).float().mean() < 1e-3
    for x, y in ((p[3], a[1][:, 0]), (logp[3], a[2]), (ent[3], a[3])):
        torch.testing.assert_close(x, y, rtol=2e-5, atol=2e-5)
