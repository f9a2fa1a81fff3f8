"""Launch forms of the steering kernels at the sizes where one takes over from the other: the direction in one workgroup,
from one slice of the rows, from several; the injection with a wavefront or a workgroup per row.  On a real MI355X."""
import numpy as np
import pytest
import torch

import oracle.lens_oracle as O
from paper_2604_06483_amd import binding as LL
from paper_2604_06483_amd import workloads as WL
from tests.conftest import say

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def rows(n, d, seed, offset=0.0):
    g = torch.Generator(device=DEV).manual_seed(seed)
    return (3 * torch.randn((n, d), generator=g, device=DEV) + offset).to(torch.bfloat16)


@pytest.mark.parametrize("use_ws", [False, True])
@pytest.mark.parametrize("nb,nt,d", [(1, 16, 8192), (16, 2, 8), (17, 1, 72), (16, 16, 8200), (128, 3, 1032), (3, 129, 1032),
                                     (2000, 7689, 200), (300, 40, 1000), (130, 700, 1096)])
def test_direction(nb, nt, d, use_ws):
    say(f"steer direction nb={nb} nt={nt} d={d} ws={use_ws}")
    base, target = rows(nb, d, nb), rows(nt, d, nt + 1, 0.5)
    ws = torch.empty(LL.ll_steer_workspace_bytes(d), dtype=torch.uint8, device=DEV) if use_ws else None
    for normalize in (False, True):
        v = LL.ll_steer_vector(base, target, normalize, workspace=ws).cpu().numpy().astype(np.float64)
        want = O.steer_vector(WL.bf16_bits(base), WL.bf16_bits(target), normalize)
        # a sum of n terms in fp32, in any order: n - 1 roundings of at most 2^-24 of the sum of magnitudes, and one each for
        # the quotient and the difference
        mag = [float(x.float().abs().double().mean(0).max()) for x in (base, target)]
        err = 2.0 ** -24 * ((nb + 2) * mag[0] + (nt + 2) * mag[1])
        if normalize:   # the length is off by no more than the root of the summed squares of these, and rounds d + 4 times
            length = float(np.linalg.norm(O.steer_vector(WL.bf16_bits(base), WL.bf16_bits(target), False)))
            err = err / length + np.abs(want).max() * (err * d ** 0.5 / length + (d + 4) * 2.0 ** -24)
        assert np.abs(v - want).max() <= err


@pytest.mark.parametrize("d", [1024, 1032, 2048, 2056, 4096, 4104, 8192, 8200])
def test_injection_has_the_same_bits_in_both_forms(d):
    say(f"steer inject forms d={d}")
    N = 1536   # the most rows that get a workgroup each
    h = rows(N + 1, d, d)
    h[3] = 0
    gamma = (1 + rows(1, d, 5)[0].float() / 30).to(torch.bfloat16)
    v = torch.randn((d,), generator=torch.Generator(device=DEV).manual_seed(7), device=DEV)
    both = LL.ll_steer_inject(h, gamma, 1e-5, v, 2.5)
    few = LL.ll_steer_inject(h[:N], gamma, 1e-5, v, 2.5)
    assert torch.equal(few, both[:N])
    assert torch.equal(LL.ll_steer_inject(h[N:], gamma, 1e-5, v, 2.5), both[N:])
    LL.ll_steer_inject(h[:N], gamma, 1e-5, v, 2.5, out=h[:N])
    assert torch.equal(h[:N], few)
