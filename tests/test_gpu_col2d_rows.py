"""The 2D column-streaming transport at the sizes where its rows per wave (2, 4
or 8) change, in whole chunks and one row more, with every kind of side,
against the FP64 oracle; and the allocation-free step's limit of 4096
workgroups, which does not depend on the chunks a launch takes.  Tolerances as
in test_gpu_parity: 1e-12 and 2e-5."""
import pytest

from paper_2605_27534_amd import surf as S
from paper_2605_27534_amd import synth
from tests.harness import compare_totals, rel_max, run_gpu, run_oracle

pytestmark = pytest.mark.gpu

TOL = {1: 1e-12, 0: 2e-5}
W, P, OP = 0, 1, 2

CASES = [
    # n, sides: 2 rows a wave, the last such box and the first of 4, the last of 4
    # (FP32) and the first of 8, 4 in FP64
    ((5, 4), ((W, OP), (P, P))),
    ((61, 33), ((P, P), (OP, W))),
    ((58, 4096), ((OP, OP), (W, W))),
    ((58, 4097), ((OP, OP), (P, P))),
    ((116, 8192), ((P, P), (W, OP))),
    ((117, 8193), ((W, W), (OP, OP))),
]


@pytest.mark.parametrize("prec", [1, 0])
@pytest.mark.parametrize("n,bc", CASES)
def test_rows(n, bc, prec):
    h = 1.0 / max(n)
    prob = dict(dim=2, n=n, h=h, bc=bc, eos=1, eos_E=0.3)
    mid = [0.45 * h * m for m in n]
    chi = synth.distance_ball(n, h, mid + [0], 0.35 * h * min(n), 18.0 * h)
    u = synth.random_faces(n, 2, 7, 0.4)
    c0 = synth.uniform_field(n, 3, 0.5, 1.5)
    args = (prob, None, 2, min(0.05 * h * h / 1e-2, 0.2 * h))
    kw = dict(u=u, chi=chi, c0=c0, gamma0=0.3)
    o, g = run_oracle(*args, **kw), run_gpu(*args, prec, **kw)
    for i in (1, 2, 3):
        assert rel_max(g[i], o[i]) <= TOL[prec], i
    compare_totals(g[4][-1], o[4][-1], TOL[prec], o[1], o[2])


def test_allocation_free_step_limit():
    import torch
    t = [torch.zeros(16, device="cuda") for _ in range(5)]
    prob = dict(dim=3, n=(384, 384, 384), h=1.0 / 384, bc=((W, W),) * 3)
    # 7 x 28 x 24 workgroups by the documented count
    assert S.step_static(prob, 1e-5, S.SURF_F32, t[0], t[1], t[2], t[3], t[4]) == -2
