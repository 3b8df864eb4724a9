"""The 3D ACDI step as marching waves at the edges of its work units (strips of
60 and 62 columns, blocks of 4 and 2 rows, chunks of 1 to 8 planes), every kind
of side, with and without flow, against the FP64 oracle: phi and the phase of
the level set after two steps.  Tolerances as in test_gpu_acdi: 1e-12 and 2e-5."""
import pytest

from paper_2605_27534_amd import synth
from tests.harness import rel_max
from tests.test_gpu_acdi import F32, F64, TOL, phase_of, run_both

pytestmark = pytest.mark.gpu

W, P, OP = 0, 1, 2

CASES = [
    # n, sides, flow
    ((4, 4, 4), ((W, OP), (P, P), (OP, W)), True),
    ((5, 7, 9), ((P, P), (OP, OP), (P, P)), True),
    ((60, 4, 17), ((OP, OP), (W, OP), (W, W)), True),
    ((61, 9, 8), ((P, P), (P, P), (OP, OP)), True),
    ((62, 18, 16), ((W, W), (W, W), (P, P)), False),
    ((63, 17, 5), ((OP, W), (P, P), (W, OP)), True),
    ((125, 33, 26), ((P, P), (OP, W), (P, P)), True),
    ((124, 129, 66), ((W, OP), (W, W), (OP, OP)), True),
]


@pytest.mark.parametrize("prec", [F64, F32])
@pytest.mark.parametrize("n,bc,flow", CASES)
def test_edges(n, bc, flow, prec):
    h = 1.0 / max(n)
    mid = [0.47 * h * m for m in n]
    u = synth.random_faces(n, 3, 7, 0.4) if flow else None
    prob = dict(dim=3, n=n, h=h, bc=bc, eos=0, acdi_zeta=0.5)
    o, g = run_both(prob, synth.vof_ball(n, h, mid, 0.35 * h * min(n), 3), 2, 0.05 * h, prec, u=u)
    eps = 1.5 * h
    assert rel_max(g[1], o[1]) <= TOL[prec]
    assert rel_max(phase_of(g[0], eps), phase_of(o[0], eps)) <= TOL[prec]
