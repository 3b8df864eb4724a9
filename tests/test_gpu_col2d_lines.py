"""The 2D column-streaming transport at the sizes where 4 and 8 rows per wave
change places, the last box on each side of a line, with every kind of side,
against the FP64 oracle.  Tolerances as in test_gpu_parity: 1e-12 and 2e-5."""
import pytest

from paper_2605_27534_amd import synth
from tests.harness import compare_totals, rel_max, run_gpu, run_oracle

pytestmark = pytest.mark.gpu

TOL = {1: 1e-12, 0: 2e-5}
W, P, OP = 0, 1, 2

CASES = [
    # n, sides: 3072 waves of 4 rows and one more; 2048 waves of 8 rows and one
    # more; 5120 waves of 4 rows and one more
    ((58, 12288), ((W, OP), (P, P))),
    ((116, 6145), ((P, P), (OP, W))),
    ((116, 8192), ((OP, W), (W, W))),
    ((58, 16385), ((OP, OP), (W, OP))),
    ((290, 4096), ((P, P), (P, P))),
    ((58, 20481), ((W, W), (OP, OP))),
]


@pytest.mark.parametrize("prec", [1, 0])
@pytest.mark.parametrize("n,bc", CASES)
def test_lines(n, bc, prec):
    h = 1.0 / n[0]
    prob = dict(dim=2, n=n, h=h, bc=bc, eos=1, eos_E=0.3)
    mid = [0.45 * h * m for m in n]
    chi = synth.distance_ball(n, h, mid + [0], 0.35 * h * n[0], 18.0 * h)
    u = synth.random_faces(n, 2, 7, 0.4)
    c0 = synth.uniform_field(n, 3, 0.5, 1.5)
    args = (prob, None, 2, min(0.05 * h * h / 1e-2, 0.2 * h))
    kw = dict(u=u, chi=chi, c0=c0, gamma0=0.3)
    o, g = run_oracle(*args, **kw), run_gpu(*args, prec, **kw)
    for i in (1, 2, 3):
        assert rel_max(g[i], o[i]) <= TOL[prec], i
    compare_totals(g[4][-1], o[4][-1], TOL[prec], o[1], o[2])
