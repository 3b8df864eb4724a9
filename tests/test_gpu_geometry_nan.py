"""A NaN among the fractions given to a warm start, two cells or more from the
interface: the level set is that of the clean fractions (the cell is taken for
the side its level set lies on), on the whole box, in the moving geometry of the
2D steps, and in that of the 3D steps in a tile without a cut cell.  Tolerances as in test_gpu_geometry_build: 1e-12 and 2e-5 of the
clamp."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2605_27534_amd import synth
from tests.harness import rel_max

pytestmark = pytest.mark.gpu

TOL = {1: 1e-12, 0: 2e-5}
W, P, OP = 0, 1, 2

CASES = [
    # n, sides, warm sweeps, cells (x, y, z) that hold a NaN: inside, outside; a step
    ((64, 48), ((W, W), (OP, OP)), 8, ((32, 24), (60, 3)), False),
    ((64, 48), ((W, W), (OP, OP)), 8, ((32, 24), (60, 3)), True),
    ((64, 48), ((P, P), (W, OP)), 16, ((36, 22), (0, 47)), False),
    ((64, 48), ((P, P), (W, OP)), 16, ((36, 22), (0, 47)), True),
    ((30, 28), ((W, W), (P, P)), 3, ((15, 14), (29, 0)), True),
    ((36, 34, 40), ((P, P), (OP, W), (P, P)), 4, ((18, 17, 20), (35, 0, 39)), False),
    ((30, 28, 26), ((W, W), (P, P), (OP, OP)), 5, ((15, 13, 14), (1, 27, 2)), True),
    # the first cell of the tile of 16^3 in the middle of a ball, and another
    ((80, 80, 80), ((W, W), (P, P), (OP, OP)), 4, ((32, 32, 32),), True),
    ((80, 80, 80), ((P, P), (W, W), (OP, OP)), 4, ((41, 36, 46), (5, 5, 5)), True),
]


@pytest.mark.parametrize("prec", [1, 0])
@pytest.mark.parametrize("n,bc,warm,cells,step", CASES)
def test_level_set(n, bc, warm, cells, step, prec):
    from paper_2605_27534_amd import surf as S
    dim, h = len(n), 1.0 / max(n)
    prob = dict(dim=dim, n=n, h=h, bc=bc, hj_iters_step=warm)
    ball = lambda s: synth.vof_ball(n, h, [0.5 * h * m + s * h for m in n] + [0] * (3 - dim),
                                    0.29 * min(n) * h, dim)
    vof, nxt = ball(0.0), ball(0.3)
    chi = O.geometry(prob, vof, 72 if dim == 2 else 108)
    chi = O.geometry(prob, nxt, warm, chi=chi)
    bad = nxt.copy()
    for c in cells:
        at = tuple(([0] * (3 - dim) + list(c[::-1]))[-bad.ndim:])
        assert nxt[at] in (0.0, 1.0)
        bad[at] = np.nan
    s = S.Surf(prob, 1e-4 * h, prec)
    s.set_geometry(s.tensor(vof), full=True)
    if step:
        F, Q = s.init_state(None, 1.0, 0.0)
        s.step(F, Q, s.empty(), s.empty(), vof_next=s.tensor(bad))
    else:
        s.set_geometry(s.tensor(bad), full=False)
    assert rel_max(s.levelset().double().cpu().numpy(), chi) <= TOL[prec]
