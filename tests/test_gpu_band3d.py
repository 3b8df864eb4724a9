"""The 3D moving geometry (tiles of 16^3 cells, sweeps over the live tiles) at
the edges of its work units: boxes smaller than a tile, of whole tiles, one
cell or row or plane more and fewer, every kind of side, few and many sweeps.
A sphere moves across tile faces and sides for three steps, the first on tiles
that are all live and the others on the band; the level set against the FP64
oracle's global sweeps.  Tolerances as in test_gpu_parity: 1e-12 and 2e-5."""
import pytest

from paper_2605_27534_amd import synth
from tests.harness import rel_max, run_gpu, run_oracle

pytestmark = pytest.mark.gpu

TOL = {1: 1e-12, 0: 2e-5}
W, P, OP = 0, 1, 2

CASES = [
    # n, sides, sweeps, centre and radius in cells
    ((4, 4, 4), ((W, W), (P, P), (OP, OP)), 2, (1.8, 2.1, 2.0), 1.2),
    ((16, 16, 16), ((P, P), (P, P), (P, P)), 4, (0.5, 15.2, 8.0), 4.4),
    ((17, 15, 33), ((OP, W), (W, OP), (P, P)), 16, (15.4, 7.3, 16.2), 3.7),
    ((15, 33, 17), ((P, P), (W, W), (OP, W)), 6, (14.6, 16.1, 15.7), 5.1),
    ((49, 20, 31), ((P, P), (OP, OP), (W, W)), 16, (47.8, 9.6, 16.0), 6.2),
    ((100, 17, 48), ((W, W), (P, P), (P, P)), 2, (48.3, 0.4, 47.0), 5.0),
]


@pytest.mark.parametrize("prec", [1, 0])
@pytest.mark.parametrize("n,bc,sweeps,centre,radius", CASES)
def test_levelset(n, bc, sweeps, centre, radius, prec):
    h = 1.0 / max(n)
    prob = dict(dim=3, n=n, h=h, bc=bc, eos=0, hj_iters_step=sweeps)
    at = lambda k: synth.vof_ball(n, h, [h * (c + 0.3 * k) for c in centre], radius * h, 3)
    args = (prob, at(0), 3, 0.05 * h * h / 1e-2)
    kw = dict(vof_seq=lambda k: at(k + 1), hj_step=sweeps)
    o, g = run_oracle(*args, **kw), run_gpu(*args, prec, **kw)
    assert rel_max(g[0], o[0]) <= TOL[prec]
    assert g[5].status() & 8 == 0
