"""The 3D whole-box redistancing where blocks of 60 x 4 x 4 cells that hold one
value are filled instead of swept, on periodic axes whose last block has one,
two or three cells: a small ball whose front crosses the wrapped sides while the
blocks beyond still hold one value.  Against the FP64 oracle, with tolerances as
in test_gpu_geometry_build: 1e-12 and 2e-5 of the clamp.  Filling also where a
wrapped halo of two cells reaches past a last block of one cell would be off by
3e-5 to 1.3e-4 of the clamp after 8 sweeps and by 3e-11 to 3e-10 after 108."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2605_27534_amd import synth
from tests.harness import rel_max

pytestmark = pytest.mark.gpu

TOL = {1: 1e-12, 0: 2e-5}

# n, centre in cells: near the last whole block of each axis, near the first
CASES = [
    ((181, 57, 65), (173.2, 49.1, 58.4)),
    ((181, 57, 65), (9.1, 8.3, 7.9)),
    ((182, 58, 66), (172.6, 48.2, 57.7)),
    ((183, 59, 67), (173.9, 50.4, 59.3)),
    ((182, 58, 67), (8.8, 9.2, 9.7)),
]


def box(n, centre):
    h = 1.0 / max(n)
    prob = dict(dim=3, n=n, h=h, bc=((1, 1),) * 3)
    return prob, synth.vof_ball(n, h, [h * c for c in centre], 4.3 * h, 3)


@pytest.mark.parametrize("prec", [1, 0])
@pytest.mark.parametrize("sweeps", [8, 108])
@pytest.mark.parametrize("n,centre", CASES)
def test_front_crosses_the_wrap(n, centre, sweeps, prec):
    from paper_2605_27534_amd import surf as S
    prob, vof = box(n, centre)
    chi_o = O.geometry(prob, vof, sweeps)
    s = S.Surf(dict(prob, hj_iters_init=sweeps), 1e-4, prec)
    s.set_geometry(s.tensor(vof), full=True)
    assert rel_max(s.levelset().double().cpu().numpy(), chi_o) <= TOL[prec]
