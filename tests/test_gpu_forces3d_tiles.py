"""The 3D interfacial forces at the edges of their work units (8^3 tiles, 64
cells along x per listing workgroup, tiles with and without the box's sides in
reach, the smallest boxes): a ball and single interfacial cells scattered over
the box, its corners and sides among them, so that faces with one and with two
interfacial cells, columns that do not close and lone cells all appear, against
the FP64 oracle.  Tolerances as in test_gpu_capillary3d: 1e-12 and 2e-5."""
import numpy as np
import pytest

from paper_2605_27534_amd import synth
from tests.test_gpu_capillary3d import F32, F64, compare

pytestmark = pytest.mark.gpu

W, P, OP = 0, 1, 2

CASES = [
    # n, sides
    ((4, 4, 4), ((W, OP), (P, P), (OP, W))),
    ((5, 8, 9), ((P, P), (W, W), (P, P))),
    ((18, 18, 18), ((P, P), (P, P), (P, P))),
    ((26, 17, 18), ((OP, W), (W, W), (W, OP))),
    ((64, 8, 10), ((P, P), (OP, OP), (W, W))),
    ((67, 19, 18), ((W, W), (P, P), (OP, OP))),
    ((130, 7, 4), ((P, P), (P, P), (W, OP))),
]


@pytest.mark.parametrize("prec", [F64, F32])
@pytest.mark.parametrize("n,bc", CASES)
def test_tiles(n, bc, prec):
    h = 1.0 / n[0]
    rng = np.random.default_rng(sum(n))
    z, y, x = np.meshgrid(*[(np.arange(m) + 0.5) * h for m in n[::-1]], indexing="ij")
    mid = [0.5 * h * m for m in n]
    chi = 0.4 * h * min(n) - np.sqrt((x - mid[0]) ** 2 + (y - mid[1]) ** 2 + (z - mid[2]) ** 2)
    vof = np.clip(0.5 + chi / h, 0.0, 1.0)
    some = rng.random(vof.shape) < 30.0 / vof.size
    for corner in ((0, 0, 0), (-1, -1, -1), (n[2] // 2, -1, 0), (-1, 0, n[0] // 2)):
        some[corner] = True
    vof[some] = rng.uniform(0.01, 0.99, int(some.sum()))
    chi = chi + 0.05 * h * rng.standard_normal(vof.shape)
    sig = 1.0 + 0.2 * synth.smooth_modes(n, h, 5, dim=3)
    compare(dict(dim=3, n=n, h=h, bc=bc), vof, chi, sig, prec)
