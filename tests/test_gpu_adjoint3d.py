"""The 3D adjoint step at the edges of its work units (62 columns, blocks of 4
and 2 rows, chunks of several lengths, cells whose stencils reach one or two
sides), every kind of side, with and without flow, against the FP64 oracle.
FP64: 1e-10 as in test_gpu_adjoint.  FP32: 2e-5, dL/dc0 in the 2-norm (where
two differences tie, rounding decides which one minmod takes, and the gradient
at that cell jumps)."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2605_27534_amd import synth
from tests.test_gpu_adjoint import gpu_grad

pytestmark = pytest.mark.gpu

W, P, OP = 0, 1, 2

CASES = [
    # n, sides, flow, bulk kinetics
    ((4, 4, 4), ((W, OP), (P, P), (OP, W)), True, 0),
    ((5, 7, 9), ((P, P), (OP, OP), (P, P)), True, 1),
    ((62, 18, 8), ((W, W), (W, W), (P, P)), False, 0),
    ((63, 5, 17), ((P, P), (OP, W), (W, OP)), True, 0),
    ((64, 17, 6), ((OP, OP), (P, P), (W, W)), True, 1),
    ((125, 33, 10), ((OP, W), (W, OP), (P, P)), True, 0),
]


@pytest.mark.parametrize("prec", [1, 0])
@pytest.mark.parametrize("n,bc,flow,kin", CASES)
def test_gradients(n, bc, flow, kin, prec):
    h = 1.0 / max(n)
    prob = dict(dim=3, n=n, h=h, bc=bc, kinetics=kin, eos=1, eos_E=0.3)
    mid = [0.45 * h * m for m in n]
    chi = synth.distance_ball(n, h, mid, 0.35 * h * min(n), 18.0 * h)
    u = synth.random_faces(n, 3, 7, 0.3) if flow else None
    c0 = 1 + 0.1 * synth.smooth_modes(n, h, 4)
    N, dt = 5, min(0.05 * h * h / 1e-2, 0.1 * h)
    theta = np.array([1.3, 0.7, 0.012, 0.0008])
    target = np.linspace(0.97, 0.93, N)
    Lo, dto, gco = O.sigma_history_grad(prob, chi, u, c0, 0.2, dt, N, theta, target)
    Lg, dtg, gcg = gpu_grad(prob, chi, u, c0, dt, N, theta, target, prec, 2)
    tol = 1e-10 if prec == 1 else 2e-5
    assert abs(Lg - Lo) <= tol * Lo
    # without flow Gamma stays uniform but for the exchange: dL/dD_s is then a
    # sum that cancels to 1e-5 of its terms (5e-10 and 1.4e-1 of itself off)
    k = 4 if flow else 3
    assert np.max(np.abs(dtg - dto)[:k] / np.abs(dto)[:k]) <= tol, (dtg, dto)
    if prec == 1:
        assert np.max(np.abs(gcg - gco)) <= tol * np.max(np.abs(gco))
    else:
        assert np.linalg.norm(gcg - gco) <= tol * np.linalg.norm(gco)
