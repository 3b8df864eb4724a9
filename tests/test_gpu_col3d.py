"""The 3D plane-marching transport at the edges of its work units (58-column
strips, 14-row blocks, plane chunks of several lengths, the smallest box),
random flow, every kind of side, against the FP64 oracle.  Tolerances as in
test_gpu_parity: 1e-12 and 2e-5."""
import pytest

from oracle import oracle as O
from paper_2605_27534_amd import synth
from tests.harness import compare_totals, rel_max, run_gpu, run_oracle

pytestmark = pytest.mark.gpu

TOL = {1: 1e-12, 0: 2e-5}
W, P, OP = 0, 1, 2

CASES = [
    # n, sides, flow, bulk, kinetics, equation of state
    ((4, 4, 4), ((W, OP), (P, P), (OP, W)), True, 1, 0, 0),
    ((4, 5, 9), ((P, P), (OP, OP), (P, P)), True, 1, 1, 2),
    ((58, 14, 8), ((W, W), (W, W), (W, W)), True, 1, 0, 2),
    ((59, 15, 9), ((P, P), (P, P), (P, P)), True, 1, 0, 2),
    ((61, 13, 25), ((OP, OP), (W, OP), (P, P)), True, 0, 0, 2),
    ((62, 29, 17), ((OP, W), (OP, W), (W, OP)), True, 1, 1, 0),
    ((119, 16, 33), ((P, P), (OP, OP), (OP, OP)), True, 1, 0, 2),
    ((125, 30, 12), ((W, OP), (P, P), (W, W)), False, 1, 0, 2),
    ((60, 43, 5), ((OP, OP), (W, W), (P, P)), False, 0, 0, 0),
]


@pytest.mark.parametrize("prec", [1, 0])
@pytest.mark.parametrize("n,bc,flow,bulk,kin,eos", CASES)
def test_edges(n, bc, flow, bulk, kin, eos, prec):
    h = 1.0 / max(n)
    prob = dict(dim=3, n=n, h=h, bc=bc, kinetics=kin, eos=eos, eos_E=0.3, bulk_enabled=bulk)
    ext = [h * v for v in n]
    chi = synth.distance_ball(n, h, (0.45 * ext[0], 0.55 * ext[1], 0.5 * ext[2]),
                              0.35 * min(ext), 18.0 * h)
    u = synth.random_faces(n, 3, 7, 0.5) if flow else None
    c0 = synth.uniform_field(n, 3, 0.5, 1.5)
    dt = min(0.05 * h * h / 1e-2, 0.2 * h)
    o = run_oracle(prob, None, 3, dt, u=u, chi=chi, c0=c0, gamma0=0.3)
    g = run_gpu(prob, None, 3, dt, prec, u=u, chi=chi, c0=c0, gamma0=0.3)
    tol = TOL[prec]
    for i, name in ((1, "F"), (2, "psi"), (3, "sigma")):
        if name == "F" and not bulk:
            continue
        assert rel_max(g[i], o[i]) <= tol, name
    compare_totals(g[4][-1], o[4][-1], tol, o[1] if bulk else None, o[2])
