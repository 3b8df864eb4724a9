"""The ACDI step with a regularization of s below FP32's smallest normal number,
on a flat interface whose phi reaches 0 and 1 exactly: phi stays finite and
meets the FP64 oracle.  Tolerance as in test_gpu_acdi: 2e-5."""
import numpy as np
import pytest

from oracle import acdi as A
from paper_2605_27534_amd import surf as S
from paper_2605_27534_amd import synth
from tests.harness import rel_max, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ve", [1e-39, 1e-300])
@pytest.mark.parametrize("n,flow", [((320, 8), True), ((320, 8, 6), True), ((320, 8, 6), False)])
def test_denormal_regularization(n, flow, ve):
    dim, h, zeta = len(n), 1.0 / 64, 0.5
    prob = dict(dim=dim, n=n, h=h, bc=((2, 2), (1, 1), (1, 1))[:dim], interface=1, acdi_zeta=zeta,
                acdi_vareps=ve, chi_max_eps=120.0)
    x = (np.arange(n[0]) + 0.5) * h
    chi = np.broadcast_to(x - 0.5 * n[0] * h + 0.2 * h, n[::-1]).copy()  # to 107 eps either way
    if dim == 2:
        chi = chi[None]
    u = synth.u_uniform(n, dim, (0.3, 0.0, 0.0)[:dim]) if flow else None
    dt = 0.05 * h
    phi = A.phi_of_chi(prob, chi)
    s = S.Surf(prob, dt, S.SURF_F32)
    s.set_levelset(s.tensor(chi))
    start = to_np(s.phase())
    assert start.min() == 0.0 and start.max() == 1.0
    F, P = s.init_state(None, 1.0, 0.3)
    F2, P2 = s.empty(), s.empty()
    ud = None if u is None else [s.tensor(v) for v in u]
    for _ in range(2):
        phi = A.acdi_step(prob, phi, u, dt, zeta, ve)
        s.step(F, P, F2, P2, u=ud)
        F, P, F2, P2 = F2, P2, F, P
    got = to_np(s.phase())
    assert np.isfinite(got).all() and np.isfinite(to_np(s.levelset())).all()
    assert rel_max(got, phi) <= 2e-5
