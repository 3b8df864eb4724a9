"""The allocation-free step's limit of 4096 workgroups, decided on the host
before anything touches a device: the last accepted and the first refused grids
by the count of the header.  Without a GPU an accepted call ends at the device
lookup (SURF_EDEVICE), so that no pointer is ever used; with one the calls are
not made."""
import ctypes

import pytest
import torch

from paper_2605_27534_amd import surf as S

ENOMEM, EDEVICE = -2, -3

pytestmark = pytest.mark.skipif(torch.cuda.is_available(),
                                reason="an accepted call would launch on made-up pointers")


def call(n, prec):
    prob = dict(dim=len(n), n=n, h=1.0 / 64, bc=((0, 0),) * len(n))
    g, p, _ = S.make_structs(prob, 1e-5, prec)
    q = [ctypes.c_void_p(4096 * (k + 1)) for k in range(5)]
    return S.lib().surf_step_static(ctypes.byref(g), ctypes.byref(p), 1e-5, q[0], None, q[1], q[2],
                                    q[3], q[4], None, None, None)


@pytest.mark.parametrize("prec,planes", [(S.SURF_F32, 16), (S.SURF_F64, 8)])
def test_3d(prec, planes):
    n = (58 * 16, 14 * 16, planes * 16)
    assert call(n, prec) == EDEVICE
    for d in range(3):
        assert call(tuple(v + (e == d) for e, v in enumerate(n)), prec) == ENOMEM
    # long chunks of planes launch fewer workgroups; the limit does not follow
    assert call((384, 384, 384), prec) == ENOMEM


@pytest.mark.parametrize("prec", [S.SURF_F32, S.SURF_F64])
def test_2d(prec):
    for n in ((58 * 64, 32 * 64), (58 * 4096, 4), (58, 32 * 4096)):
        assert call(n, prec) == EDEVICE, n
        for m in ((n[0] + 1, n[1]), (n[0], n[1] + 1)):
            if m != (58 * 4096, 5):  # still one group of rows
                assert call(m, prec) == ENOMEM, m
