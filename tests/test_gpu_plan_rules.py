"""The built-in rules of hub_get_plan at sectors on either side of their lines:
each plan below is the one that was measured faster there."""
import pytest

import paper_2005_13498_amd as hub
from synth import ring

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
C128, C64 = hub.HUB_C128, hub.HUB_C64


def _plan(lat, nu, nd, prec, nvec, propagate=True, setup=None):
    B = hub.Basis(lat, 8.0, nu, nd, device=0)
    try:
        if setup:
            setup(B.handle)
        return hub.hub_get_plan(B.handle, prec, nvec, propagate)
    finally:
        B.close()


@pytest.mark.parametrize("n,nu,nd,prec,kernels", [
    (14, 7, 2, C64, 0), (14, 5, 2, C128, 0), (15, 5, 2, C64, 0),       # tall: few columns
    (16, 1, 5, C128, 0),                                               # 16 rows
    (13, 6, 3, C64, 1), (12, 4, 5, C64, 1), (13, 2, 6, C64, 1), (11, 5, 5, C128, 1),
    (12, 6, 6, C128, 1), (14, 7, 2, C128, 1)])                         # above 4 MiB: whatever the shape
def test_two_pass_iterations(n, nu, nd, prec, kernels):
    assert _plan(ring(n), nu, nd, prec, 1) == [(1, kernels)]
