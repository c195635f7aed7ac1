"""Plain products of vectors larger than 32 MiB (hub_apply_H): the column pass
that gathers its up hops, after a row pass in LDS or, where a row is too long,
from global memory.  Column counts that are no multiple of a workgroup's or a
lane's columns, row counts that are no multiple of its rows, both precisions,
on-site energies, vectors at odd offsets, an infinite component.  The terms
are added in the order of the one-pass kernels: bit-identical to them."""
import pytest
import torch

import paper_2005_13498_amd as hub
from synth import chain, ring

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _onsite(lat):
    return lat.with_onsite([0.1 * i - 0.4 for i in range(lat.n_sites)])


@pytest.mark.parametrize("lat,nu,nd,dtype", [
    (ring(13), 6, 6, torch.complex128), (chain(14), 6, 7, torch.complex64), (_onsite(ring(14)), 5, 6, torch.complex128),
    (chain(15), 4, 7, torch.complex128), (ring(15), 4, 7, torch.complex64), (_onsite(ring(16)), 3, 8, torch.complex128),
    (ring(16), 4, 8, torch.complex64), (ring(15), 7, 5, torch.complex64)])
def test_gather_matches_one_pass(lat, nu, nd, dtype):
    B = hub.Basis(lat, 6.0, nu, nd, device=0)
    prec = hub.HUB_C128 if dtype == torch.complex128 else hub.HUB_C64
    assert B.dim * (16 if prec == hub.HUB_C128 else 8) > 32 << 20
    assert hub.hub_get_plan(B.handle, prec, 1, False) == [(1, 1)]
    gen = torch.Generator(device=DEV).manual_seed(5)
    x = torch.randn(2, B.dim, dtype=dtype, device=DEV, generator=gen)
    x[1, B.dim // 3] = float("inf")
    y, z = torch.full_like(x, float("nan")), torch.full_like(x, float("nan"))
    A = [0.43, -0.2]
    for k in range(2):
        hub.hub_apply_H(B.handle, A[k], x[k], y[k])
    hub.hub_set_apply_path(B.handle, 0)
    for k in range(2):
        hub.hub_apply_H(B.handle, A[k], x[k], z[k])
    assert torch.equal(y[0], z[0])
    # where a hop is missing the one-pass kernels add 0 times a zero, so an
    # infinite component reaches the same places
    assert torch.equal(torch.isfinite(torch.view_as_real(y[1])), torch.isfinite(torch.view_as_real(z[1])))
    fin = torch.isfinite(torch.view_as_real(z[1]))
    assert torch.equal(torch.view_as_real(y[1])[fin], torch.view_as_real(z[1])[fin])
    B.close()
