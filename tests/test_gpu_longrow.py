"""Sectors whose down rows are too long for LDS while their up columns fit
(few up electrons, many down ones): propagations, Krylov steps and their apply
timing, against the one-pass kernels and against the sector with the spins
exchanged, whose tile is the transpose and whose rows fit.  Vectors of 1 to 4
MiB, above 4 MiB and above 32 MiB, both precisions, singles and groups.  Four
steps within the tolerance of 1e-11 each on either side leave 8e-11 and the
rounding of some forty products in complex128; complex64 rounds 1.2e-7 in each
of them."""
import numpy as np
import pytest
import torch

import paper_2005_13498_amd as hub
from synth import PulseParams, chain, ring

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
BAR = {torch.complex128: 1e-10, torch.complex64: 1e-5}


def _state(nvec, du, dd, dtype):
    g = torch.Generator(device=DEV).manual_seed(11)
    x = torch.randn(nvec, du, dd, dtype=torch.complex128, device=DEV, generator=g)
    return (x / torch.linalg.vector_norm(x, dim=(1, 2), keepdim=True)).to(dtype).contiguous()


def _opts(dtype):
    return hub.make_opts(tol=1e-11 if dtype == torch.complex128 else 1e-7, m_max=30)


@pytest.mark.parametrize("lat,nu,nd,dtype,nvec", [
    (chain(15), 1, 6, torch.complex128, 1), (ring(16), 1, 8, torch.complex64, 1), (chain(16), 15, 7, torch.complex64, 1),
    (chain(16), 1, 8, torch.complex128, 2), (ring(15), 2, 6, torch.complex128, 1), (ring(16), 2, 8, torch.complex64, 3),
    (chain(16), 3, 8, torch.complex128, 1)])
def test_long_rows_propagate(lat, nu, nd, dtype, nvec):
    B, T = hub.Basis(lat, 8.0, nu, nd, device=0), hub.Basis(lat, 8.0, nd, nu, device=0)
    try:
        _, du, dd = hub.hub_basis_info(B.handle)
        x = _state(nvec, du, dd, dtype)
        pulses = [PulseParams(0, 0.3 * (k + 1), 8.0, 0.02, 0.05) for k in range(nvec)]

        def run(H, v):
            _, obs, _ = hub.hub_propagate(H.handle, pulses, 0.0, 0.01, 4, _opts(dtype), v)
            return obs

        v = x.clone()
        obs = run(B, v)
        hub.hub_set_apply_path(B.handle, 0)
        one = x.clone()
        obs_one = run(B, one)
        hub.hub_set_apply_path(B.handle, 1)
        two = x.clone()
        run(B, two)
        tr = x.transpose(1, 2).contiguous()
        obs_tr = run(T, tr)
        bar = BAR[dtype]
        for w in (one, two, tr.transpose(1, 2)):
            assert float(torch.linalg.vector_norm(v - w)) <= bar * np.sqrt(nvec)
        scale = hub.hub_basis_classes(B.handle)[2]
        assert np.max(np.abs(obs - obs_one)) <= bar * scale
        assert np.max(np.abs(obs - obs_tr)) <= bar * scale
    finally:
        B.close()
        T.close()
        torch.cuda.empty_cache()


@pytest.mark.parametrize("lat,nu,nd,dtype", [(chain(15), 1, 6, torch.complex128), (ring(16), 2, 8, torch.complex64)])
def test_long_rows_step_and_timing(lat, nu, nd, dtype):
    """A single Krylov step, and the apply timing of its iterations and of a
    plain product (one kernel each), on the kernels the plan reports."""
    B = hub.Basis(lat, 8.0, nu, nd, device=0)
    try:
        prec = hub.HUB_C128 if dtype == torch.complex128 else hub.HUB_C64
        assert hub.hub_get_plan(B.handle, prec, 1, True) == [(1, 0)]
        _, du, dd = hub.hub_basis_info(B.handle)
        x = _state(1, du, dd, dtype)
        v, w = x.clone(), x.clone()
        hub.hub_profile_enable(B.handle, 1)
        hub.hub_krylov_expm_step(B.handle, [0.4], 0.02, _opts(dtype), v)
        hub.hub_apply_H(B.handle, [0.4], x, torch.empty_like(x))
        launches, ms, _ = hub.hub_profile_read(B.handle)
        assert launches >= 2 and ms > 0.0
        hub.hub_profile_enable(B.handle, 0)
        hub.hub_set_apply_path(B.handle, 0)
        hub.hub_krylov_expm_step(B.handle, [0.4], 0.02, _opts(dtype), w)
        assert float(torch.linalg.vector_norm(v - w)) <= BAR[dtype]
    finally:
        B.close()
        torch.cuda.empty_cache()
