"""Lanes created while the null stream is busy: their workspaces are cleared in
their own streams' order, so a propagation on another stream gives the states
and observables of a quiet run bit for bit."""
import numpy as np
import pytest
import torch

import paper_2005_13498_amd as hub
from synth import PulseParams, ring

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("n,nvec,dtype,steps", [(10, 12, torch.complex128, 400), (11, 3, torch.complex64, 400)])
def test_new_lanes_beside_a_busy_null_stream(n, nvec, dtype, steps):
    pulses = [PulseParams(0, 0.1 * (k + 1), 8.0, 0.5, 0.15) for k in range(nvec)]
    m = torch.randn(8192, 8192, device=DEV)
    out = torch.empty_like(m)
    torch.mm(m, m, out=out)
    side = torch.cuda.Stream()
    got = []
    for busy in (False, True):
        B = hub.Basis(ring(n), 8.0, n // 2, n // 2, device=0)
        try:
            hub.hub_set_propagate_path(B.handle, 0)
            assert len(hub.hub_get_plan(B.handle, hub.HUB_C128 if dtype == torch.complex128 else hub.HUB_C64, nvec)) > 1
            g = torch.Generator(device=DEV).manual_seed(3)
            x = torch.randn(nvec, B.dim, dtype=dtype, device=DEV, generator=g)
            x /= torch.linalg.vector_norm(x, dim=1, keepdim=True)
            torch.cuda.synchronize()
            if busy:  # about as long as a third of the propagation
                for _ in range(4):
                    torch.mm(m, m, out=out)
            _, obs, _ = hub.hub_propagate(B.handle, pulses, 0.0, 0.002, steps, hub.make_opts(tol=1e-7, m_max=30), x,
                                          stream=side)
            got.append((x.clone(), obs))
            torch.cuda.synchronize()
        finally:
            B.close()
    assert torch.equal(got[0][0], got[1][0])
    assert np.array_equal(got[0][1], got[1][1])
