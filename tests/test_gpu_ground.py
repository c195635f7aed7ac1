"""Ground states at the edges of their iteration (hub_ground_state): runs that
close in an invariant subspace, spaces of fewer vectors than a batch of
iterations and of no whole number of batches, restarts, and a tolerance below
what two orthogonalisations a batch can hold.  The residual
|H x - E0 x| is at most the tolerance's share of |H|_inf and the rounding of
the combination, the product and the norms, allowed 256 eps |H|_inf; E0 is a
Rayleigh quotient, within as much of the lowest eigenvalue."""
import numpy as np
import pytest
import torch

import paper_2005_13498_amd as hub
from oracle import HubbardOracle, ground_state
from synth import chain, ring

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("lat,nu,nd,tol,m_max", [
    (ring(5), 0, 0, 1e-12, 60), (chain(3), 1, 1, 1e-12, 60), (chain(4), 2, 1, 1e-12, 2), (ring(6), 3, 3, 1e-13, 60),
    (ring(6), 3, 3, 1e-8, 5), (chain(8), 4, 4, 1e-10, 8), (chain(8), 4, 4, 1e-15, 60), (chain(8), 4, 3, 1e-12, 100)])
def test_ground_state_residual(lat, nu, nd, tol, m_max):
    U = 8.0
    B = hub.Basis(lat, U, nu, nd, device=0)
    norm = hub.hub_basis_classes(B.handle)[2]
    v = torch.full((1, B.dim), float("nan"), dtype=torch.complex128, device=DEV)
    w = torch.empty_like(v)
    if norm == 0.0:  # no residual is below a tolerance of zero: refused, as it always was
        with pytest.raises(hub.HubError, match="NOT_CONVERGED"):
            hub.hub_ground_state(B.handle, 0.3, v, hub.make_opts(tol=tol, m_max=m_max))
        B.close()
        return
    st, e0, gap = hub.hub_ground_state(B.handle, 0.3, v, hub.make_opts(tol=tol, m_max=m_max), allow_degenerate=True)
    hub.hub_apply_H(B.handle, 0.3, v, w)
    x, y = v[0].cpu().numpy(), w[0].cpu().numpy()
    B.close()
    bound = (tol + 256 * 2.0 ** -52) * max(norm, 1.0)
    assert abs(np.linalg.norm(x) - 1.0) <= 256 * 2.0 ** -52
    assert np.linalg.norm(y - e0 * x) <= bound
    ham = HubbardOracle(lat, U, nu, nd)
    E0 = ground_state(ham, 0.3)[0] if ham.dim > 2 else float(np.real(y[0] / x[0]))
    assert abs(e0 - E0) <= bound + 1e-10 * abs(E0)


@pytest.mark.parametrize("lat,nu,nd", [(chain(3), 1, 1), (chain(4), 2, 1), (ring(6), 3, 3), (chain(6), 3, 2), (ring(5), 2, 1),
                                       (chain(5), 2, 2)])
@pytest.mark.parametrize("tol,m_max", [(1e-6, 60), (1e-8, 16), (1e-12, 60), (1e-12, 10), (1e-15, 60)])
def test_energy_and_gap_against_dense_eigenvalues(lat, nu, nd, tol, m_max):
    """E0 within (tol + 256 eps) |H|_inf of the lowest eigenvalue, and the gap,
    whose vector has a residual of 1e-6 |H|, second order in that but for the
    quarter of 1e-9 |H| that its vectors may have lost of their orthogonality:
    runs that close, that restart, and that converge within one batch."""
    U = 8.0
    ham = HubbardOracle(lat, U, nu, nd)
    H = np.column_stack([ham.apply(0.3, e) for e in np.eye(ham.dim, dtype=complex)])
    ev = np.linalg.eigvalsh(H)
    B = hub.Basis(lat, U, nu, nd, device=0)
    norm = hub.hub_basis_classes(B.handle)[2]
    v = torch.empty(1, B.dim, dtype=torch.complex128, device=DEV)
    st, e0, gap = hub.hub_ground_state(B.handle, 0.3, v, hub.make_opts(tol=tol, m_max=m_max))
    B.close()
    assert abs(e0 - ev[0]) <= (tol + 256 * 2.0 ** -52) * norm
    assert abs(gap - (ev[1] - ev[0])) <= (1e-6 * norm) ** 2 / (ev[2] - ev[1]) + (tol + 1e-9) * norm
