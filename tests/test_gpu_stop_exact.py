"""Stop rules without slack: tol = 0 waits until the lowest Ritz value does not
change at all (two steps in the same cell of the bisection), alone, with a
residual rule and through the batch, and still ends converged well before niter."""
import functools

import pytest
from scipy.sparse.linalg import eigsh

from oracle import fock
from paper_2105_06806_amd import inputs

pytestmark = pytest.mark.gpu

SECTORS = [(1, 7, 4, 4), (1, 8, 3, 5), (2, 3, 4, 3), (3, 2, 4, 4)]


@pytest.fixture(scope="module")
def edx():
    import torch
    from paper_2105_06806_amd import edx as E
    assert torch.cuda.is_available()
    return E


def _model(norb, nbath):
    return inputs.make_model(norb, nbath, 2.5, Jh=0.3 if norb > 1 else 0.0, seed=61, symmetric=False)


@functools.lru_cache(maxsize=None)
def _oracle_energy(norb, nbath, nup, ndw):
    return float(eigsh(fock.explicit_hamiltonian(_model(norb, nbath), nup, ndw), k=1, which="SA",
                       return_eigenvectors=False)[0])


@pytest.mark.parametrize("norb,nbath,nup,ndw", SECTORS)
@pytest.mark.parametrize("reorth,rtol", [(0, 0.0), (0, 1e-9), (1, 0.0), (2, 0.0), (3, 1e-9)])
def test_energy_settles_exactly(edx, norb, nbath, nup, ndw, reorth, rtol):
    S = edx.build_sector(_model(norb, nbath), nup, ndw)
    e = _oracle_energy(norb, nbath, nup, ndw)
    for seed in range(4):
        e0, _, rep, st = edx.lanczos_ground_state(S, want_psi=False, niter=300, tol=0.0, rtol=rtol, seed=seed,
                                                  reorth=reorth, allow=(edx.EDX_E_NOCONV,))
        assert st == edx.EDX_OK and rep["converged"] == 1 and rep["iters"] < 150
        assert abs(e0 - e) <= 1e-12 * abs(e)


def test_batch_energies_settle_exactly(edx):
    ms = [inputs.make_model(1, 8, 2.5, seed=62 + k, symmetric=False) for k in range(4)]
    secs = [edx.build_sector(m, a, b) for m in ms for a, b in ((4, 5), (5, 4), (3, 4))]
    out, _ = edx.batch_ground_state(secs, vtype="f64", niter=300, tol=0.0, check_every=4, seed=3)
    assert all(r["status"] == 0 and r["iters"] < 200 for r in out)
