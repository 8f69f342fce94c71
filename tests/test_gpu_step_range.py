"""Lanczos steps at the ends of FP64's range.

Start vectors of any norm whose square FP64 holds, and parameters of any unit:
a power of two scales every number of a run exactly (sums and products round
alike), so energies, step counts and Green's functions of the scaled problem are
the scaled ones of the plain problem, to the rounding of a run (1e-12 of E,
1e-10 of G).
"""
import numpy as np
import pytest

from paper_2105_06806_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def edx():
    import torch
    from paper_2105_06806_amd import edx as E
    assert torch.cuda.is_available()
    return E


def _scaled(m, s):
    out = dict(m)
    for k in ("eps_imp", "eps_bath", "vhyb", "U", "Ust", "Jh", "xmu", "Jx", "Jp"):
        if k in m:
            out[k] = np.asarray(m[k], dtype=np.float64) * s
    return out


@pytest.mark.parametrize("reorth", [0, 1, 2])
@pytest.mark.parametrize("power", [511, -480])
def test_start_vector_of_any_norm(edx, power, reorth):
    """Unit vector times 2^511: its square is 2^1022, and <u, H u> beyond FP64."""
    import torch
    m = dict(inputs.make_model(1, 7, 2.0, seed=41, symmetric=False), xmu=30.0)
    S = edx.build_sector(m, 4, 3)
    g = torch.Generator(device="cuda").manual_seed(2)
    x = torch.randn(S.dim, dtype=torch.float64, device="cuda", generator=g)
    x /= x.norm()
    kw = dict(niter=300, tol=1e-13, rtol=1e-10, reorth=reorth)
    e, psi, rep, _ = edx.lanczos_ground_state(S, start=x, **kw)
    y = x * 2.0 ** power
    es, ps, reps, _ = edx.lanczos_ground_state(S, start=y, **kw)
    assert rep["converged"] and reps["converged"]
    assert abs(es - e) <= 1e-12 * abs(e) and reps["iters"] == rep["iters"]
    assert abs(abs(float(psi @ ps)) - 1.0) <= 1e-12


def test_energy_of_parameters_of_any_unit(edx):
    """Parameters of the order 2^350: their cubes are beyond FP64."""
    s = 2.0 ** 350
    m = dict(inputs.make_model(1, 7, 2.0, seed=42, symmetric=False), xmu=10.0)
    S, T = edx.build_sector(m, 4, 4), edx.build_sector(_scaled(m, s), 4, 4)
    kw = dict(niter=300, tol=1e-13, seed=3)
    e, psi, rep, _ = edx.lanczos_ground_state(S, **kw)
    es, ps, reps, _ = edx.lanczos_ground_state(T, **kw)
    assert abs(es / s - e) <= 1e-12 * abs(e) and reps["iters"] == rep["iters"]
    assert abs(abs(float(psi @ ps)) - 1.0) <= 1e-12


@pytest.mark.parametrize("power", [320, -320])
def test_green_of_parameters_of_any_unit(edx, power):
    """As far as the continued fraction goes, which forms cubes itself."""
    s = 2.0 ** power
    m = dict(inputs.make_model(1, 7, 2.0, seed=42, symmetric=False), xmu=10.0)
    S, T = edx.build_sector(m, 4, 4), edx.build_sector(_scaled(m, s), 4, 4)
    e, psi, _, _ = edx.lanczos_ground_state(S, niter=300, tol=1e-13, seed=3)
    g, _ = edx.green_cf(S, psi, e, 0, 0, ngf=40, beta=50.0, lmats=64)
    gs, _ = edx.green_cf(T, psi, e * s, 0, 0, ngf=40, beta=50.0 / s, lmats=64)
    dev = np.abs(np.asarray(gs) * s - np.asarray(g)).max()
    assert dev <= 1e-10 * np.abs(np.asarray(g)).max()
