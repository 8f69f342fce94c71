"""The FP32 product's row loops over 8, 10, 12 and all slots of a padded hop row.

Norb=1 columns with N electrons have N or Ns - N hops, so the sectors below have
blocks for each loop: at most 8, 9, 10, 11, 12 and 13 real hops of 16 slots, with
one to three columns a workgroup (the last one short), with phonons, and for
Norb=2 rows with mixed counts.  An element is a sum of about 2 x 16 terms, each
rounded to FP32: 32 half-ulps of 2^-24 of the largest partial sum, with a factor
2 to spare 4e-6 of the largest element.
"""
import numpy as np
import pytest

from oracle import eph, fock
from paper_2105_06806_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def edx():
    import torch
    from paper_2105_06806_amd import edx as E
    assert torch.cuda.is_available()
    return E


@pytest.mark.parametrize("norb,nbath,nup,ndw,kw", [
    (1, 9, 4, 9, {}),
    (1, 10, 3, 10, {}),
    (1, 11, 2, 11, {}),
    (1, 12, 2, 12, {}),
    (1, 13, 1, 13, {}),
    (1, 13, 2, 3, {}),           # 3 or 11 hops
    (2, 6, 2, 5, {}),
    (1, 10, 2, 9, dict(nph=2, w0=0.5, g=0.3)),
])
def test_row_loops(edx, norb, nbath, nup, ndw, kw):
    import torch
    m = inputs.make_model(norb, nbath, 3.0, seed=47, symmetric=False, **kw)
    S = edx.build_sector(m, nup, ndw)
    x = torch.as_tensor(inputs.random_vector(S.dim, seed=9), device="cuda").float()
    build = eph.explicit_hamiltonian if kw else fock.explicit_hamiltonian
    y = build(m, nup, ndw) @ x.double().cpu().numpy()
    tol = 4e-6 * np.abs(y).max()
    for cols in (1, 2, 3):
        for order in (1, 2):
            edx.set_plan(S, "f32", mode=2, col_cols=cols, col_threads=256, col_order=order)
            w = torch.empty_like(x)
            edx.hv(S, x, w)
            assert np.abs(w.double().cpu().numpy() - y).max() <= tol, (cols, order)
