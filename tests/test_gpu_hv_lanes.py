"""The FP64 product on 16-byte lanes against the row-a-lane pass and the oracle.

Three columns a workgroup take the row-a-lane pass; both passes sum the same
terms in the same order, so their products agree bit for bit.  Odd and even
numbers of rows and columns, dense columns and even and odd strides, one and
two columns a workgroup (with a short last one), hop rows of 8, 16 and 24 slots,
H_nd and phonon terms; the padding rows of w come out as zero and nothing past
its end is written.
"""
import numpy as np
import pytest

from oracle import kron
from paper_2105_06806_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def edx():
    import torch
    from paper_2105_06806_amd import edx as E
    assert torch.cuda.is_available()
    return E


CASES = [  # norb, nbath, nup, ndw, model keys
    (1, 10, 5, 4, {}),                                # 462 x 330 rows x columns
    (1, 12, 5, 3, {}),                                # 1287 rows (odd), 286 columns
    (1, 13, 9, 10, {}),                               # 16-slot rows, 1001 columns
    (3, 3, 5, 7, {}),                                 # 16-slot rows of both spins
    (3, 5, 3, 1, {}),                                 # 816 rows, few columns
    (2, 5, 6, 5, dict(Jx=0.4, Jp=0.3)),
    (3, 3, 6, 3, dict(Jx=0.5, Jp=0.5)),
    (1, 10, 5, 3, dict(nph=2, w0=0.5, g=0.3)),
]


@pytest.mark.parametrize("norb,nbath,nup,ndw,kw", CASES)
def test_lanes_equal_rows(edx, norb, nbath, nup, ndw, kw):
    import torch
    m = inputs.make_model(norb, nbath, 3.0, Jh=0.4, seed=31, symmetric=False, **kw)
    S = edx.build_sector(m, nup, ndw)
    nc = S.ddw * S.dph
    x = torch.as_tensor(inputs.random_vector(S.dim, seed=8), device="cuda")
    even = S.dup + (S.dup & 1) + 6
    ref = None
    for cols in (3, 1, 2):
        for threads in (256, 512):
            edx.set_plan(S, "f64", mode=2, col_cols=cols, col_threads=threads, col_order=1)
            for ld in (S.dup, even, even + 1):
                v = torch.full((nc, ld), float("nan"), dtype=torch.float64, device="cuda")
                v[:, : S.dup] = x.view(nc, S.dup)
                buf = torch.full((nc * ld + 64,), 5.0, dtype=torch.float64, device="cuda")
                w = buf[: nc * ld].view(nc, ld)
                for _ in range(3):     # repeated: a lost store would come and go
                    edx.hv(S, v.view(-1), w.view(-1), ld=ld)
                    assert torch.count_nonzero(w[:, S.dup:]) == 0
                    if ref is None:
                        ref = w[:, : S.dup].clone()
                    assert torch.equal(w[:, : S.dup], ref), (cols, threads, ld)
                assert bool((buf[nc * ld:] == 5.0).all())
    if not kw:
        y = kron.KronH(m, nup, ndw).matvec(x.cpu().numpy())
        scale = np.abs(y).max()
        # about 40 terms an element, each rounded once: 1e-13 of the largest element is 20 times that
        assert np.abs(ref.reshape(-1).cpu().numpy() - y).max() <= 1e-13 * scale
