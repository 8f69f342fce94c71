"""Default launch plans at the edges of their rules.

FP32 products with spin exchange and pair hopping: 256 threads where columns are
short or the grid has more than two blocks a CU, else 512 (the product's result
does not depend on it).  One workgroup for the whole sector up to a state a
thread, without such terms and without phonons."""
import numpy as np
import pytest

from oracle import fock
from paper_2105_06806_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def edx():
    import torch
    from paper_2105_06806_amd import edx as E
    assert torch.cuda.is_available()
    return E


@pytest.mark.parametrize("norb,nbath,nup,ndw,threads", [
    (2, 6, 6, 12, 512),      # 3003 rows, 91 columns
    (3, 4, 10, 14, 512),     # 3003 rows, 15 columns
    (3, 3, 6, 3, 512),       # 924 rows, 220 columns
    (3, 3, 6, 6, 256),       # 924 rows, 924 columns
    (3, 3, 4, 3, 256),       # 495 rows, 220 columns
])
def test_threads_with_nd_terms(edx, norb, nbath, nup, ndw, threads):
    import torch
    m = inputs.make_model(norb, nbath, 2.5, Jh=0.4, seed=91, symmetric=False, Jx=0.4, Jp=0.3)
    S = edx.build_sector(m, nup, ndw)
    assert edx.get_plan(S, "f32")["col_threads"] == threads
    x = torch.as_tensor(inputs.random_vector(S.dim, seed=3), dtype=torch.float32, device="cuda")
    y = edx.hv(S, x, torch.empty_like(x)).clone()
    for other in (256, 512):
        edx.set_plan(S, "f32", col_threads=other)
        assert torch.equal(edx.hv(S, x, torch.empty_like(x)), y)
    if S.dim <= 50000:
        ref = fock.explicit_hamiltonian(m, nup, ndw) @ x.double().cpu().numpy()
        # FP32 terms, about 25 an element, each rounded once
        assert np.abs(y.double().cpu().numpy() - ref).max() <= 2e-6 * np.abs(ref).max()


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("norb,nbath,nup,ndw,kw,mode", [
    (1, 0, 1, 0, {}, 0),
    (1, 7, 2, 2, {}, 0),                              # 784 states
    (2, 2, 3, 3, {}, 0),
    (1, 6, 3, 3, {}, 2),                              # 1225 states
    (1, 7, 4, 4, {}, 2),
    (2, 2, 3, 3, dict(Jx=0.4, Jp=0.3), 2),
    (1, 4, 2, 2, dict(nph=2, w0=0.5, g=0.3), 2),
])
def test_smallest_sectors_in_one_workgroup(edx, norb, nbath, nup, ndw, kw, mode, dtype):
    import torch
    m = inputs.make_model(norb, nbath, 2.5, Jh=0.4 if norb > 1 else 0.0, seed=92, symmetric=False, **kw)
    S = edx.build_sector(m, nup, ndw)
    assert edx.get_plan(S, dtype)["mode"] == mode
    td = torch.float64 if dtype == "f64" else torch.float32
    x = torch.as_tensor(inputs.random_vector(S.dim, seed=4), dtype=td, device="cuda")
    y = edx.hv(S, x, torch.empty_like(x)).double().cpu().numpy()
    if not kw.get("nph"):
        ref = fock.explicit_hamiltonian(m, nup, ndw) @ x.double().cpu().numpy()
        # at most 25 terms an element, each rounded once
        assert np.abs(y - ref).max() <= (1e-14 if dtype == "f64" else 2e-6) * max(1.0, np.abs(ref).max())
    p = S.ld
    v = edx.pad(S, x)
    w = edx.unpad(S, edx.hv(S, v, torch.full_like(v, float("nan")), ld=p))
    assert np.array_equal(w.double().cpu().numpy(), y)


@pytest.mark.parametrize("nbath,nup,ndw,nph", [
    (11, 6, 6, 2), (11, 6, 6, 3),          # 8-slot rows below and above 12 MiB of slices
    (13, 10, 10, 2), (13, 10, 10, 3),      # 16-slot rows
    (13, 9, 7, 1), (10, 5, 4, 40),         # one spin's rows wide; many slices
])
def test_phonon_slices_by_either_load_path(edx, nbath, nup, ndw, nph):
    """FP32 products on dense, odd and padded columns take buffer or global loads
    by their size and stride: the same terms in the same order, so the same bits."""
    import torch
    m = inputs.make_model(1, nbath, 2.5, seed=93, symmetric=False, nph=nph, w0=0.5, g=0.3)
    S = edx.build_sector(m, nup, ndw)
    nc = S.ddw * S.dph
    x = torch.as_tensor(inputs.random_vector(S.dim, seed=5), device="cuda").view(nc, S.dup)
    y64 = edx.hv(S, x.reshape(-1), torch.empty(S.dim, dtype=torch.float64, device="cuda")).view(nc, S.dup)
    ref = None
    for ld in (S.dup, S.dup + 1, (S.dup + 31) // 32 * 32):
        v = torch.full((nc, ld), float("nan"), dtype=torch.float32, device="cuda")
        v[:, : S.dup] = x
        w = torch.full((nc, ld), 5.0, dtype=torch.float32, device="cuda")
        edx.hv(S, v.view(-1), w.view(-1), ld=ld)
        assert torch.count_nonzero(w[:, S.dup:]) == 0
        if ref is None:
            ref = w[:, : S.dup].clone()
            # FP32 against the FP64 product: about 20 terms an element
            assert float((ref.double() - y64).abs().max()) <= 2e-6 * float(y64.abs().max())
        assert torch.equal(w[:, : S.dup], ref), ld


@pytest.mark.parametrize("nup,ndw,nph,threads,order", [
    (6, 6, 1, 512, 4),       # 3003 x 3003: a second round of 256-thread blocks would be half empty
    (7, 7, 1, 256, 4),       # 3432 x 3432
    (10, 7, 1, 256, 1),      # 1001 x 3432: below 16 MiB a slice
    (6, 6, 0, 256, 1),
])
def test_plans_with_nd_terms_and_phonons(edx, nup, ndw, nph, threads, order):
    import torch
    m = inputs.make_model(2, 6, 2.5, Jh=0.4, seed=94, symmetric=False, Jx=0.4, Jp=0.3, nph=nph, w0=0.5, g=0.3)
    S = edx.build_sector(m, nup, ndw)
    p = edx.get_plan(S, "f32")
    assert (p["col_threads"], p["col_order"]) == (threads, order)
    x = torch.rand(S.dim, device="cuda", generator=torch.Generator(device="cuda").manual_seed(6))
    y = edx.hv(S, x, torch.empty_like(x)).clone()
    edx.set_plan(S, "f32", col_threads=512, col_order=0)
    assert torch.equal(edx.hv(S, x, torch.empty_like(x)), y)
