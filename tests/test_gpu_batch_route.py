"""Batched ground states without a threshold: every job off the lanes.

The energies and step counts are those of the lanes (tol looked at every
check_every steps); a workspace that only holds the lanes' vectors sends the
jobs there.  FP64 energies of two runs that stop at the same step differ by
rounding (1e-11 of |T|); FP32 ones by the FP32 floor of the stop rule (2e-5).
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

RTOL = {"f64": 1e-11, "f32": 2e-5}


@pytest.fixture(scope="module")
def edx():
    import torch
    from paper_2105_06806_amd import edx as E
    assert torch.cuda.is_available()
    return E


def _tiles(n, wide):
    return {"lane_wgs": 32, "multi_k": 0, "ccols": np.full(n, 1, np.int32),
            "rcols": np.full(n, 32, np.int32), "wide_min_dim": wide}


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("nsets,cycle,spread,every", [
    (1, (4,), 0, 4),            # one job
    (2, (3, 3), 1, 1),          # groups of two sets, edge sectors
    (5, (6, 8, 9), 2, 4),       # groups and single jobs
    (9, (7,), 1, 8),            # groups of eight and one left over
])
def test_default_route_gives_the_lanes_results(edx, dtype, nsets, cycle, spread, every):
    from paper_2105_06806_amd import inputs
    jobs = inputs.batch_jobs(nsets, seed_base=7100, ns_cycle=cycle, spread=spread)
    secs = [edx.build_sector(m, a, b) for _, m, a, b in jobs]
    kw = dict(vtype=dtype, niter=256, tol=1e-9, check_every=every, seed=23)
    lanes, _ = edx.batch_ground_state(secs, tiles=_tiles(len(secs), -1), **kw)
    need = edx.batch_workspace_bytes(secs, dtype, 32, -1)
    for ws in (None, edx.alloc_workspace(need)):
        out, _ = edx.batch_ground_state(secs, ws=ws, **kw)
        for a, b in zip(out, lanes):
            assert a["status"] == b["status"] == 0
            assert abs(a["e0"] - b["e0"]) <= RTOL[dtype] * max(1.0, abs(b["e0"]))
            if dtype == "f64" and not b["breakdown"]:
                assert a["iters"] == b["iters"]


def test_mixed_sectors_of_one_shape(edx):
    """Sectors of one shape of which only some suit the multi-set pass (spin
    exchange, phonons, per-orbital counts) each get their own ground energy."""
    from paper_2105_06806_amd import inputs
    kan = [inputs.make_model(2, 2, 2.0, Jh=j, seed=7200 + i, symmetric=False)
           for i, j in enumerate((0.0, 0.3, 0.0, 0.3))]
    ph = [inputs.make_model(1, 5, 2.0, seed=7210 + i, symmetric=False, **kw)
          for i, kw in enumerate((dict(), dict(nph=2, w0=0.6, g=0.35), dict()))]
    secs = [edx.build_sector(m, 3, 3) for m in kan + ph]
    secs += [edx.build_sector_orbital(kan[i], (2, 1), (1, 2)) for i in (0, 2)]
    kw = dict(vtype="f64", niter=256, tol=1e-12, check_every=4, seed=29)
    out, _ = edx.batch_ground_state(secs, **kw)
    for s, r in zip(secs, out):
        e0, _, _, _ = edx.lanczos_ground_state(s, want_psi=False, **kw)
        assert r["status"] == 0 and abs(r["e0"] - e0) <= 1e-10 * max(1.0, abs(e0))
