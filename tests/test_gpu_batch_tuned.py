"""A tuned batch against the untuned one: the choice of lanes or whole-GPU path,
which depends on timings, must not change where a job stops.

Sectors below every threshold above 0 that the autotuner tries, so all jobs take
one path; the stop rule is tol alone, looked at every check_every steps, on
either (rtol would stop later, a check at every step earlier).
"""
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def edx():
    import torch
    from paper_2105_06806_amd import edx as E
    assert torch.cuda.is_available()
    return E


@pytest.mark.parametrize("nsets,cycle,spread", [(1, (11,), 0), (1, (11,), 1), (3, (7, 9), 1)])
def test_tuned_batch_stops_where_the_untuned_does(edx, nsets, cycle, spread):
    from paper_2105_06806_amd import inputs
    jobs = inputs.batch_jobs(nsets, seed_base=7300, ns_cycle=cycle, spread=spread)
    secs = [edx.build_sector(m, a, b) for _, m, a, b in jobs]
    assert max(s.dim for s in secs) < 250000
    kw = dict(vtype="f64", niter=256, tol=1e-7, rtol=1e-10, check_every=8, seed=31)
    ref, _ = edx.batch_ground_state(secs, **kw)
    assert any(r["iters"] % 8 == 0 for r in ref)
    ws = edx.alloc_workspace(edx.batch_workspace_bytes(secs, "f64", 8))
    tiles = edx.batch_autotune(secs, ws=ws, **kw)
    assert tiles["wide_min_dim"] in (-1, 0, 250000, 1000000, 2000000, 4000000, 8000000)
    out, _ = edx.batch_ground_state(secs, tiles=tiles, **kw)
    for a, b in zip(out, ref):
        assert (a["status"], a["iters"]) == (b["status"], b["iters"])
        # FP64 energies of runs that stop at the same step: rounding of |T|
        assert abs(a["e0"] - b["e0"]) <= 1e-11 * max(1.0, abs(b["e0"]))
