"""Which kernels a solve runs on (gmres_gang_counts): whole solves in
one launch (gang.hip) where the plan's options leave the choice to
the library and the system fits, with no launch given up; the kernel-per-phase
engine (or one workgroup per system of a batch) where an option asks for it or
the system is too large.  The comparisons of test_gpu_gang.py compare the two
only if this holds."""
import numpy as np
import pytest

from paper_1906_04051_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

GANG = dict(gang=1, given_up=0, other=0)
OTHER = dict(gang=0, given_up=0, other=1)


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    from paper_1906_04051_amd import gmres as G
    G.load_library()
    yield


def _plan(mesh, s=0, **opts):
    from paper_1906_04051_amd import gmres as G
    return G.plan_for(W.convection_diffusion_manufactured(mesh, s=s), **opts)


FIXED = dict(m=12, rtol=0.0, max_iters=20)


@pytest.mark.parametrize("mesh,s,opts", [
    (15, 0, FIXED),
    (16, 2, FIXED),
    (100, 16, FIXED),
    (254, 4, FIXED),
    (256, 8, dict(m=80, rtol=0.0, max_iters=90)),
    (362, 8, FIXED),
    (512, 4, FIXED),
    (100, 4, dict(FIXED, spmv_lanes=-64)),
    (100, 4, dict(FIXED, record_history=1)),
    (100, 4, dict(FIXED, use_graph=0)),
    (40, 0, dict(FIXED, adapt_rmax=3)),
    (512, 0, dict(FIXED, adapt_rmax=3)),
])
def test_solves_in_one_launch(mesh, s, opts):
    plan, d = _plan(mesh, s, **opts)
    plan.solve(d["b"])
    assert plan.gang_counts() == GANG
    plan.close()


@pytest.mark.parametrize("mesh,opts", [
    (100, dict(num_blocks=64)),
    (100, dict(spmv_lanes=8)),
    (100, dict(spmv_lanes=-256)),
    (100, dict(ortho=0)),
    (100, dict(ortho=2)),
    (100, dict(adapt_rmax=3, num_blocks=64)),
    (800, dict()),            # 641,601 rows
])
def test_solves_on_the_engine(mesh, opts):
    plan, d = _plan(mesh, **FIXED, **opts)
    plan.solve(d["b"])
    assert plan.gang_counts() == OTHER
    plan.close()


def test_timed_solves_run_on_the_engine():
    plan, d = _plan(100, 4, **FIXED)
    plan.set_timing(1)
    plan.solve(d["b"])
    assert plan.gang_counts() == OTHER
    plan.set_timing(0)
    plan.solve(d["b"])
    assert plan.gang_counts() == dict(gang=1, given_up=0, other=1)
    plan.close()


@pytest.mark.parametrize("prec,mesh", [("mixed_f32", 90), ("mixed_f16", 90), ("mixed_f32", 627), ("mixed_f16", 513)])
def test_inner_solves_in_one_launch(prec, mesh):
    plan, d = _plan(mesh, 8, m=30, rtol=1e-9, max_iters=100000, precision=prec)
    _, info = plan.solve(d["b"])
    assert plan.gang_counts() == dict(gang=info["refinements"], given_up=0, other=0)
    plan.close()


def test_adjoint_in_one_launch():
    plan, d = _plan(64, 4, need_adjoint=True, m=30, rtol=1e-10)
    x, _ = plan.solve(d["b"])
    plan.adjoint(x, torch.ones_like(x))
    assert plan.gang_counts() == dict(gang=2, given_up=0, other=0)
    plan.close()


def test_rows_past_nine_entries_in_one_launch():
    from paper_1906_04051_amd import gmres as G
    plan, d = G.plan_for(W.make_config(3, mesh=40), **FIXED)
    plan.solve(d["b"])
    assert plan.gang_counts() == GANG
    plan.close()


@pytest.mark.parametrize("lo,hi,ns,s,m", [(16, 40, 5, 2, 30), (24, 90, 6, 0, 64), (16, 96, 40, 4, 30),
                                          (230, 256, 3, 4, 10)])
def test_batches(lo, hi, ns, s, m):
    from paper_1906_04051_amd import gmres as G
    batch = W.make_batch(ns, lo, hi, s)
    for kw, want in ((dict(), GANG), (dict(batch_wg=256), OTHER), (dict(batch_lanes=8), OTHER)):
        plan, d = G.plan_for(batch, m=m, rtol=0.0, max_iters=20, **kw)
        plan.solve_batched(d["b"])
        assert plan.gang_counts() == want, kw
        plan.close()


@pytest.mark.parametrize("prec", ["fp64", "mixed_f32", "mixed_f16"])
@pytest.mark.parametrize("mesh", [140, 200, 256])
def test_wide_rows_in_every_row_slot(mesh, prec):
    """Rows of 9 to 25 entries with one, two and three row slots a thread
    (78,961, 160,801 and 263,169 rows): the gang's iterate or solution is the
    engine's (fixed count: rounding over 20 steps, the 1e-8 of the other
    trajectory tests; mixed: both residuals at 1e-10 of ||b||, and ||A^{-1}|| ||b||
    / ||x||, 6.8 at 20 elements a side, belongs to the continuous problem)."""
    from paper_1906_04051_amd import gmres as G
    s = W.make_config(3, mesh=mesh)
    kw = dict(FIXED) if prec == "fp64" else dict(m=20, rtol=1e-10, precision=prec)
    out = []
    for extra in (dict(), dict(num_blocks=256)):
        plan, d = G.plan_for(s, **kw, **extra)
        x, info = plan.solve(d["b"])
        out.append(x)
        c = plan.gang_counts()
        assert c["given_up"] == 0 and c["gang" if not extra else "other"] == max(1, info["refinements"]), c
        if prec != "fp64":
            assert info["rel_res_true"] <= 1e-10
        plan.close()
    assert float((out[0] - out[1]).norm() / out[1].norm()) <= 1e-8


@pytest.mark.parametrize("prec,mesh,s,m,gang", [
    ("fp64", 511, 0, 46, True),           # 368 KB of basis a workgroup, limit 372
    ("fp64", 511, 0, 47, False),
    ("fp64", 511, 8, 57, True),           # 456 of 462
    ("fp64", 511, 8, 58, False),
    ("fp64", 511, 16, 87, True),          # 696 of 700 (the line: 750)
    ("fp64", 511, 16, 88, False),
    ("mixed_f32", 511, 0, 50, True),      # 200 of 200
    ("mixed_f32", 511, 0, 51, False),
    ("mixed_f16", 511, 0, 55, True),      # 110 of 111
    ("mixed_f16", 511, 0, 56, False),
    ("adaptive", 511, 0, 87, True),
    ("adaptive", 511, 0, 88, False),
])
def test_the_size_rule(prec, mesh, s, m, gang):
    """Both sides of each line (1,024 rows a workgroup): the same solution
    (one step to check the path; mixed: an inner tolerance any step meets)."""
    opts = dict(m=m, rtol=0.0, max_iters=1)
    if prec == "adaptive":
        opts["adapt_rmax"] = 3
    elif prec != "fp64":
        opts.update(precision=prec, max_refine=1, inner_max_iters=1, rtol=1e-8)
    plan, d = _plan(mesh, s, **opts)
    plan.solve(d["b"])
    assert plan.gang_counts() == (GANG if gang else OTHER)
    plan.close()
