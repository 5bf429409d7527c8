"""Whole solves in one cooperative launch (gang.hip) against the
kernel-per-phase engine and the FP64 oracle, at the sizes where the launch
shape changes: one workgroup, the last workgroup nearly empty, one to four row
slots a thread, basis columns beyond LDS, a solve longer than one launch.

Both paths build the same Krylov spaces, so fixed-count iterates agree to
rounding amplified over the steps; the gate is the 1e-8 of the other
trajectory tests."""
import numpy as np
import pytest

import oracle
from paper_1906_04051_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    from paper_1906_04051_amd import gmres as G
    G.load_library()
    yield


def _solve(s, x0=None, **opts):
    from paper_1906_04051_amd import gmres as G
    plan, d = G.plan_for(s, **opts)
    x, info = plan.solve(d["b"], x0=None if x0 is None else torch.from_numpy(x0).cuda())
    h = plan.history() if opts.get("record_history") else None
    x = x.cpu().numpy()
    plan.close()
    return x, info, h


def _close(a, b, what):
    r = float(np.linalg.norm(a - b) / np.linalg.norm(b))
    print(what, f"{r:.2e}", flush=True)
    assert r <= 1e-8, (what, r)


# mesh, s, m, steps: n = (mesh + 1)^2 rows, 256 rows a workgroup up to 65,536.
@pytest.mark.parametrize("mesh,s,m,steps", [
    (15, 0, 7, 20),       # 256 rows: one workgroup
    (15, 2, 30, 31),
    (16, 2, 10, 25),      # 289: the second workgroup holds 33 rows
    (100, 16, 40, 45),    # 256 deflation columns
    (254, 4, 30, 40),     # 65,025 rows: 255 workgroups
    (256, 8, 80, 90),     # 66,049 rows, 80 columns: basis beyond LDS
    (362, 8, 12, 20),     # 131,769: two row slots
    (512, 4, 12, 20),     # 263,169: three
])
def test_gang_matches_engine_and_oracle(mesh, s, m, steps):
    sysm = W.convection_diffusion_lognormal(mesh, (20.0, 5.0), 1.0, s, W.config_seed(2))
    x0 = np.random.default_rng(5).uniform(-1, 1, sysm.n)
    kw = dict(m=m, rtol=0.0, max_iters=steps)
    xg, ig, hg = _solve(sysm, x0, record_history=1, **kw)
    xe, ie, he = _solve(sysm, x0, record_history=1, num_blocks=64, **kw)   # the per-phase engine
    assert ig["iters"] == ie["iters"] == steps and ig["cycles"] == ie["cycles"]
    assert abs(ig["rho0"] - ie["rho0"]) <= 1e-12 * ie["rho0"]
    _close(xg, xe, "engine")
    _close(hg, he, "history")
    if sysm.n <= 70000:
        _close(xg, oracle.gmres(sysm, m, 0.0, steps, x0=x0).x, "oracle")


def test_gang_sorted_wide_rows():
    """Q2 rows (9 to 25 entries): chunked row products."""
    s = W.make_config(3, mesh=40)
    kw = dict(m=30, rtol=0.0, max_iters=45)
    _close(_solve(s, **kw)[0], oracle.gmres(s, 30, 0.0, 45).x, "q2")


@pytest.mark.parametrize("prec,mesh", [("mixed_f32", 90), ("mixed_f16", 90), ("mixed_f32", 627), ("mixed_f16", 513)])
def test_gang_mixed_reaches_tolerance(prec, mesh):
    """Reduced-precision inner solves (627 x 627: four row slots): the FP64
    true residual meets the tolerance and the engine's solution is met within
    the two residuals (the smooth load makes ||A^-1|| ||r|| / ||x|| at most
    the relative residual)."""
    s = W.convection_diffusion_manufactured(mesh, s=8)
    kw = dict(m=30, rtol=1e-9, max_iters=100000, precision=prec)
    xg, ig, _ = _solve(s, **kw)
    xe, ie, _ = _solve(s, num_blocks=256, **kw)
    assert ig["status_name"] == ie["status_name"] == "OK"
    assert ig["rel_res_true"] <= 1e-9
    _close(xg, xe, prec)


@pytest.mark.parametrize("mesh,m,rmax,steps", [
    (15, 7, 2, 40),       # one workgroup; columns of U removed
    (40, 20, 22, 130),    # fewer cycles than columns
    (128, 64, 9, 150),    # U's columns cross a group of eight
    (362, 12, 3, 50),     # two row slots
    (512, 30, 4, 70),     # three row slots, basis beyond LDS
])
def test_gang_adaptive_matches_engine(mesh, m, rmax, steps):
    """One launch a cycle, the Ritz step between them."""
    sysm = W.convection_diffusion_manufactured(mesh, beta=(20.0, 5.0), s=0)
    kw = dict(m=m, rtol=0.0, max_iters=steps, adapt_rmax=rmax, record_history=1)
    xg, ig, hg = _solve(sysm, **kw)
    xe, ie, he = _solve(sysm, num_blocks=64, **kw)
    assert ig["iters"] == ie["iters"] == steps and ig["cycles"] == ie["cycles"]
    assert ig["defl_r"] == ie["defl_r"]
    _close(xg, xe, "engine")
    _close(hg, he, "history")


def test_gang_solve_longer_than_one_launch():
    """m = 2: a launch ends after 4,096 cycles; the next ones resume."""
    s = W.convection_diffusion_manufactured(20, beta=(60.0, 10.0), s=0)
    kw = dict(m=2, rtol=0.0, max_iters=8301)
    xg, ig, _ = _solve(s, **kw)
    xe, ie, _ = _solve(s, num_blocks=8, **kw)
    assert ig["iters"] == ie["iters"] == 8301 and ig["cycles"] == ie["cycles"]
    _close(xg, xe, "resumed")


def test_gang_converges_like_the_engine():
    """To tolerance, with cycles that end on the estimate and x aliasing x0."""
    from paper_1906_04051_amd import gmres as G
    s = W.make_config(1)
    ref = oracle.gmres(s, 30, 1e-8, 2000)
    plan, d = G.plan_for(s, m=30, rtol=1e-8, max_iters=2000)
    x = torch.zeros_like(d["b"])
    _, info = plan.solve(d["b"], x0=x, out=x)
    assert info["status_name"] == "OK" and abs(info["iters"] - ref.iters) <= 1
    _close(x.cpu().numpy(), ref.x, "aliased")
    bad = d["b"].clone()
    bad[7] = float("nan")
    with pytest.raises(G.GmresError):
        plan.solve(bad)
    z, info = plan.solve(torch.zeros_like(bad))
    assert info["iters"] == 0 and float(z.abs().max()) == 0.0
    plan.close()


@pytest.mark.parametrize("lo,hi,ns,s,m,steps", [
    (16, 40, 5, 2, 30, 60),      # one- to four-workgroup gangs
    (24, 90, 6, 0, 64, 70),      # no deflation basis; basis beyond LDS
    (16, 96, 40, 4, 30, 60),     # several systems a gang
    (230, 256, 3, 4, 10, 25),    # gangs of 128 and more
])
def test_gang_batch_matches_one_workgroup_a_system(lo, hi, ns, s, m, steps):
    from paper_1906_04051_amd import gmres as G
    batch = W.make_batch(ns, lo, hi, s)
    x0 = torch.from_numpy(np.random.default_rng(3).uniform(-1, 1, batch.b.size)).cuda()
    res = []
    for kw in (dict(), dict(batch_wg=256)):
        plan, d = G.plan_for(batch, m=m, rtol=0.0, max_iters=steps, **kw)
        x = x0.clone()
        plan.solve_batched(d["b"], x0=x, out=x)
        y, infos = plan.solve_batched(d["b"])
        res.append((x.cpu().numpy(), y.cpu().numpy(), infos))
        plan.close()
    for i in range(ns):
        a, b = (r[2][i] for r in res)
        assert a["iters"] == b["iters"] == steps and a["cycles"] == b["cycles"]
        r0, r1 = batch.row_off[i], batch.row_off[i + 1]
        _close(res[0][0][r0:r1], res[1][0][r0:r1], f"system {i} from x0")
        _close(res[0][1][r0:r1], res[1][1][r0:r1], f"system {i}")


def test_gang_batch_to_tolerance():
    from paper_1906_04051_amd import gmres as G
    batch = W.make_batch(12, 16, 110, 4)
    plan, d = G.plan_for(batch, m=30, rtol=1e-9, max_iters=20000)
    x, infos = plan.solve_batched(d["b"])
    for i, sysm in enumerate(batch.systems):
        r0, r1 = batch.row_off[i], batch.row_off[i + 1]
        xi = x[r0:r1].cpu().numpy()
        res = np.linalg.norm(sysm.b - oracle.spmv(sysm.rowptr, sysm.colind, sysm.vals, xi))
        assert infos[i]["status_name"] == "OK"
        assert res <= 1.001e-9 * np.linalg.norm(sysm.b)
    plan.close()
