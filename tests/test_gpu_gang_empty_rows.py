"""Gang solves (gang.hip) of systems with empty rows (zero right-hand side
there: singular but consistent, as when a system is padded to a size).  64 of
them side by side make a slice of the sliced-ELL copy without entries: the
first one, one between others, the last one with a single row; Q1 rows are
held in registers (at most nine entries), Q2 rows are read in chunks and
sorted.

The padded rows never enter the iteration, so the iterate is that of the
system without them: against the oracle on it, with the 1e-8 of the other
trajectory tests, and exactly zero on the padding."""
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


def _pad(s, at, k):
    """s with k empty rows and columns in front of row `at`; kept: rows of s."""
    kept = np.concatenate([np.arange(at), np.arange(at, s.n) + k])
    lens = np.zeros(s.n + k, np.int32)
    zlens = np.zeros(s.n + k, np.int32)
    lens[kept] = np.diff(s.rowptr)
    zlens[kept] = np.diff(s.z_rowptr)
    b = np.zeros(s.n + k)
    b[kept] = s.b
    ptr = lambda v: np.concatenate([[0], np.cumsum(v)]).astype(np.int32)
    return W.System(s.n + k, ptr(lens), kept[s.colind].astype(np.int32), s.vals, b, s.r, ptr(zlens),
                    s.z_colind, s.z_vals), kept


def _check(x, kept, ref, what):
    assert not np.delete(x, kept).any(), what
    r = float(np.linalg.norm(x[kept] - ref) / np.linalg.norm(ref))
    print(what, f"{r:.2e}", flush=True)
    assert r <= 1e-8, (what, r)


# mesh, order, s: rows (64 x 64 for 63, 1); at, k: the padding.
@pytest.mark.parametrize("prec", ["fp64", "mixed_f32"])
@pytest.mark.parametrize("mesh,order,s,at,k", [
    (63, 1, 4, 0, 64),        # the first slice
    (63, 1, 0, 4096, 1),      # the last one, of one row
    (40, 1, 2, 640, 200),     # between others
    (300, 1, 4, 0, 130),      # two row slots a thread
    (20, 2, 2, 0, 64),        # Q2
    (20, 2, 0, 512, 300),
])
def test_solve_with_empty_slices(mesh, order, s, at, k, prec):
    from paper_1906_04051_amd import gmres as G
    base = (W.convection_diffusion_manufactured(mesh, s=s) if order == 1 else W.make_config(3, mesh=mesh))
    if order == 2 and s == 0:
        base.r, base.z_rowptr = 0, np.zeros(base.n + 1, np.int32)
        base.z_colind, base.z_vals = np.zeros(0, np.int32), np.zeros(0)
    sysm, kept = _pad(base, at, k)
    if prec == "fp64":
        kw, ref = dict(rtol=0.0, max_iters=45), oracle.gmres(base, 20, 0.0, 45).x
    else:
        kw, ref = dict(rtol=1e-11, max_iters=50000, precision=prec), oracle.gmres(base, 20, 1e-12, 50000).x
    plan, d = G.plan_for(sysm, m=20, **kw)
    x, info = plan.solve(d["b"])
    plan.close()
    if prec == "fp64":
        assert info["iters"] == 45
    else:
        assert info["rel_res_true"] <= 1e-11
    _check(x.cpu().numpy(), kept, ref, (mesh, order, at, k, prec))


def test_batch_with_empty_slices():
    from paper_1906_04051_amd import gmres as G
    base = [W.convection_diffusion_manufactured(mesh, s=2) for mesh in (31, 40, 24, 47)]
    pads = [_pad(s, at, k) for s, (at, k) in zip(base, ((0, 200), (1000, 130), (0, 64), (2304, 129)))]
    batch = W.concat_systems([p[0] for p in pads])
    plan, d = G.plan_for(batch, m=20, rtol=0.0, max_iters=45)
    x, infos = plan.solve_batched(d["b"])
    x = x.cpu().numpy()
    plan.close()
    for i, s in enumerate(base):
        assert infos[i]["iters"] == 45
        _check(x[batch.row_off[i]:batch.row_off[i + 1]], pads[i][1], oracle.gmres(s, 20, 0.0, 45).x, i)


@pytest.mark.parametrize("n", [1, 64, 300])
def test_matrix_without_entries(n):
    """b = 0 is solved by x0; nothing may be read from the empty copy."""
    from paper_1906_04051_amd import gmres as G
    rp = torch.zeros(n + 1, dtype=torch.int32, device="cuda")
    plan = G.Plan(rp, torch.zeros(0, dtype=torch.int32, device="cuda"),
                  torch.zeros(0, dtype=torch.float64, device="cuda"), m=5, rtol=1e-8, max_iters=20)
    x0 = torch.arange(n, dtype=torch.float64, device="cuda")
    x, info = plan.solve(torch.zeros(n, dtype=torch.float64, device="cuda"), x0=x0)
    assert info["iters"] == 0 and info["status_name"] == "OK" and torch.equal(x, x0)
    plan.close()
