"""Adjoint solves where A has a sliced-ELL copy and A^T has none: every row of A
holds two entries, and every 64th column holds 64 of them, so the copy of A^T is
past the padding that a plan allows."""
import numpy as np
import pytest

from paper_1906_04051_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _system(n, r):
    rng = np.random.default_rng(n)
    i = np.arange(n)
    hub = i - i % 64
    rp = np.concatenate([[0], np.cumsum(1 + (hub != i))]).astype(np.int32)
    ci = np.stack([hub, i], 1)[np.stack([hub != i, i == i], 1)].astype(np.int32)
    v = rng.uniform(-0.05, 0.05, ci.size)
    v[ci == np.repeat(i, np.diff(rp))] = 4.0
    zrp = np.arange(n + 1, dtype=np.int32) if r else np.zeros(n + 1, np.int32)
    zci = (i * r // n).astype(np.int32) if r else np.zeros(0, np.int32)
    return W.System(n, rp, ci, v, rng.uniform(-1, 1, n), r, zrp, zci, np.ones(zci.size))


def test_no_copy_of_the_transpose():
    """The premise, from the sizes alone: a copy keeps at most 5/4 of the entries
    and 4096 more; rows are sorted within blocks of 256."""
    for n in (2048, 3000):
        s = _system(n, 0)
        for rows, fits in ((np.diff(s.rowptr), True), (np.bincount(s.colind, minlength=n), False)):
            rows = np.concatenate([rows, np.zeros(-n % 256, rows.dtype)]).reshape(-1, 256)
            stored = 64 * int((-np.sort(-rows, axis=1))[:, ::64].sum())
            assert (stored <= s.colind.size * 5 // 4 + 4096) == fits


@pytest.mark.parametrize("m", [1, 2, 20])
@pytest.mark.parametrize("lanes", [0, -64])
@pytest.mark.parametrize("n,r", [(2048, 0), (2048, 4), (3000, 0), (3000, 70)])
def test_adjoint(n, r, lanes, m):
    """||A|| ||A^{-1}|| <= 3.1 (rows and columns of A are dominated by 4 against
    0.05 and 3.2), so residuals of 1e-10 leave x and lambda within 3.1e-10 of
    their norms.  spmv_lanes = -64 is accepted only where A has its copy."""
    from paper_1906_04051_amd import gmres as G
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    s = _system(n, r)
    A = np.zeros((n, n))
    rows = np.repeat(np.arange(n), np.diff(s.rowptr))
    A[rows, s.colind] = s.vals
    gx = np.random.default_rng(r).uniform(-1, 1, n)
    xr, lr = np.linalg.solve(A, s.b), np.linalg.solve(A.T, gx)
    plan, d = G.plan_for(s, m=m, rtol=1e-10, need_adjoint=True, spmv_lanes=lanes)
    for scale in (1.0, 2.0):
        plan.update_values(d["vals"] * scale)
        x, info = plan.solve(d["b"])
        gb, gv, adj = plan.adjoint(x, torch.from_numpy(gx).cuda())
        assert info["status_name"] == adj["status_name"] == "OK"
        assert adj["rel_res_true"] <= 1.01e-10
        nx, nl = np.linalg.norm(xr) / scale, np.linalg.norm(lr) / scale
        assert np.linalg.norm(x.cpu().numpy() - xr / scale) <= 1e-9 * nx
        assert np.linalg.norm(gb.cpu().numpy() - lr / scale) <= 1e-9 * nl
        assert np.abs(gv.cpu().numpy() + (lr[rows] * xr[s.colind]) / scale**2).max() <= 2e-9 * nx * nl
    plan.close()
