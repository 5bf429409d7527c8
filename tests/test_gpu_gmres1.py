"""GMRES(1), and GMRES(3) with a deflation basis, on the per-phase engine: a
cycle makes as many products with A as it has steps (the restart's residual is
not counted) -- not one more for the second half of a pair -- in every
precision; other restart lengths take pairs."""
import numpy as np
import pytest

import oracle
from paper_1906_04051_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _system(n, r):
    """Tridiagonal, diagonally dominant; r indicator columns."""
    rng = np.random.default_rng(n)
    i = np.arange(n)
    c = i[:, None] + np.array([-1, 0, 1])[None, :]
    keep = (c >= 0) & (c < n)
    rp = np.concatenate([[0], np.cumsum(keep.sum(1))]).astype(np.int32)
    ci = c[keep].astype(np.int32)
    v = rng.uniform(-1, 1, ci.size)
    v[ci == np.repeat(i, np.diff(rp))] = 3.0
    zrp = np.arange(n + 1, dtype=np.int32) if r else np.zeros(n + 1, np.int32)
    zci = (i * r // n).astype(np.int32) if r else np.zeros(0, np.int32)
    return W.System(n, rp, ci, v, rng.uniform(-1, 1, n), r, zrp, zci, np.ones(zci.size))


@pytest.mark.parametrize("prec", ["fp64", "mixed_f32", "mixed_f16"])
@pytest.mark.parametrize("r", [0, 4])
@pytest.mark.parametrize("m", [1, 2, 3])
def test_products_of_a_cycle(prec, r, m):
    """Reduction by at least 0.9 a step (rows of 3 against at most 2), so the
    mixed solves end; ||A^{-1}|| ||b|| / ||x|| is at most 5, which leaves both
    solutions within 1e-8 at residuals of 1e-10."""
    from paper_1906_04051_amd import gmres as G
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    s = _system(3001, r)
    if prec == "fp64":
        kw, ref = dict(rtol=0.0, max_iters=6), oracle.gmres(s, m, 0.0, 6).x
    else:
        kw, ref = dict(rtol=1e-10, precision=prec), oracle.gmres(s, m, 1e-12, 20000).x
    plan, d = G.plan_for(s, m=m, num_blocks=32, **kw)
    plan.set_timing(1)
    x, info = plan.solve(d["b"])
    t = plan.kernel_times()
    plan.close()
    if prec == "fp64":
        assert info["iters"] == 6
    else:
        assert info["rel_res_true"] <= 1e-10
    single = m == 1 or (m == 3 and r > 0)
    if single:
        assert t["spmv"]["launches"] == info["iters"]
    elif prec == "fp64":   # mixed: a cycle may end in the middle of a pair
        assert t["spmv"]["launches"] == (6 if m == 2 else 8)
        pairs = 3 if m == 2 else 4
        assert t["pass1"]["launches"] + t["pass1_lag"]["launches"] == t["pass2"]["launches"] == pairs
    x = x.cpu().numpy()
    assert np.linalg.norm(x - ref) <= 1e-8 * np.linalg.norm(ref)
