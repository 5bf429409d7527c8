"""Coarse matrix, its factors and inverse (setup.hip) at the sizes where the
kernels change form: one column, one and several entries a lane, the largest
matrix factored in LDS, one past it, the largest at all.

Deflated fixed-count solves against the oracle, which forms E and solves with it
by itself; the gate is the 1e-8 of the other trajectory tests."""
import copy

import numpy as np
import pytest

import oracle
from paper_1906_04051_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("r", [1, 2, 63, 65, 96, 97, 200, 256])
def test_coarse_inverse_matches_oracle(r):
    from paper_1906_04051_amd import gmres as G
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    s = copy.copy(W.make_config(1, mesh=48))      # 2,401 unknowns
    s.r = r
    s.z_rowptr = np.arange(s.n + 1, dtype=np.int32)
    s.z_colind = (np.arange(s.n) * r // s.n).astype(np.int32)
    s.z_vals = np.random.default_rng(r).uniform(0.5, 1.5, s.n)
    ref = oracle.gmres(s, 20, 0.0, 25)
    plan, d = G.plan_for(s, m=20, rtol=0.0, max_iters=25)
    x, info = plan.solve(d["b"])
    plan.update_values(torch.from_numpy(s.vals).cuda())
    y, _ = plan.solve(d["b"])
    x, y = x.cpu().numpy(), y.cpu().numpy()
    plan.close()
    e = float(np.linalg.norm(x - ref.x) / np.linalg.norm(ref.x))
    print(r, f"{e:.2e}", flush=True)
    assert e <= 1e-8 and np.array_equal(x, y)


@pytest.mark.parametrize("r", [2, 40, 120])
def test_singular_coarse_matrix(r):
    """The last two columns of Z are equal: the last pivot is zero."""
    from paper_1906_04051_amd import gmres as G
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    s = copy.copy(W.make_config(1, mesh=24))      # 625 unknowns
    g = np.arange(s.n) * (r - 1) // s.n           # r - 1 row groups, the last one twice
    cnt = np.where(g == r - 2, 2, 1)
    s.r = r
    s.z_rowptr = np.concatenate([[0], np.cumsum(cnt)]).astype(np.int32)
    s.z_colind = np.concatenate([[c] if c < r - 2 else [c, c + 1] for c in g]).astype(np.int32)
    s.z_vals = np.ones(len(s.z_colind))
    with pytest.raises(G.GmresError) as e:
        G.plan_for(s, m=5)
    assert e.value.status == -2
