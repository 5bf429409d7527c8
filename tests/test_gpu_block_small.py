"""Small dense kernels of block GMRES (block.hip: Cholesky factor, reflectors,
back substitution) at the edges of their layouts, against the block oracle: one
step a cycle, widths next to 8 and 16, a full 16-entry window, 256 Krylov
vectors (32 strips).  The second cycle starts from the first one's solution.

Both sides build the same block Krylov spaces; the gate is the 1e-8 of the
other trajectory tests."""
import copy

import numpy as np
import pytest

import oracle
from paper_1906_04051_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k,m,steps", [(4, 1, 3), (7, 5, 9), (9, 3, 6), (15, 16, 18), (16, 7, 9), (16, 16, 17)])
def test_block_widths_match_oracle(k, m, steps):
    _check(W.make_config(1, mesh=40), k, m, steps)   # 1,681 unknowns: 17 rows past a multiple of 64


@pytest.mark.parametrize("k", [5, 16])
def test_block_rows_beyond_one_stage(k):
    """Q2 rows (9 to 25 entries): the eight (sixteen) rows of a wavefront hold
    more entries than one stage of the SpMM."""
    _check(W.make_config(3, mesh=20), k, 4, 6)


def _check(s, k, m, steps):
    from paper_1906_04051_amd import gmres as G
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    s = copy.copy(s)
    s.r = 0
    s.z_rowptr = np.zeros(s.n + 1, np.int32)
    s.z_colind = np.zeros(0, np.int32)
    s.z_vals = np.zeros(0)
    B = np.random.default_rng(40 + k).standard_normal((s.n, k))
    ref = oracle.bgmres(s.rowptr, s.colind, s.vals, B, m, 0.0, steps)
    plan, d = G.plan_for(s, m=8, rtol=0.0, max_iters=steps)
    X, info = plan.solve_block(torch.from_numpy(B).cuda(), m)
    X = X.cpu().numpy()
    plan.close()
    r = float(np.linalg.norm(X - ref.x) / np.linalg.norm(ref.x))
    print(k, m, f"{r:.2e}", flush=True)
    assert info["iters"] == ref.iters == steps
    assert r <= 1e-8
