"""The two products of block GMRES (block.hip): entries staged in LDS, and
rows that read their own entries.  Rows longer than a stage holds of a row, a
wavefront whose entries take several stages, very long rows among short ones,
and matrices on both sides of the rule that chooses, against the block oracle
(1e-8 as for the other trajectory tests; the matrices are diagonally dominant,
so few steps are far from amplifying rounding)."""
import numpy as np
import pytest

import oracle
from paper_1906_04051_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _matrix(n, short, every=0, long=0):
    """Rows of `short` entries around the diagonal (cyclic), every `every`-th
    one with up to `long` more, seven columns apart."""
    rng = np.random.default_rng(n + short)
    base = np.arange(-(short // 2), short - short // 2)
    parts = []
    for i in range(n):
        c = (i + base) % n
        if every and i % every == 0:
            c = np.concatenate([c, (i + 7 * np.arange(1, long + 1)) % n])
        parts.append(np.unique(c))
    rp = np.concatenate([[0], np.cumsum([p.size for p in parts])]).astype(np.int32)
    ci = np.concatenate(parts).astype(np.int32)
    rows = np.repeat(np.arange(n), np.diff(rp))
    v = rng.uniform(-1, 1, ci.size)
    v[ci == rows] = 1.5 * np.diff(rp)
    return W.System(n, rp, ci, v, rng.uniform(-1, 1, n), 0, np.zeros(n + 1, np.int32), np.zeros(0, np.int32),
                    np.zeros(0))


# n, entries a row, one row in `every` with `long` more, right-hand sides.
@pytest.mark.parametrize("n,short,every,long,k", [
    (700, 101, 0, 0, 5),         # rows read their own entries: long rows
    (700, 101, 0, 0, 16),
    (700, 700, 0, 0, 3),         # dense
    (3000, 9, 0, 0, 16),         # few entries
    (11200, 9, 0, 0, 16),        # 100,800 entries: staged
    (11100, 9, 0, 0, 16),        # 99,900: not
    (5003, 21, 16, 150, 16),     # staged, 30 entries a row on average, a wavefront's rows in several stages
    (60001, 35, 0, 0, 16),       # staged: every wavefront of eight rows has 280 entries for 256 places
    (59999, 35, 0, 0, 16),       # not
    (40003, 22, 32, 300, 5),     # 8-wide panels, staged, in several stages
    (200003, 35, 0, 0, 5),       # every wavefront of sixteen rows has 560 entries for 512 places
    (3000, 27, 0, 0, 8),         # few entries
])
def test_block_products_match_oracle(n, short, every, long, k):
    from paper_1906_04051_amd import gmres as G
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    s = _matrix(n, short, every, long)
    B = np.random.default_rng(k).standard_normal((n, k))
    X0 = np.random.default_rng(k + 1).standard_normal((n, k))
    plan, _ = G.plan_for(s, m=8, rtol=0.0, max_iters=3)
    X, info = plan.solve_block(torch.from_numpy(B).cuda(), 2, X0=torch.from_numpy(X0).cuda())
    X = X.cpu().numpy()
    plan.close()
    ref = oracle.bgmres(s.rowptr, s.colind, s.vals, B, 2, 0.0, 3, X0=X0)
    r = float(np.linalg.norm(X - ref.x) / np.linalg.norm(ref.x))
    print(n, short, every, k, f"{r:.2e}", flush=True)
    assert info["iters"] == ref.iters == 3
    assert r <= 1e-8
