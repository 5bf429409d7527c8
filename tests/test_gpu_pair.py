"""Two Arnoldi steps per pair of sweeps (k_pair1, k_pair2, k_pair_step) on the
per-phase engine against the oracle: odd and even restart lengths, one and two
steps a cycle, caps in the middle of a pair, every lane split of the sweeps
(restart lengths past 8, 16, 32, 64), no deflation, scaled matrices.

Fixed-count iterates are gated at 1e-8, as the other trajectory tests."""
import copy

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


def _engine(s, **opts):
    from paper_1906_04051_amd import gmres as G
    plan, d = G.plan_for(s, num_blocks=32, **opts)     # the per-phase engine
    x, info = plan.solve(d["b"])
    h = plan.history() if opts.get("record_history") else None
    x = x.cpu().numpy()
    plan.close()
    return x, info, h


@pytest.mark.parametrize("mesh,s,m,steps", [
    (12, 0, 1, 5), (12, 2, 2, 7), (20, 2, 3, 8), (20, 0, 9, 19), (33, 4, 17, 40),
    (40, 4, 24, 47), (40, 2, 33, 66), (48, 4, 50, 75), (48, 0, 66, 131), (60, 8, 96, 150),
])
def test_pairs_match_oracle(mesh, s, m, steps):
    sysm = W.convection_diffusion_lognormal(mesh, (30.0, 10.0), 0.5, s, W.config_seed(2))
    x, info, h = _engine(sysm, m=m, rtol=0.0, max_iters=steps, record_history=1)
    ref = oracle.gmres(sysm, m, 0.0, steps, history=True)
    assert info["iters"] == steps and info["cycles"] == -(-steps // m)
    r = float(np.linalg.norm(x - ref.x) / np.linalg.norm(ref.x))
    print(mesh, s, m, steps, f"{r:.2e}", flush=True)
    assert r <= 1e-8
    assert np.max(np.abs(h - ref.history[:steps])) <= 1e-8 * np.max(ref.history)


@pytest.mark.parametrize("scale", [1e-60, 1e60])
def test_pairs_scaled_matrix(scale):
    """Powers of ||A|| must not leave the range: x scales with 1 / scale."""
    s = W.convection_diffusion_manufactured(24, s=2)
    big = copy.copy(s)
    big.vals = s.vals * scale
    x, info, _ = _engine(big, m=20, rtol=0.0, max_iters=40)
    ref = oracle.gmres(s, 20, 0.0, 40).x
    assert np.linalg.norm(x * scale - ref) <= 1e-8 * np.linalg.norm(ref)


@pytest.mark.parametrize("prec", ["mixed_f32", "mixed_f16"])
def test_pairs_mixed(prec):
    s = W.make_config(1)
    x, info, _ = _engine(s, m=30, rtol=1e-9, max_iters=20000, precision=prec)
    ref = oracle.gmres(s, 30, 1e-11, 20000).x
    assert info["status_name"] == "OK" and info["rel_res_true"] <= 1e-9
    assert np.linalg.norm(x - ref) <= 1e-8 * np.linalg.norm(ref)


def test_pairs_end_inside_a_pair():
    """Exact termination at the first and at the second step of a pair:
    k distinct eigenvalues end after k steps."""
    for k in (1, 2, 3, 4, 5):
        n = 60
        dvals = 1.0 + np.arange(n) % k
        b = np.random.default_rng(k).uniform(0.5, 1.0, n)
        s = W.from_dense(np.diag(dvals), b)
        x, info, _ = _engine(s, m=12, rtol=1e-10, max_iters=100)
        assert info["status_name"] == "OK" and info["iters"] == k
        assert np.max(np.abs(x - b / dvals)) <= 1e-10
