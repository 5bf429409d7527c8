"""The Ritz step of adaptive deflation (adapt.hip, k_ritz) against the oracle's
dense one at the sizes where the kernel changes form: a 1 x 1 and a 2 x 2
Hessenberg matrix, one row a lane (64), the first second row (65), the largest
restart length (96).

Every cycle starts from a residual above 1e-2 of the first one, so its start
vector carries at most about 1e-13 of rounding; the gate on the iterate and on
|mu| is the 1e-8 of the other trajectory tests."""
import numpy as np
import pytest

import oracle
from paper_1906_04051_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,steps,rmax", [(1, 5, 3), (2, 9, 3), (64, 140, 5), (65, 140, 5), (96, 200, 2)])
def test_ritz_step_matches_oracle(m, steps, rmax):
    from paper_1906_04051_amd import gmres as G
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    s = W.convection_diffusion_manufactured(128, beta=(20.0, 5.0), s=0)
    ref = oracle.dgmres(s, m, 0.0, steps, rmax=rmax)
    plan, d = G.plan_for(s, m=m, rtol=0.0, max_iters=steps, adapt_rmax=rmax)
    x, info = plan.solve(d["b"])
    x = x.cpu().numpy()
    plan.close()
    r = float(np.linalg.norm(x - ref.x) / np.linalg.norm(ref.x))
    print(m, f"{r:.2e}", info["mu"], ref.mu, flush=True)
    assert info["iters"] == steps and info["defl_r"] == ref.r
    assert abs(info["mu"] - ref.mu) <= 1e-8 * ref.mu
    assert r <= 1e-8
