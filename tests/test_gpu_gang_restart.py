"""Restarts of deflated gang solves (gang.hip): the projected residual of a
restart and the coarse solve behind it share LDS.  Cycles of two to four steps
make restarts as frequent as steps.

Every sum of a gang is formed in a fixed order, so a repeated solve gives the
same bits, whatever the timing of its wavefronts and workgroups; against the
oracle the gate is the 1e-8 of the other trajectory tests (well-conditioned
systems: the iterates differ by rounding over at most 240 steps;
the oracle itself moves by 3e-14 when its right-hand side is rounded anew)."""
import numpy as np
import pytest

import oracle
from paper_1906_04051_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

REPEATS = 6


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    from paper_1906_04051_amd import gmres as G
    G.load_library()
    yield


# mesh, s, m, steps: columns touched by few workgroups (s large) leave most
# wavefronts of the coarse solve without members to wait for.
@pytest.mark.parametrize("mesh,s,m,steps", [
    (16, 2, 2, 240),      # two workgroups
    (64, 4, 2, 240),      # 17 workgroups, 16 columns (four member rows a load)
    (64, 5, 3, 240),      # 25 columns (two)
    (100, 8, 4, 200),     # 64 columns (one)
    (100, 16, 2, 120),    # 256 columns: four rounds of Z^T sums
])
def test_restarts_repeat_bit_for_bit(mesh, s, m, steps):
    from paper_1906_04051_amd import gmres as G
    sysm = W.convection_diffusion_manufactured(mesh, s=s)
    plan, d = G.plan_for(sysm, m=m, rtol=0.0, max_iters=steps)
    first = None
    for _ in range(REPEATS):
        x, info = plan.solve(d["b"])
        assert info["iters"] == steps and info["cycles"] == -(-steps // m)
        if first is None:
            first = x.clone()
        assert torch.equal(x, first)
    plan.close()
    ref = oracle.gmres(sysm, m, 0.0, steps).x
    r = float(np.linalg.norm(first.cpu().numpy() - ref) / np.linalg.norm(ref))
    print(mesh, s, m, f"{r:.2e}", flush=True)
    assert r <= 1e-8


# Meshes of 16 to 96 elements: gangs of one to 19 workgroups, and several
# systems a gang, so which gang takes the last ones depends on the others.
@pytest.mark.parametrize("ns,lo,hi,m,steps", [(24, 96, 96, 3, 60), (64, 16, 96, 3, 60), (48, 16, 128, 20, 25)])
def test_batches_repeat_bit_for_bit(ns, lo, hi, m, steps):
    from paper_1906_04051_amd import gmres as G
    batch = W.make_batch(ns, lo, hi, 4)
    plan, d = G.plan_for(batch, m=m, rtol=0.0, max_iters=steps)
    first = None
    for _ in range(REPEATS):
        x, infos = plan.solve_batched(d["b"])
        assert all(i["iters"] == steps for i in infos)
        if first is None:
            first = x.clone()
        assert torch.equal(x, first)
    assert plan.gang_counts() == dict(gang=REPEATS, given_up=0, other=0)
    plan.close()
    for i, sysm in enumerate(batch.systems):
        ref = oracle.gmres(sysm, m, 0.0, steps).x
        r = float(np.linalg.norm(first[batch.row_off[i]:batch.row_off[i + 1]].cpu().numpy() - ref)
                  / np.linalg.norm(ref))
        assert r <= 1e-8, (i, r)


def test_a_batch_to_tolerance_repeats_bit_for_bit():
    """Systems that take different numbers of steps, beside a second batch on
    another stream that changes when gangs become free."""
    from paper_1906_04051_amd import gmres as G
    batch = W.make_batch(64, 16, 96, 4)
    plan, d = G.plan_for(batch, m=30, rtol=1e-10, max_iters=20000)
    first = plan.solve_batched(d["b"])[0].clone()
    noise = torch.rand(1 << 24, device="cuda")
    side = torch.cuda.Stream()
    for i in range(REPEATS):
        with torch.cuda.stream(side):
            for _ in range(3 * i):
                noise = noise * 1.0000001
        x, infos = plan.solve_batched(d["b"])
        assert torch.equal(x, first)
    torch.cuda.synchronize()
    plan.close()
