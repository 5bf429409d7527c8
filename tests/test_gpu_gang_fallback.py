"""Launches that are given up (gang.hip): limits of microseconds,
set from the host, make a wait of the launch give up -- at its first rendezvous
or in the middle of the iteration -- and every kernel ends normally.  The solve
is then repeated on the other kernels from the caller's own data: the result
has the bits of a plan that never launches a gang."""
import threading

import numpy as np
import pytest

from paper_1906_04051_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

AT_START = dict(start_us=0.0, wait_us=0.0)    # the first wait that is not over at once
INSIDE = dict(start_us=1e6, wait_us=0.0)      # a wait after all of the gang is there
NEVER = dict(start_us=-1.0)


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    from paper_1906_04051_amd import gmres as G
    G.load_library()
    yield


def _system(mesh, s):
    return W.convection_diffusion_lognormal(mesh, (20.0, 5.0), 1.0, s, W.config_seed(2))


def _x0(n):
    return torch.from_numpy(np.random.default_rng(5).uniform(-1, 1, n)).cuda()


@pytest.mark.parametrize("limits", [AT_START, INSIDE], ids=["start", "inside"])
@pytest.mark.parametrize("opts", [dict(), dict(adapt_rmax=3), dict(precision="mixed_f32"),
                                  dict(precision="mixed_f16")], ids=["fp64", "adaptive", "f32", "f16"])
@pytest.mark.parametrize("start", ["zero", "x0", "aliased"])
def test_a_solve_given_up_is_repeated(limits, opts, start):
    from paper_1906_04051_amd import gmres as G
    sysm = _system(100, 0 if "adapt_rmax" in opts else 4)
    kw = dict(m=20, rtol=1e-9 if "precision" in opts else 0.0, max_iters=20000 if "precision" in opts else 50)
    out = []
    for lim in (limits, NEVER):
        plan, d = G.plan_for(sysm, **kw, **opts)
        plan.set_gang_wait(**lim)
        x0 = None if start == "zero" else _x0(sysm.n)
        x, info = plan.solve(d["b"], x0=x0, out=x0 if start == "aliased" else None)
        if start == "x0":
            assert torch.equal(x0, _x0(sysm.n))
        out.append((x, info["iters"], info["cycles"], info["rho0"], info["defl_r"]))
        counts = plan.gang_counts()
        assert counts["gang"] == 0 and (counts["given_up"] > 0) == (lim is limits) and counts["other"] > 0
        plan.close()
    assert out[0][1:] == out[1][1:]
    assert torch.equal(out[0][0], out[1][0])


@pytest.mark.parametrize("limits", [AT_START, INSIDE], ids=["start", "inside"])
def test_an_adjoint_given_up_is_repeated(limits):
    from paper_1906_04051_amd import gmres as G
    sysm = _system(64, 4)
    out = []
    for lim in (limits, NEVER):
        plan, d = G.plan_for(sysm, need_adjoint=True, m=20, rtol=0.0, max_iters=50)
        plan.set_gang_wait(**lim)
        out.append(plan.adjoint(_x0(sysm.n), d["b"])[:2])
        assert plan.gang_counts() == dict(gang=0, given_up=1 if lim is limits else 0, other=1)
        plan.close()
    assert all(torch.equal(a, b) for a, b in zip(*out))


@pytest.mark.parametrize("limits", [AT_START, INSIDE], ids=["start", "inside"])
@pytest.mark.parametrize("aliased", [False, True])
def test_a_batch_given_up_is_repeated(limits, aliased):
    from paper_1906_04051_amd import gmres as G
    batch = W.make_batch(12, 40, 96, 4)
    x0 = _x0(batch.b.size)
    out = []
    for lim in (limits, NEVER):
        plan, d = G.plan_for(batch, m=20, rtol=0.0, max_iters=45)
        plan.set_gang_wait(**lim)
        x = x0.clone()
        y, infos = plan.solve_batched(d["b"], x0=x, out=x if aliased else None)
        assert all(i["iters"] == 45 for i in infos)
        assert plan.gang_counts() == dict(gang=0, given_up=1 if lim is limits else 0, other=1)
        out.append(y)
        plan.close()
    assert torch.equal(out[0], out[1])


def test_launches_are_left_out_after_one_was_given_up():
    """1, 2, 4 solves on the other kernels after launches given up in a row;
    the first launch that runs to its end starts over."""
    from paper_1906_04051_amd import gmres as G
    plan, d = G.plan_for(_system(64, 4), m=20, rtol=0.0, max_iters=25)
    plan.set_gang_wait(**AT_START)
    seen = []
    for _ in range(11):
        before = plan.gang_counts()["given_up"]
        plan.solve(d["b"])
        seen.append(plan.gang_counts()["given_up"] - before)
    assert seen == [1, 0, 1, 0, 0, 1, 0, 0, 0, 0, 1]
    plan.set_gang_wait()
    plan.solve(d["b"])
    plan.solve(d["b"])
    assert plan.gang_counts()["gang"] == 2
    plan.close()


def test_limits_are_checked():
    from paper_1906_04051_amd import gmres as G
    plan, _ = G.plan_for(_system(16, 0), m=5)
    for bad in (dict(start_us=2e9), dict(wait_us=-1.0), dict(wait_us=2e9), dict(start_us=float("nan")),
                dict(wait_us=float("nan"))):
        with pytest.raises(G.GmresError):
            plan.set_gang_wait(**bad)
    plan.close()


def test_solves_of_several_threads():
    """Plans of different sizes and restart lengths, each on its own stream
    and thread: whatever the kernels, the solutions of solves alone, within the
    rounding of 40 steps (the 1e-8 of the other trajectory tests)."""
    from paper_1906_04051_amd import gmres as G
    jobs = []
    for mesh, s, m in ((40, 2, 10), (100, 4, 40), (256, 8, 20), (200, 0, 30)):
        st = torch.cuda.Stream()
        with torch.cuda.stream(st):
            plan, d = G.plan_for(_system(mesh, s), m=m, rtol=0.0, max_iters=40, stream=st)
            jobs.append([st, plan, d, plan.solve(d["b"])[0].clone(), None])
    torch.cuda.synchronize()

    def work(j):
        with torch.cuda.stream(j[0]):
            try:
                j[4] = [j[1].solve(j[2]["b"])[0].clone() for _ in range(10)]
            except Exception as e:   # seen by the assertion below
                j[4] = e

    ts = [threading.Thread(target=work, args=(j,)) for j in jobs]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    torch.cuda.synchronize()
    for _, plan, _, ref, got in jobs:
        assert isinstance(got, list), got
        print(plan.n, plan.gang_counts(), flush=True)
        for x in got:
            assert float((x - ref).norm() / ref.norm()) <= 1e-8
        plan.close()


def test_solves_beside_a_chip_filling_batch():
    """A batch with a workgroup per system on another stream and thread holds
    the compute units: the solves beside it give the solutions of solves
    alone, on whichever kernels (gate as above)."""
    from paper_1906_04051_amd import gmres as G
    batch = W.make_batch(300, 60, 100, 4)
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        bplan, bd = G.plan_for(batch, m=30, rtol=1e-8, max_iters=5000, batch_wg=512, stream=st)
    plan, d = G.plan_for(_system(100, 4), m=20, rtol=0.0, max_iters=40)
    ref = plan.solve(d["b"])[0].clone()
    done = []

    def work():
        with torch.cuda.stream(st):
            done.append(bplan.solve_batched(bd["b"])[1])

    t = threading.Thread(target=work)
    t.start()
    for _ in range(20):
        x, _ = plan.solve(d["b"])
        assert float((x - ref).norm() / ref.norm()) <= 1e-8
    t.join()
    print(plan.gang_counts(), flush=True)
    assert done and all(i["status_name"] == "OK" for i in done[0])
    plan.close()
    bplan.close()


@pytest.mark.parametrize("limits", [dict(), AT_START, INSIDE, NEVER], ids=["gang", "start", "inside", "engine"])
@pytest.mark.parametrize("shift", [-700, 700])
def test_x_may_reach_into_b(limits, shift):
    """x and b are ranges of one buffer (they may not start together): the
    solution is that of separate buffers, and nothing of the right-hand side is
    written before the iteration has read it for the last time."""
    from paper_1906_04051_amd import gmres as G
    sysm = _system(100, 4)
    plan, d = G.plan_for(sysm, m=20, rtol=0.0, max_iters=50)
    plan.set_gang_wait(**limits)
    ref, _ = plan.solve(d["b"])
    plan.set_gang_wait(**limits)
    buf = torch.zeros(sysm.n + 1400, dtype=torch.float64, device="cuda")
    buf[700:700 + sysm.n] = d["b"]
    x = buf[700 + shift:700 + shift + sysm.n]
    plan.solve(buf[700:700 + sysm.n], out=x)
    assert torch.equal(x, ref)
    plan.close()


def test_gangs_that_do_not_fit_together_wait_for_each_other():
    """Five threads whose gangs take 207 or 256 compute units each, with
    places for one, and a batch: nobody's workgroups wait on the chip in vain
    (a second is enough for all that is in front of a thread)."""
    from paper_1906_04051_amd import gmres as G
    jobs = []
    for mesh, s, m in ((256, 8, 20), (256, 0, 30), (300, 4, 20), (400, 2, 20)):
        st = torch.cuda.Stream()
        with torch.cuda.stream(st):
            plan, d = G.plan_for(_system(mesh, s), m=m, rtol=0.0, max_iters=40, stream=st)
        jobs.append([st, plan, d, lambda plan=plan, d=d: plan.solve(d["b"])[0]])
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        plan, d = G.plan_for(W.make_batch(40, 16, 96, 4), m=20, rtol=0.0, max_iters=40, stream=st)
    jobs.append([st, plan, d, lambda plan=plan, d=d: plan.solve_batched(d["b"])[0]])
    torch.cuda.synchronize()
    refs, got = [], [None] * len(jobs)
    for j in jobs:
        j[1].set_gang_wait(start_us=1e6)
        with torch.cuda.stream(j[0]):
            refs.append(j[3]().clone())

    def work(i):
        with torch.cuda.stream(jobs[i][0]):
            try:
                got[i] = [jobs[i][3]().clone() for _ in range(12)]
            except Exception as e:   # seen by the assertion below
                got[i] = e

    ts = [threading.Thread(target=work, args=(i,)) for i in range(len(jobs))]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    torch.cuda.synchronize()
    for j, ref, g in zip(jobs, refs, got):
        assert isinstance(g, list), g
        assert j[1].gang_counts() == dict(gang=13, given_up=0, other=0)
        assert all(torch.equal(x, ref) for x in g)
        j[1].close()
