"""Coarse matrices of a large batch: 1,024 systems of 256 columns, 2^26
entries in all, as many as fill a launch with a wavefront an entry.

Z = I makes E_s = A_s and x = Z E^{-1} Z^T b the solution at no Arnoldi step:
every entry of every E enters the answer.  Rows of diagonal 3.75 to 4.25 and
off-diagonals -1.25 to -0.75 have a condition number of at most 5.4; the gate of
3e-13 is that times 256 roundings of 2.2e-16."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def test_coarse_matrices_of_a_thousand_systems():
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    from paper_1906_04051_amd import gmres as G
    ns, r = 1024, 256
    n = ns * r
    gen = torch.Generator(device="cuda").manual_seed(11)
    row = torch.arange(n, device="cuda")
    cols = torch.stack([row - 1, row, row + 1], 1)
    vals = torch.rand((n, 3), generator=gen, device="cuda", dtype=torch.float64) * 0.5 - 1.25
    vals[:, 1] += 5.0
    keep = (cols >= 0) & (cols // r == row[:, None] // r)
    keep &= cols < n
    rowptr = torch.zeros(n + 1, dtype=torch.int32, device="cuda")
    rowptr[1:] = keep.sum(1).cumsum(0).int()
    zrp = torch.arange(n + 1, device="cuda").int()
    off = np.arange(ns + 1, dtype=np.int64) * r
    plan = G.Plan(rowptr, cols[keep].int().contiguous(), vals[keep].contiguous(), zrp, row.int(),
                  torch.ones(n, dtype=torch.float64, device="cuda"), sys_row_off=off, sys_zcol_off=off,
                  m=2, rtol=1e-10, max_iters=20)
    xt = torch.rand(n, generator=gen, device="cuda", dtype=torch.float64) + 0.5
    gather = torch.where(keep, vals * xt[cols.clamp(0, n - 1)], torch.zeros_like(vals))
    x, infos = plan.solve_batched(gather.sum(1))
    plan.close()
    assert all(i["status_name"] == "OK" and i["iters"] == 0 for i in infos)
    err = float((x - xt).abs().max() / xt.abs().max())
    print(f"{err:.2e}", flush=True)
    assert err <= 3e-13
