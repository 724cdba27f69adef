"""Patterns without entries: the value array then has no element, and nothing may be
copied from it ahead of a solve.  Every method breaks down on the zero matrix."""
import ctypes as C

import numpy as np
import pytest

from paper_2308_08417_amd import batchsolve as bs


@pytest.mark.parametrize("n", [1, 12, 16, 30, 54, 64])
@pytest.mark.parametrize("fmt", [bs.CSR, bs.ELL])
@pytest.mark.parametrize("solver", [bs.CG, bs.BICGSTAB, bs.GMRES])
def test_plan_copies_nothing(n, fmt, solver):
    assert bs.bs_plan(fmt, n, 0, 0, solver)["stage_values"] == 0


@pytest.mark.gpu
@pytest.mark.parametrize("n,team", [(1, 0), (12, 0), (54, 0), (54, 128), (64, 0), (70, 0), (200, 0)])
@pytest.mark.parametrize("solver,precond", [
    (bs.CG, bs.PREC_JACOBI), (bs.BICGSTAB, bs.PREC_JACOBI), (bs.GMRES, bs.PREC_NONE),
    (bs.BICGSTAB, bs.PREC_ILU), (bs.GMRES, bs.PREC_ILU), (bs.TRSV_LOWER, bs.PREC_NONE),
    (bs.TRSV_UPPER, bs.PREC_NONE)])
def test_breaks_down(n, team, solver, precond):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    B = 300
    print(f"n={n} team={team} solver={solver} precond={precond}", flush=True)
    P = bs.Pattern.from_csr(np.zeros(n + 1, np.int32), np.zeros(0, np.int32))
    b = torch.rand((B, n), dtype=torch.float64, device="cuda") + 0.5
    x = torch.full_like(b, 7.0)
    it, st = (torch.full((B,), -1, dtype=torch.int32, device="cuda") for _ in range(2))
    res = torch.empty(B, dtype=torch.float64, device="cuda")
    # a C caller's array of no element: an address, of which nothing may be read
    # (here b's, so that the call is in bounds either way)
    o = bs.make_options(team=team, flags=bs.FLAG_X0_ZERO)
    rc = bs.lib().bs_batch_solve(bs.CSR, B, n, P.handle, b.data_ptr(), b.data_ptr(), x.data_ptr(),
                                 solver, precond, 1e-10, 20, it.data_ptr(), res.data_ptr(),
                                 st.data_ptr(), C.byref(o), None)
    torch.cuda.synchronize()
    assert rc == 0
    assert bool((st == bs.BREAKDOWN).all()) and bool((x == 0).all())
    # ||b - 0|| / ||b||: two sums of n squares, roundings of n + 4 operations each
    assert bool(((res - 1).abs() <= (n + 4) * 2.0 ** -52).all())
