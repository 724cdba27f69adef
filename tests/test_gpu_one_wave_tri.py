"""One-wave ILU(0) and BatchTrsv (systems of up to 64 rows) where their kernels
can go wrong: sizes around the sweeps' groups of eight columns, batches of
several systems per wave (the values of the next one travel in registers), blocks
that start at odd multiples of 8 bytes, and quotients outside the range the
reciprocal form covers."""
import numpy as np
import pytest

import oracle as O
from paper_2308_08417_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2308_08417_amd import batchsolve as bs  # noqa: E402

SOLVER_O = {bs.BICGSTAB: O.BICGSTAB, bs.GMRES: O.GMRES, bs.TRSV_LOWER: O.TRSV_LOWER,
            bs.TRSV_UPPER: O.TRSV_UPPER}
N_BATCH = 5000  # more than the 2048 waves of the widest grid can hold at once


@pytest.fixture(scope="module", autouse=True)
def device():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    bs.lib()


def solve(bt, fmt, solver, scale=1.0):
    P = bs.Pattern.from_csr(bt.row_ptr, bt.col_idx)
    vals = torch.from_numpy(bt.values * scale).cuda()
    if fmt == bs.ELL:
        ell = torch.empty((bt.n_batch, P.ell_width * bt.n), dtype=torch.float64, device="cuda")
        bs.bs_values_csr_to_ell(P.handle, vals, ell)
        vals = ell
    prec = bs.PREC_ILU if solver in (bs.BICGSTAB, bs.GMRES) else bs.PREC_NONE
    out = bs.solve(P, vals, torch.from_numpy(bt.b * scale).cuda(), fmt=fmt, solver=solver,
                   precond=prec, tol=1e-10, max_iter=200)
    torch.cuda.synchronize()
    return [t.cpu().numpy() for t in out]


@pytest.mark.parametrize("n,fill", [(1, 1.0), (2, 0.5), (7, 0.4), (8, 0.4), (9, 0.4), (17, 0.3),
                                    (33, 0.35), (54, 0.35), (57, 0.1), (63, 0.3), (64, 0.35),
                                    (64, 0.45), (40, 1.0)])
@pytest.mark.parametrize("solver", [bs.BICGSTAB, bs.GMRES, bs.TRSV_LOWER, bs.TRSV_UPPER])
def test_sizes(n, fill, solver):
    print(f"n={n} fill={fill} solver={solver}", flush=True)
    bt = W.chem_jacobian(n_batch=N_BATCH, n=n, fill=fill, gamma=1e-4, seed=n)
    OP = O.Pattern(bt.n, bt.row_ptr, bt.col_idx)
    prec = O.PREC_ILU if solver in (bs.BICGSTAB, bs.GMRES) else O.PREC_NONE
    xo, io, _, so = O.batch_solve(OP, bt.values, bt.b, solver=SOLVER_O[solver], precond=prec,
                                  tol=1e-10, max_iter=200)
    for fmt in (bs.CSR, bs.ELL):
        x, it, _, st = solve(bt, fmt, solver)
        assert np.array_equal(st, so)
        assert np.all(np.abs(it.astype(int) - io) <= 2)
        err = np.linalg.norm(x - xo, axis=1) / np.linalg.norm(xo, axis=1)
        assert err.max() <= 1e-8, err.max()


@pytest.mark.parametrize("solver", [bs.BICGSTAB, bs.GMRES])
def test_quotients_out_of_range(solver):
    """Scaling the matrix and b by 2^-430 scales every pivot and residual by it, exactly,
    and leaves x as it is; the pivots are then outside the reciprocal form's range and the
    sweeps divide.  Both forms round correctly, so x has to keep its bits."""
    bt = W.chem_jacobian(n_batch=300, n=54, gamma=1e-4, seed=3)
    x, it, _, st = solve(bt, bs.CSR, solver)
    xs, its, _, sts = solve(bt, bs.CSR, solver, scale=2.0 ** -430)
    assert np.all(st == bs.CONVERGED) and np.array_equal(st, sts)
    assert np.array_equal(it, its)
    assert np.array_equal(x, xs)
