"""ILU(0) and BatchTrsv on teams of more than one wave where their schedules can
go wrong: one lane or a whole wave without rows, rows of more terms than a
record holds, levels of more rows than a wave, factors beyond 15-bit byte
offsets, a row without a stored diagonal, and quotients outside the range the
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
ITERATIVE = (bs.BICGSTAB, bs.GMRES)


@pytest.fixture(scope="module", autouse=True)
def device():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    bs.lib()


def solve(bt, fmt, solver, team=0, scale=1.0, prec=bs.PREC_ILU, max_iter=200):
    P = bs.Pattern.from_csr(bt.row_ptr, bt.col_idx)
    vals = torch.from_numpy(bt.values * scale).cuda()
    if fmt == bs.ELL:
        ell = torch.empty((bt.n_batch, P.ell_width * bt.n), dtype=torch.float64, device="cuda")
        bs.bs_values_csr_to_ell(P.handle, vals, ell)
        vals = ell
    out = bs.solve(P, vals, torch.from_numpy(bt.b * scale).cuda(), fmt=fmt, solver=solver,
                   precond=prec if solver in ITERATIVE else bs.PREC_NONE, tol=1e-10,
                   max_iter=max_iter, opts=bs.make_options(team=team))
    torch.cuda.synchronize()
    return [t.cpu().numpy() for t in out]


def without_diagonal(bt, r):
    """The batch with row r's diagonal entry taken out of the pattern."""
    rows = np.repeat(np.arange(bt.n), np.diff(bt.row_ptr))
    keep = ~((rows == r) & (bt.col_idx == r))
    rp = bt.row_ptr.copy()
    rp[r + 1:] -= 1
    return W.Batch(bt.name, bt.n, rp, bt.col_idx[keep], np.ascontiguousarray(bt.values[:, keep]),
                   bt.b, np.zeros_like(bt.b))


@pytest.mark.parametrize("n,fill,team", [(1, 1.0, 128), (5, 0.6, 128), (54, 0.35, 128),
                                         (64, 0.4, 256), (65, 0.4, 0), (128, 0.3, 0),
                                         (129, 0.01, 0), (250, 0.12, 0), (257, 0.004, 0),
                                         (500, 0.02, 0), (513, 0.002, 0), (1024, 0.004, 0)])
@pytest.mark.parametrize("solver", [bs.BICGSTAB, bs.GMRES, bs.TRSV_LOWER, bs.TRSV_UPPER])
def test_sizes(n, fill, team, solver):
    if solver == bs.GMRES and n > 512:
        pytest.skip("GMRES with ILU(0) takes up to 512 rows")
    print(f"n={n} fill={fill} team={team} solver={solver}", flush=True)
    bt = W.chem_jacobian(n_batch=40, n=n, fill=fill, gamma=1e-4, seed=n)
    OP = O.Pattern(bt.n, bt.row_ptr, bt.col_idx)
    prec = O.PREC_ILU if solver in ITERATIVE else O.PREC_NONE
    xo, io, _, so = O.batch_solve(OP, bt.values, bt.b, solver=SOLVER_O[solver], precond=prec,
                                  tol=1e-10, max_iter=200)
    for fmt in (bs.CSR, bs.ELL):
        x, it, _, st = solve(bt, fmt, solver, team)
        assert np.array_equal(st, so)
        assert np.all(np.abs(it.astype(int) - io) <= 2)
        err = np.linalg.norm(x - xo, axis=1) / np.linalg.norm(xo, axis=1)
        assert err.max() <= 1e-8, err.max()


@pytest.mark.parametrize("n", [54, 250])
@pytest.mark.parametrize("solver", [bs.BICGSTAB, bs.GMRES, bs.TRSV_LOWER, bs.TRSV_UPPER])
def test_quotients_out_of_range(n, solver):
    """Scaling the matrix and b by 2^-430 scales every pivot and residual by it, exactly,
    and leaves x as it is; the pivots are then outside the reciprocal form's range and the
    sweeps divide.  Both forms round correctly, so x has to keep its bits."""
    bt = W.chem_jacobian(n_batch=40, n=n, fill=0.1, gamma=1e-4, seed=3)
    x, it, _, st = solve(bt, bs.CSR, solver, 128 if n == 54 else 0)
    xs, its, _, sts = solve(bt, bs.CSR, solver, 128 if n == 54 else 0, scale=2.0 ** -430)
    assert np.all(st == bs.CONVERGED) and np.array_equal(st, sts)
    assert np.array_equal(it, its)
    assert np.array_equal(x, xs)


@pytest.mark.parametrize("r", [0, 70, 191])
def test_row_without_diagonal(r):
    """Its pivot is zero: M is the identity, bit for bit the unpreconditioned solve, and a
    triangular solve breaks down."""
    bt = without_diagonal(W.collision_stencil(12, nx=16, ny=12, seed=50), r)
    for fmt in (bs.CSR, bs.ELL):
        for solver in ITERATIVE:
            g = solve(bt, fmt, solver, max_iter=20)
            h = solve(bt, fmt, solver, prec=bs.PREC_NONE, max_iter=20)
            for u, v in zip(g, h):
                assert np.array_equal(u, v, equal_nan=True)
        for solver in (bs.TRSV_LOWER, bs.TRSV_UPPER):
            x, _, _, st = solve(bt, fmt, solver)
            assert np.all(st == bs.BREAKDOWN) and np.all(x == 0)


@pytest.mark.parametrize("n", [1, 2, 3, 5])
def test_after_a_zero_pivot(n):
    """Forced teams of the smallest systems, many per workgroup: a system whose pivots vanish
    (infinite quotients) leaves nothing behind that the next ones of its workgroup read; they
    give what they give alone."""
    bt = W.chem_jacobian(n_batch=9000, n=n, fill=1.0, gamma=1e-4, seed=n)
    bt.values[::3, 0] = 0.0
    for solver in ITERATIVE:
        x, it, _, st = solve(bt, bs.CSR, solver, 128, max_iter=20)
        keep = np.flatnonzero(np.arange(9000) % 3 != 0)
        ok = W.Batch(bt.name, n, bt.row_ptr, bt.col_idx, np.ascontiguousarray(bt.values[keep]),
                     np.ascontiguousarray(bt.b[keep]), np.zeros((keep.size, n)))
        xo, ito, _, sto = solve(ok, bs.CSR, solver, 128, max_iter=20)
        assert np.all(sto == bs.CONVERGED)
        assert np.array_equal(st[keep], sto) and np.array_equal(it[keep], ito)
        assert np.array_equal(x[keep], xo)
