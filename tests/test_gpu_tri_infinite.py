"""Triangular solves whose matrix holds an infinite diagonal entry: that row's x is
b / inf = 0 and every other row's is what the rest of the triangle gives, whatever
the sweep reads beside its own row."""
import numpy as np
import pytest

from paper_2308_08417_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2308_08417_amd import batchsolve as bs  # noqa: E402


@pytest.fixture(scope="module", autouse=True)
def device():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    bs.lib()


def substitution(bt, lower):
    """Row by row in FP64; an infinite diagonal divides to zero."""
    rows = np.repeat(np.arange(bt.n), np.diff(bt.row_ptr))
    a = np.zeros((bt.n_batch, bt.n, bt.n))
    a[:, rows, bt.col_idx] = bt.values
    x = np.zeros((bt.n_batch, bt.n))
    for i in range(bt.n) if lower else range(bt.n - 1, -1, -1):
        j = np.arange(i) if lower else np.arange(i + 1, bt.n)
        x[:, i] = (bt.b[:, i] - (a[:, i, j] * x[:, j]).sum(1)) / a[:, i, i]
    return x


# sizes on both sides of a multiple of eight; 128: the form of several waves
@pytest.mark.parametrize("n,team", [(2, 0), (7, 0), (9, 0), (16, 0), (33, 0), (54, 0), (63, 0), (64, 0),
                                    (54, 128), (130, 0)])
@pytest.mark.parametrize("solver", [bs.TRSV_LOWER, bs.TRSV_UPPER])
def test_infinite_diagonal(n, team, solver):
    bt = W.chem_jacobian(n_batch=6 * n, n=n, fill=0.3, gamma=1e-6, seed=n)
    rows = np.repeat(np.arange(n), np.diff(bt.row_ptr))
    diag = np.flatnonzero(rows == bt.col_idx)
    s = np.arange(bt.n_batch)
    bt.values[s, diag[s % n]] = np.inf
    xo = substitution(bt, solver == bs.TRSV_LOWER)
    P = bs.Pattern.from_csr(bt.row_ptr, bt.col_idx)
    csr = torch.from_numpy(bt.values).cuda()
    ell = torch.empty((bt.n_batch, P.ell_width * n), dtype=torch.float64, device="cuda")
    bs.bs_values_csr_to_ell(P.handle, csr, ell)
    for fmt, vals in ((bs.CSR, csr), (bs.ELL, ell)):
        x, _, _, st = bs.solve(P, vals, torch.from_numpy(bt.b).cuda(), fmt=fmt, solver=solver,
                               precond=bs.PREC_NONE, opts=bs.make_options(team=team))
        x, st = x.cpu().numpy(), st.cpu().numpy()
        assert np.all(st == bs.CONVERGED)
        # well-conditioned rows: a few roundings per entry
        assert np.abs(x - xo).max() <= 1e-12 * np.abs(xo).max()
