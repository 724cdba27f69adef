"""GMRES steps on teams of a wave and more where their blocks and groups of four end: restart
lengths around multiples of four up to the longest, several cycles (the blocks then reach past
the newest vector into those of the cycle before), one wave and several, against the oracle."""
import numpy as np
import pytest

import oracle as O
from paper_2308_08417_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2308_08417_amd import batchsolve as bs  # noqa: E402


@pytest.fixture(scope="module", autouse=True)
def device():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    bs.lib()


@pytest.mark.parametrize("restart", [1, 2, 3, 4, 5, 8, 9, 27, 28, 29, 30])
@pytest.mark.parametrize("nx,ny", [(7, 5), (8, 8), (9, 8), (16, 15), (20, 16), (27, 20)])
def test_restart_lengths(nx, ny, restart):
    print(f"n={nx * ny} restart={restart}", flush=True)
    bt = W.collision_stencil(24, nx=nx, ny=ny, seed=nx * ny)
    P = bs.Pattern.from_csr(bt.row_ptr, bt.col_idx)
    x, it, rs, st = [t.cpu().numpy() for t in bs.solve(
        P, torch.from_numpy(bt.values).cuda(), torch.from_numpy(bt.b).cuda(), solver=bs.GMRES,
        precond=bs.PREC_JACOBI, tol=1e-10, max_iter=3000, opts=bs.make_options(restart=restart))]
    xo, io, ro, so = O.batch_solve(O.Pattern(bt.n, bt.row_ptr, bt.col_idx), bt.values, bt.b,
                                   solver=O.GMRES, precond=O.PREC_JACOBI, tol=1e-10,
                                   max_iter=3000, restart=restart)
    assert np.all(so == O.CONVERGED) and np.array_equal(st, so)
    # modified against blocked Gram-Schmidt: rounding may move a count by a step per cycle
    assert np.all(np.abs(it.astype(int) - io) <= 2 + io // restart)
    assert np.all(rs <= 1e-10)
    # both residuals are below 1e-10 ||b||; the dominant diagonals keep the error near them
    err = np.linalg.norm(x - xo, axis=1) / np.linalg.norm(xo, axis=1)
    assert err.max() <= 1e-7, err.max()
