"""Triangular sweeps of several waves whose pivots lie in the reciprocal form's range and
whose results do not: the sweep is run a second time, with divisions, on the same
right-hand side.  Scaling b alone by a power of two scales every vector by it, exactly."""
import numpy as np
import pytest

from paper_2308_08417_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2308_08417_amd import batchsolve as bs  # noqa: E402

ITERATIVE = (bs.BICGSTAB, bs.GMRES)


@pytest.fixture(scope="module", autouse=True)
def device():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    bs.lib()


# 2^-430: below the results' range of 2^-400, products of two still normal numbers
@pytest.mark.parametrize("n,team", [(54, 128), (250, 0)])
@pytest.mark.parametrize("solver", [bs.BICGSTAB, bs.GMRES, bs.TRSV_LOWER, bs.TRSV_UPPER])
@pytest.mark.parametrize("exponent", [-430, 430])
def test_results_out_of_range(n, team, solver, exponent):
    bt = W.chem_jacobian(n_batch=40, n=n, fill=0.1, gamma=1e-4, seed=5)
    P = bs.Pattern.from_csr(bt.row_ptr, bt.col_idx)
    vals, b = torch.from_numpy(bt.values).cuda(), torch.from_numpy(bt.b).cuda()
    prec = bs.PREC_ILU if solver in ITERATIVE else bs.PREC_NONE
    (x, it, rs, st), (xs, its, rss, sts) = (
        [t.cpu().numpy() for t in bs.solve(P, vals, v, solver=solver, precond=prec, tol=1e-10, max_iter=200,
                                           opts=bs.make_options(team=team))]
        for v in (b, b * 2.0 ** exponent))
    assert np.all(st == bs.CONVERGED) and np.array_equal(st, sts)
    assert np.array_equal(it, its) and np.array_equal(rs, rss)
    assert np.array_equal(x * 2.0 ** exponent, xs)
