"""BiCGSTAB on 512 lanes x 2 rows takes another kernel when a launch has more tasks than the
device has compute units.  On both sides of that line a system keeps its bits."""
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


def run(vb, B, walk):
    h = bs.VarBatch(vb.pat_rows, vb.pat_rowptr_off, vb.rowptr_all, vb.pat_col_off, vb.col_all, vb.pat_id[:B])
    bs.bs_varbatch_set_plan(h.handle, [1 + 3 * walk] * 5)
    b = torch.from_numpy(vb.b[:vb.row_off[B]]).cuda()
    x = torch.empty_like(b)
    it = torch.empty(B, dtype=torch.int32, device="cuda")
    rs = torch.empty(B, dtype=torch.float64, device="cuda")
    st = torch.empty(B, dtype=torch.int32, device="cuda")
    bs.bs_varbatch_solve(h.handle, torch.from_numpy(vb.values[:vb.val_off[B]]).cuda(), b, x, bs.BICGSTAB,
                         bs.PREC_JACOBI, 1e-10, 60, it, rs, st, bs.make_options(flags=bs.FLAG_X0_ZERO))
    torch.cuda.synchronize()
    return [t.cpu().numpy() for t in (x, it, rs, st)]


@pytest.mark.parametrize("width", [3, 9, 10])  # 8 and 10 slots
@pytest.mark.parametrize("walk", [0, 1])
@pytest.mark.parametrize("n_min,n_max,teams", [(65, 128, 8), (257, 512, 2), (513, 1024, 1)])
def test_both_sides_of_the_line(width, walk, n_min, n_max, teams):
    print(f"width={width} walk={walk} n={n_min}..{n_max}", flush=True)
    few = torch.cuda.get_device_properties(0).multi_processor_count * teams
    vb = W.uneven_banded(n_batch=few + 1, n_min=n_min, n_max=n_max, w_min=width, w_max=width, seed=width)
    a, b = run(vb, few, walk), run(vb, few + 1, walk)
    assert np.array_equal(a[0], b[0][:a[0].size])
    for u, v in zip(a[1:], b[1:]):
        assert np.array_equal(u, v[:few])
    assert np.all(b[3] == bs.CONVERGED)
