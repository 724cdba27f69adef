"""The learned start's kernels at every tile size (64, 32 or 16 samples, chosen by
the number of samples) and at ragged ends.  A sample's outputs do not depend on
the tile it falls into, so a batch must repeat, bit for bit, what a call on its
first samples alone gives."""
import numpy as np
import pytest

from paper_2308_08417_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2308_08417_amd import batchsolve as bs  # noqa: E402

H = 256
# FP32 sums of at most 512 + 64 terms (a chunk of samples, then the chunks): 2^-24 * 576 of
# the sum of their magnitudes, which exceeds the sum of M terms of either sign by about
# sqrt(M) <= 128
TOL = 2.0 ** -24 * 576 * 128


@pytest.fixture(scope="module", autouse=True)
def device():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    bs.lib()


def model(n, M, seed):
    bt = W.chem_jacobian(n_batch=M, n=n, seed=seed)
    m = bs.WarmStartModel(n, bt.row_ptr, bt.col_idx)
    p = W.mlp_init(n, seed=seed)
    rng = np.random.default_rng(seed)
    for at, k in ((3 * n * H, H), (3 * n * H + H + H * H, H), (p.size - n, n)):
        p[at:at + k] = 0.1 * rng.standard_normal(k)
    bs.bs_ws_set_params(m.handle, p)
    values, b = torch.from_numpy(bt.values).cuda(), torch.from_numpy(bt.b).cuda()
    x_prev = b * (1 + 0.01 * torch.rand_like(b))
    feat = torch.empty((M, 3 * n), dtype=torch.float32, device="cuda")
    delta = torch.empty((M, n), dtype=torch.float32, device="cuda")
    bs.bs_ws_features(m.handle, values, b, x_prev, feat, b.clone(), delta)
    bs.bs_ws_fit_scaling(m.handle, feat, delta)
    return m, p, bt, values, b, x_prev, feat, delta


@pytest.mark.parametrize("n,M", [(54, 1), (54, 15), (54, 4097), (54, 8193), (54, 16500), (33, 9000),
                                 (64, 5000), (1, 300), (22, 12345)])
def test_forward_and_infer_tiles(n, M):
    print(f"n={n} M={M}", flush=True)
    m, _, bt, values, b, x_prev, feat, _ = model(n, M, n + M)
    y, x0 = torch.empty((M, n), dtype=torch.float32, device="cuda"), torch.empty_like(b)
    bs.bs_ws_forward(m.handle, feat, y)
    bs.bs_ws_infer(m.handle, values, b, x_prev, x0)
    rows = np.repeat(np.arange(n), np.diff(bt.row_ptr))
    diag = values[:, torch.from_numpy(np.flatnonzero(rows == bt.col_idx)).cuda()].contiguous()
    weights = torch.empty(bs.bs_ws_packed_bytes(n), dtype=torch.uint8, device="cuda")
    bs.bs_ws_pack(m.handle, weights)
    xp = torch.empty_like(b)
    bs.bs_ws_infer_packed(weights, n, diag, b, x_prev, xp)
    assert torch.equal(x0, xp)
    for k0 in (0, max(0, M - 40)):  # the first samples and the ragged end, alone
        k = slice(k0, k0 + 40)
        ys = torch.empty_like(y[k])
        bs.bs_ws_forward(m.handle, feat[k].contiguous(), ys)
        xs = torch.empty_like(b[k])
        bs.bs_ws_infer(m.handle, values[k].contiguous(), b[k].contiguous(), x_prev[k].contiguous(), xs)
        torch.cuda.synchronize()
        assert torch.equal(ys, y[k]) and torch.equal(xs, x0[k])


@pytest.mark.parametrize("n,M,times", [(54, 1, 8192), (54, 63, 128), (54, 63, 256), (54, 2048, 4),
                                       (54, 2048, 8), (33, 700, 16), (64, 500, 32), (8, 1000, 16)])
def test_gradient_tiles(n, M, times):
    """The mean over a list of samples repeated 2^k times is the mean over the list; every
    rounded factor scales by 2^-k exactly, so only the order of the sums differs between the
    small tiles of the one call and the large ones of the other."""
    print(f"n={n} M={M} times={times}", flush=True)
    m, p, *_, feat, delta = model(n, M, n + M)
    got = []
    for t in (1, times):
        grad = torch.full((p.size,), float("nan"), dtype=torch.float32, device="cuda")
        loss = torch.empty(1, dtype=torch.float32, device="cuda")
        rows = torch.arange(M, device="cuda", dtype=torch.int32).repeat(t)
        bs.bs_ws_grad(m.handle, feat, delta, grad, loss, rows=rows)
        got.append((grad.double(), loss.double()))
    (g, lo), (r, lr) = got
    assert torch.isfinite(g).all() and abs(lo - lr) <= TOL * lr
    sizes = [3 * n * H, H, H * H, H, H * n, n]
    for a, c in zip(torch.split(g, sizes), torch.split(r, sizes)):
        assert torch.linalg.norm(a - c) <= TOL * torch.linalg.norm(c)
