"""What a user of this library runs, as cases to be timed and compared.

A case is a plain dict.  Its ``kind`` names the path: ``solve`` (one shared sparsity
pattern, ``bs_batch_solve``), ``uneven`` (systems of many sizes and patterns,
``bs_varbatch_solve``), ``infer`` and ``grad`` (the learned initial guess).  The matrices
follow the families of ``workloads.py``, drawn on the GPU:

* ``tridiag``  3-point stencils, diagonally dominant (``spd``: symmetric, for CG);
* ``chem``     I - gamma J on a random pattern with |J| = 10^U(-3,3): gamma 1e-6 is the
  well-conditioned chemistry batch, 1e-4 to 1e-3 the stiff one that takes many iterations;
* ``mech``     the same model on the sizes and entry counts of reacting-flow mechanisms,
  a few dozen distinct systems replicated over the batch;
* ``grid9``    9-point nonsymmetric collision-like stencils on nx x ny grids.
"""
import numpy as np
import torch

from paper_2308_08417_amd import batchsolve as bs
from paper_2308_08417_amd import workloads as W

TOL, MAX_ITER = 1e-10, 500
SOLVERS = {"cg": bs.CG, "bicgstab": bs.BICGSTAB, "gmres": bs.GMRES, "trsv_lower": bs.TRSV_LOWER,
           "trsv_upper": bs.TRSV_UPPER}
PRECONDS = {"none": bs.PREC_NONE, "jacobi": bs.PREC_JACOBI, "block": bs.PREC_BLOCK_JACOBI,
            "ilu": bs.PREC_ILU}
FORMATS = {"csr": bs.CSR, "ell": bs.ELL, "dense": bs.DENSE}


def _solve(matrix, batch, fmt="csr", solver="bicgstab", precond="jacobi", precision="fp64", **more):
    return {"kind": "solve", "matrix": matrix, "batch": batch, "fmt": fmt, "solver": solver,
            "precond": precond, "precision": precision, **more}


def listed():
    return [
        # the small configuration: one call on a handful of little systems, where the
        # host path and the launch are what a time step waits for
        dict(_solve("tridiag", 64, n=32), name="tridiag_n32_b64"),
        # the paper's batch: one chemistry Jacobian per cell of a mesh
        dict(_solve("chem", 131072, n=54, fill=0.35, gamma=1e-6), name="chem_n54_b131072"),
        # the same cells kept in ELL and solved in mixed precision, an ordinary batch
        dict(_solve("chem", 16384, "ell", precision="mixed", n=54, fill=0.35, gamma=1e-6),
             name="chem_ell_mixed_b16384"),
        # the largest reacting-flow mechanism: rows of ~43 entries, teams of several waves
        dict(_solve("mech", 16384, mech="isooctane", gamma=1e-6), name="isooctane_b16384"),
        # stiff cells, where the solver and not the load decides: restarted GMRES
        dict(_solve("chem", 16384, solver="gmres", n=54, fill=0.35, gamma=1e-3),
             name="stiff_gmres_b16384"),
        # stiff cells with the strongest preconditioner
        dict(_solve("chem", 16384, precond="ilu", n=54, fill=0.35, gamma=3e-4),
             name="stiff_ilu_b16384"),
        # direct triangular solves of a chemistry batch
        dict(_solve("chem", 65536, solver="trsv_lower", precond="none", n=54, fill=0.35,
                    gamma=1e-6), name="trsv_n54_b65536"),
        # collision operators of a plasma mesh: one workgroup per system
        dict(_solve("grid9", 4096, nx=32, ny=31), name="grid9_n992_b4096"),
        # the same operators with ILU(0), level-scheduled sweeps
        dict(_solve("grid9", 1024, precond="ilu", nx=32, ny=31), name="grid9_ilu_n992_b1024"),
        # a batch of systems of every size from 16 to 1024 rows
        {"kind": "uneven", "batch": 16384, "n_min": 16, "n_max": 1024, "fmt": "csr",
         "solver": "bicgstab", "precision": "fp64", "name": "uneven_b16384"},
        # the learned initial guess of every cell of a time step
        {"kind": "infer", "n": 54, "batch": 65536, "packed": False, "name": "infer_n54_b65536"},
        # its training: forward, backward and gradients of a minibatch
        {"kind": "grad", "n": 54, "samples": 65536, "minibatch": 8192, "name": "grad_n54_m8192"},
    ]


def _log_int(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng):
    kind = rng.choice(["chem", "chem", "stiff", "stiff", "mech", "tridiag", "grid9", "grid9", "trsv",
                       "dense", "uneven", "infer", "grad"])
    fmt = rng.choice(["csr", "csr", "ell"])
    precision = rng.choice(["fp64", "fp64", "mixed"])
    if kind == "chem":
        return _solve("chem", _log_int(rng, 64, 65536), rng.choice(["csr", "ell", "dense"]),
                      rng.choice(["bicgstab", "gmres"]), "jacobi", precision,
                      n=rng.randint(10, 64), fill=round(rng.uniform(0.2, 0.5), 2), gamma=1e-6)
    if kind == "stiff":
        precond = rng.choice(["jacobi", "block", "ilu"])
        return _solve("chem", _log_int(rng, 64, 8192), fmt, rng.choice(["bicgstab", "gmres"]),
                      precond, "fp64", n=rng.randint(33, 64), fill=round(rng.uniform(0.2, 0.4), 2),
                      gamma=round(rng.uniform(1e-4, 3e-4), 6))
    if kind == "mech":
        return _solve("mech", _log_int(rng, 256, 16384), fmt, rng.choice(["bicgstab", "gmres"]),
                      mech=rng.choice(sorted(W.MECHANISMS)), gamma=1e-6)
    if kind == "tridiag":
        spd = rng.random() < 0.5
        return _solve("tridiag", _log_int(rng, 64, 8192), fmt, "cg" if spd else "bicgstab", spd=spd,
                      precond=rng.choice(["none", "jacobi"]), n=_log_int(rng, 8, 300))
    if kind == "grid9":
        solver = rng.choice(["bicgstab", "gmres"])
        precond = rng.choice(["jacobi", "block", "ilu"])
        # GMRES takes at most 512 rows with these preconditioners
        most = 16 if solver == "gmres" and precond != "jacobi" else 32
        return _solve("grid9", _log_int(rng, 64, 768), fmt, solver, precond,
                      precision if precond == "jacobi" else "fp64",
                      nx=rng.randint(9, 32), ny=rng.randint(8, most))
    if kind == "trsv":
        solver = rng.choice(["trsv_lower", "trsv_upper"])
        if rng.random() < 0.5:
            return _solve("chem", _log_int(rng, 64, 65536), fmt, solver, "none",
                          n=rng.randint(10, 64), fill=round(rng.uniform(0.2, 0.4), 2), gamma=1e-6)
        return _solve("grid9", _log_int(rng, 64, 2048), fmt, solver, "none",
                      nx=rng.randint(9, 32), ny=rng.randint(8, 32))
    if kind == "dense":  # rows too long for registers: the streamed placement
        return _solve("chem", _log_int(rng, 64, 1024), "dense", "bicgstab", "jacobi", precision,
                      n=rng.randint(65, 150), fill=1.0, gamma=1e-6)
    if kind == "uneven":
        solver = rng.choice(["bicgstab", "bicgstab", "cg"])
        return {"kind": "uneven", "batch": _log_int(rng, 256, 8192), "n_min": 16,
                "n_max": rng.randint(200, 1024), "fmt": fmt, "solver": solver,
                "precision": precision if solver == "bicgstab" else "fp64"}
    if kind == "infer":
        return {"kind": "infer", "n": rng.randint(16, 64), "batch": _log_int(rng, 64, 65536),
                "packed": rng.random() < 0.5}
    return {"kind": "grad", "n": rng.randint(16, 64), "samples": 65536,
            "minibatch": _log_int(rng, 64, 8192)}


# ------------------------------------------------------------------ shared-pattern matrices
def _pattern(case, rng):
    """(n, row_ptr, col_idx) of the case's shared pattern."""
    m = case["matrix"]
    if m == "tridiag":
        n = case["n"]
        mask = np.abs(np.subtract.outer(np.arange(n), np.arange(n))) <= 1
    elif m == "chem":
        n = case["n"]
        mask = rng.random((n, n)) < case["fill"]
        np.fill_diagonal(mask, True)
    elif m == "mech":
        _, n, nnz = W.MECHANISMS[case["mech"]]
        return (n, *W.mechanism_pattern(n, nnz, rng))
    else:
        rp, ci, _, _ = W.grid9_pattern(case["nx"], case["ny"])
        return case["nx"] * case["ny"], rp, ci
    row_ptr = np.concatenate([[0], np.cumsum(mask.sum(1))]).astype(np.int32)
    return n, row_ptr, np.nonzero(mask)[1].astype(np.int32)


def _uniform(shape, lo, hi, gen):
    return torch.rand(shape, dtype=torch.float64, device="cuda", generator=gen) * (hi - lo) + lo


def _matrices(case, seed, distinct=False):
    """Host pattern, CSR values [B][nnz] and right-hand sides [B][n] of a case (``distinct``:
    before the replication of a mechanism's systems)."""
    rng = np.random.default_rng(seed)
    gen = torch.Generator(device="cuda").manual_seed(seed)
    n, rp, ci = _pattern(case, rng)
    B, nnz, m = case["batch"], ci.size, case["matrix"]
    rows = np.repeat(np.arange(n), np.diff(rp))
    diag = torch.from_numpy(np.flatnonzero(rows == ci)).cuda()
    if m == "tridiag":
        values = _uniform((B, nnz), -1.1, -0.9, gen)
        if case.get("spd"):  # entry (i+1, i) takes the value of (i, i+1)
            values[:, torch.from_numpy(np.flatnonzero(ci < rows)).cuda()] = \
                values[:, torch.from_numpy(np.flatnonzero(ci > rows)).cuda()]
        values[:, diag] = _uniform((B, n), 4.0, 5.0, gen)
        b = _uniform((B, n), -1.0, 1.0, gen)
    elif m in ("chem", "mech"):
        k = B if m == "chem" else min(B, W.MECHANISMS[case["mech"]][0])
        values = torch.empty((k, nnz), dtype=torch.float64, device="cuda")
        for s in range(0, k, 16384):
            v = values[s:s + 16384]
            v.copy_(torch.pow(10.0, _uniform(v.shape, -3.0, 3.0, gen)))
            v.mul_((torch.rand(v.shape, device="cuda", generator=gen) < 0.5).double() * 2 - 1)
        values.mul_(-case["gamma"])
        values[:, diag] += 1.0
        b = _uniform((k, n), -1.0, 1.0, gen)
        if k < B and not distinct:  # the distinct systems in turn
            pick = torch.arange(B, device="cuda") % k
            values, b = values[pick], b[pick]
    else:
        _, _, dx, dy = W.grid9_pattern(case["nx"], case["ny"])
        dx, dy = torch.from_numpy(dx).cuda().double(), torch.from_numpy(dy).cuda().double()
        u = _uniform((B, 2), -1.0, 1.0, gen)
        c = torch.where((dx != 0) & (dy != 0), 0.5, 1.0)
        values = -(1 + 0.5 * (dx * u[:, :1] + dy * u[:, 1:])) * c
        values.mul_(_uniform((B, nnz), 0.95, 1.05, gen))
        values[:, diag] = 0.0
        total = torch.zeros((B, n), dtype=torch.float64, device="cuda")
        for s in range(9):  # slot by slot: each row's sum in a fixed order
            has = np.flatnonzero(np.diff(rp) > s)
            total[:, torch.from_numpy(has).cuda()] += values[:, torch.from_numpy(rp[has] + s).cuda().long()].abs()
        values[:, diag] = 1.2 * total
        b = _uniform((B, n), -1.0, 1.0, gen)
    return n, rp, ci, values, b


# ------------------------------------------------------------------ uneven batches
_SLOTS = 9  # widest band


def _uneven(case, seed):
    """Band systems of sizes spread evenly over n_min..n_max in random order, width
    U{5..9}: the handle's host arrays and, on the GPU, the band rows [rows][9], which of
    their slots are stored, their columns among all rows, and b."""
    rng = np.random.default_rng(seed)
    gen = torch.Generator(device="cuda").manual_seed(seed)
    B = case["batch"]
    n = rng.permutation(np.linspace(case["n_min"], case["n_max"], B).round().astype(np.int64))
    w = rng.integers(5, 10, size=B)
    spd = case["solver"] == "cg"
    if spd:
        w |= 1
    kl = (w - 1) // 2
    ku = w - 1 - kl
    keys, pat = np.unique(np.stack([n, kl, ku], 1), axis=0, return_inverse=True)
    rps, cis = [], []
    for pn, pl, pu in keys:
        i = np.arange(pn)[:, None]
        j = i + np.arange(-pl, pu + 1)[None, :]
        ok = (j >= 0) & (j < pn)
        rps.append(np.concatenate([[0], np.cumsum(ok.sum(1))]).astype(np.int32))
        cis.append(j[ok].astype(np.int32))
    rp_off = np.concatenate([[0], np.cumsum([r.size for r in rps])[:-1]]).astype(np.int64)
    ci_off = np.concatenate([[0], np.cumsum([c.size for c in cis])[:-1]]).astype(np.int64)
    host = (keys[:, 0].astype(np.int32), rp_off, np.concatenate(rps), ci_off, np.concatenate(cis),
            pat.reshape(-1).astype(np.int32))
    row_off = torch.from_numpy(np.concatenate([[0], np.cumsum(n)])).cuda()
    sys_of = torch.repeat_interleave(torch.arange(B, device="cuda"), torch.from_numpy(n).cuda())
    i = torch.arange(sys_of.numel(), device="cuda") - row_off[sys_of]
    off = torch.arange(_SLOTS, device="cuda") - torch.from_numpy(kl).cuda()[sys_of][:, None]
    j = i[:, None] + off
    has = (off <= torch.from_numpy(ku).cuda()[sys_of][:, None]) & (j >= 0)
    has &= j < torch.from_numpy(n).cuda()[sys_of][:, None]
    skew = _uniform((B, 1), -1.0, 1.0, gen)[sys_of]
    v = _uniform((sys_of.numel(), _SLOTS), 0.9, 1.1, gen)
    if spd:
        v.fill_(1.0).sub_(0.02 * off.abs()).mul_(0.9 + 0.1 * skew.abs())
    else:
        v.mul_(1.0 + 0.3 * skew * off.sign())
    v = torch.where(has & (off != 0), -v, 0.0)
    v = torch.where(off == 0, 1.2 * v.abs().sum(1, keepdim=True), v)
    b = _uniform((sys_of.numel(),), -1.0, 1.0, gen)
    col = (row_off[sys_of][:, None] + j).clamp_(0, sys_of.numel() - 1)
    return host, v, has, col, b


def _band_slots(host):
    """The same patterns as ELL: (rows, widths, offsets, columns, pattern of each system)
    and each pattern's slot-major position of every CSR entry."""
    rows, rp_off, rps, ci_off, cis, pat = host
    widths, offs, cols, pos, at = [], [], [], [], 0
    for p, pn in enumerate(rows):
        rp = rps[rp_off[p]:rp_off[p] + pn + 1]
        ci = cis[ci_off[p]:ci_off[p] + rp[-1]]
        r = np.repeat(np.arange(pn), np.diff(rp))
        k = np.arange(rp[-1]) - rp[r]
        wd = int(np.diff(rp).max())
        c = np.full(wd * pn, -1, np.int32)
        c[k * pn + r] = ci
        widths.append(wd)
        offs.append(at)
        cols.append(c)
        pos.append(k * pn + r)
        at += c.size
    return (rows, np.asarray(widths, np.int32), np.asarray(offs, np.int64), np.concatenate(cols),
            pat), pos


# ------------------------------------------------------------------ learned initial guess
def _cells(n, batch, seed):
    """A time step of chemistry cells: pattern, values, b and the previous solution."""
    case = _solve("chem", batch, n=n, fill=0.35, gamma=1e-6)
    n, rp, ci, values, b = _matrices(case, seed)
    gen = torch.Generator(device="cuda").manual_seed(seed + 7919)
    x_prev = b * (1.0 + 0.01 * _uniform(b.shape, -1.0, 1.0, gen))
    x_next = b + 1e-3 * torch.tanh(50 * (b - x_prev))
    return rp, ci, values, b, x_prev, x_next


def _features(case, batch, seed):
    """The cells, their training features and a model with its weights set and its scaling
    fitted to them."""
    n = case["n"]
    rp, ci, values, b, x_prev, x_next = _cells(n, batch, seed)
    net = bs.WarmStartModel(n, rp, ci)
    bs.bs_ws_set_params(net.handle, _weights(n, seed))
    feat = torch.empty((batch, 3 * n), dtype=torch.float32, device="cuda")
    delta = torch.empty((batch, n), dtype=torch.float32, device="cuda")
    bs.bs_ws_features(net.handle, values, b, x_prev, feat, x_next, delta)
    bs.bs_ws_fit_scaling(net.handle, feat, delta)
    return rp, ci, values, b, x_prev, feat, delta, net


def _weights(n, seed):
    p = W.mlp_init(n, seed=seed)
    p[-n:] = 0.01
    return p


# ------------------------------------------------------------------ the cases
def prepare(case, seed):
    kind = case["kind"]
    if kind == "solve":
        n, rp, ci, values, b = _matrices(case, seed)
        if case["fmt"] == "dense":
            full = torch.zeros((case["batch"], n * n), dtype=torch.float64, device="cuda")
            rows = np.repeat(np.arange(n), np.diff(rp))
            full[:, torch.from_numpy(rows * n + ci).cuda()] = values
            pattern, values = bs.Pattern.dense(n), full
        else:
            pattern = bs.Pattern.from_csr(rp, ci)
            if case["fmt"] == "ell":
                ell = torch.empty((case["batch"], pattern.ell_width * n), dtype=torch.float64, device="cuda")
                bs.bs_values_csr_to_ell(pattern.handle, values, ell)
                values = ell
        opts = bs.make_options(precision=bs.MIXED if case["precision"] == "mixed" else bs.FP64)
        return {"case": case, "pattern": pattern, "values": values, "b": b, "opts": opts}
    if kind == "uneven":
        host, v, has, col, b = _uneven(case, seed)
        if case["fmt"] == "ell":
            args, pos = _band_slots(host)
            val_at = np.concatenate([[0], np.cumsum((args[1] * args[0])[args[4]].astype(np.int64))])
            at = np.concatenate([val_at[s] + pos[p] for s, p in enumerate(args[4])])
            values = torch.zeros(int(val_at[-1]), dtype=torch.float64, device="cuda")
            values[torch.from_numpy(at).cuda()] = v[has]
            vb = bs.VarBatch(*args, ell=True)
        else:
            values = v[has].contiguous()
            vb = bs.VarBatch(*host)
        # the per-class launch plan the tuner finds for such batches (1024 x 1, 512 x 2,
        # 256 x 4, 512 x 2, 512 x 2 lanes x rows), kept as a program would keep it
        bs.bs_varbatch_set_plan(vb.handle, [0, 1, 2, 1, 1])
        opts = bs.make_options(precision=bs.MIXED if case["precision"] == "mixed" else bs.FP64,
                               flags=bs.FLAG_X0_ZERO)
        B = case["batch"]
        out = (torch.empty_like(b), torch.empty(B, dtype=torch.int32, device="cuda"),
               torch.empty(B, dtype=torch.float64, device="cuda"),
               torch.empty(B, dtype=torch.int32, device="cuda"))
        return {"case": case, "vb": vb, "values": values, "b": b, "opts": opts, "out": out}
    if kind == "infer":
        rp, ci, values, b, x_prev, feat, delta, net = _features(case, case["batch"], seed)
        state = {"case": case, "net": net, "values": values, "b": b, "x_prev": x_prev,
                 "x0": torch.empty_like(b)}
        if case["packed"]:
            rows = np.repeat(np.arange(case["n"]), np.diff(rp))
            state["diag"] = values[:, torch.from_numpy(np.flatnonzero(rows == ci)).cuda()].contiguous()
            state["weights"] = torch.empty(bs.bs_ws_packed_bytes(case["n"]), dtype=torch.uint8, device="cuda")
            bs.bs_ws_pack(net.handle, state["weights"])
        return state
    *_, feat, delta, net = _features(case, case["samples"], seed)
    gen = torch.Generator(device="cuda").manual_seed(seed + 1)
    rows = torch.randperm(case["samples"], device="cuda", generator=gen)[:case["minibatch"]].int()
    grad = torch.empty(bs.bs_ws_param_count(net.handle), dtype=torch.float32, device="cuda")
    loss = torch.empty(1, dtype=torch.float32, device="cuda")
    return {"case": case, "net": net, "feat": feat, "delta": delta, "rows": rows, "grad": grad, "loss": loss}


def run(state):
    case = state["case"]
    if case["kind"] == "solve":
        x, iters, resid, status = bs.solve(
            state["pattern"], state["values"], state["b"], fmt=FORMATS[case["fmt"]],
            solver=SOLVERS[case["solver"]], precond=PRECONDS[case["precond"]], tol=TOL,
            max_iter=MAX_ITER, opts=state["opts"])
        return {"x": x, "iters": iters, "resid": resid, "status": status}
    if case["kind"] == "uneven":
        x, iters, resid, status = state["out"]
        bs.bs_varbatch_solve(state["vb"].handle, state["values"], state["b"], x,
                             SOLVERS[case["solver"]], bs.PREC_JACOBI, TOL, MAX_ITER, iters, resid,
                             status, state["opts"])
        return {"x": x, "iters": iters, "resid": resid, "status": status}
    if case["kind"] == "infer":
        if case["packed"]:
            bs.bs_ws_infer_packed(state["weights"], case["n"], state["diag"], state["b"],
                                  state["x_prev"], state["x0"])
        else:
            bs.bs_ws_infer(state["net"].handle, state["values"], state["b"], state["x_prev"], state["x0"])
        return {"x0": state["x0"]}
    bs.bs_ws_grad(state["net"].handle, state["feat"], state["delta"], state["grad"], state["loss"],
                  rows=state["rows"])
    return {"grad": state["grad"], "loss": state["loss"]}


def _shape(case):
    """(rows, stored entries, padded entries) of one system, in expectation for random patterns."""
    m = case["matrix"]
    if m == "mech":
        _, n, nnz = W.MECHANISMS[case["mech"]]
        return n, nnz
    if m == "tridiag":
        return case["n"], 3 * case["n"] - 2
    if m == "grid9":
        return case["nx"] * case["ny"], (3 * case["nx"] - 2) * (3 * case["ny"] - 2)
    n = case["n"]
    return n, n * n if case["fmt"] == "dense" else int(n + case["fill"] * n * (n - 1))


def work(case):
    """Values and b read once, x and the per-system outputs written once; operations of a
    single product with each matrix (the iteration count is the solver's)."""
    if case["kind"] == "solve":
        n, nnz = _shape(case)
        return {"bytes": case["batch"] * (8.0 * nnz + 16.0 * n + 16), "flops": 2.0 * case["batch"] * nnz}
    if case["kind"] == "uneven":
        n = case["batch"] * (case["n_min"] + case["n_max"]) / 2
        return {"bytes": 8.0 * 7 * n + 16.0 * n + 16.0 * case["batch"], "flops": 14.0 * n}
    n = case["n"]
    layers = 3 * n * 256 + 256 * 256 + 256 * n
    if case["kind"] == "infer":
        return {"bytes": 8.0 * 4 * n * case["batch"], "flops": 2.0 * layers * case["batch"]}
    return {"bytes": 4.0 * 4 * n * case["minibatch"] + 8.0 * layers, "flops": 6.0 * layers * case["minibatch"]}


def _dense(n, rp, ci, values):
    rows = np.repeat(np.arange(n), np.diff(rp))
    a = torch.zeros((values.shape[0], n * n), dtype=torch.float64, device="cuda")
    a[:, torch.from_numpy(rows * n + ci).cuda()] = values
    return a.view(-1, n, n)


def _fixed_point(v, col, diag, b):
    """x = (b - (A - D) x) / D until it stands still (diagonally dominant rows); v, col
    [..][slots], missing slots 0."""
    x = b / diag
    for _ in range(260):
        x = (b - (v * x[col]).sum(-1)) / diag
    return x


def exact(case, seed):
    if case["kind"] == "solve":
        n, rp, ci, values, b = _matrices(case, seed, distinct=True)
        tri = case["solver"].startswith("trsv")
        if case["matrix"] in ("chem", "mech"):
            x = torch.empty_like(b)
            for s in range(0, b.shape[0], 4096):
                a, r = _dense(n, rp, ci, values[s:s + 4096]), b[s:s + 4096].unsqueeze(-1)
                if tri:
                    y = torch.linalg.solve_triangular(a, r, upper=case["solver"] == "trsv_upper")
                else:
                    y = torch.linalg.solve(a, r)
                x[s:s + 4096] = y.squeeze(-1)
            x = x[torch.arange(case["batch"], device="cuda") % x.shape[0]]
        else:  # stencils: padded rows over the flattened batch
            wd = int(np.diff(rp).max())
            rows = np.repeat(np.arange(n), np.diff(rp))
            slot = np.arange(ci.size) - rp[rows]
            keep = np.ones(ci.size, bool)
            if tri:
                keep = ci <= rows if case["solver"] == "trsv_lower" else ci >= rows
            col = np.zeros((n, wd), np.int64)
            col[rows, slot] = ci
            off = keep & (ci != rows)
            at = torch.from_numpy((rows * wd + slot)[off]).cuda()
            v = torch.zeros((b.shape[0], n * wd), dtype=torch.float64, device="cuda")
            v[:, at] = values[:, torch.from_numpy(np.flatnonzero(off)).cuda()]
            diag = values[:, torch.from_numpy(np.flatnonzero(rows == ci)).cuda()]
            base = torch.arange(b.shape[0], device="cuda")[:, None] * n
            cols = (base + torch.from_numpy(col.reshape(-1)).cuda()).view(-1, wd)
            x = _fixed_point(v.view(-1, wd), cols, diag.reshape(-1), b.reshape(-1)).view_as(b)
        return {"x": x, "iters": None, "resid": None, "status": None}
    if case["kind"] == "uneven":
        _, v, has, col, b = _uneven(case, seed)
        here = torch.arange(b.numel(), device="cuda")[:, None]
        diag = torch.where(has & (col == here), v, 0.0).sum(1)
        x = _fixed_point(torch.where(has & (col != here), v, 0.0), col, diag, b)
        return {"x": x, "iters": None, "resid": None, "status": None}
    n = case["n"]
    batch = case["batch"] if case["kind"] == "infer" else case["samples"]
    rp, ci, values, b, x_prev, x_next = _cells(n, batch, seed)
    rows = np.repeat(np.arange(n), np.diff(rp))
    diag = values[:, torch.from_numpy(np.flatnonzero(rows == ci)).cuda()]
    feat = torch.cat([diag, b - x_prev, x_prev], 1)
    delta = x_next - x_prev

    def spread(t):
        s = t.std(0, unbiased=False)
        return torch.where(s > 1e-30, s, 1.0)

    z = (feat - feat.mean(0)) / spread(feat)
    flat = torch.from_numpy(_weights(n, seed)).cuda().double()
    if case["kind"] == "grad":
        flat.requires_grad_(True)
    sizes = [3 * n * 256, 256, 256 * 256, 256, 256 * n, n]
    w1, b1, w2, b2, w3, b3 = torch.split(flat, sizes)

    def net(t):
        h = torch.relu(t @ w1.view(3 * n, 256) + b1)
        return torch.relu(h @ w2.view(256, 256) + b2) @ w3.view(256, n) + b3

    if case["kind"] == "infer":
        return {"x0": x_prev + spread(delta) * net(z)}
    gen = torch.Generator(device="cuda").manual_seed(seed + 1)
    pick = torch.randperm(case["samples"], device="cuda", generator=gen)[:case["minibatch"]]
    loss = ((net(z[pick]) - (delta / spread(delta))[pick]) ** 2).mean()
    loss.backward()
    return {"grad": flat.grad.detach(), "loss": loss.detach().reshape(1)}
