"""Workloads that the library is timed on: whole calls through the public binding.

listed() names them, draw(rng) gives one more of the same ranges, prepare(case,
seed) makes what a program holds before the call (inputs on the GPU, made from
the seed, and the solver context it keeps), run(state) is one call, work(case)
the bytes and operations the call cannot do without, exact(case, seed) the same
results from plain torch in 64 bits.

Kinds of case:
  uniform   a batch of LPs of one size, all rows <=, feasible origin: the
            random LPs the method is usually timed on
  uneven    a batch of mixed sizes with >= rows (two phases), some LPs
            infeasible and some unbounded
  support   one polytope queried in many directions (shared constraints)
  warm      the same, through the scoring network's row screening
  grads     the scoring network's forward and backward pass on a minibatch
  scaled    badly scaled LPs solved with power-of-two scaling
  box       closed-form support values of hyper-rectangles

Batches that come from host memory are not among them: that call is bound by
the upload over PCIe.
"""
import math

import numpy as np
import torch

from paper_1802_08557_amd import lpbatch, warmstart, workloads

PREC = {"fp64": lpbatch.PREC_FP64, "fp32cert": lpbatch.PREC_FP32_CERT64}


def listed():
    return [
        # The smallest call in use: a thousand toy LPs, all launch latency.
        dict(name="uniform_5x5_x1000", kind="uniform", num=1000, m=5, n=5, precision="fp64"),
        # The benchmark batch, in both precisions.
        dict(name="uniform_50x50_x100000", kind="uniform", num=100000, m=50, n=50, precision="fp64"),
        dict(name="uniform_50x50_x100000_fp32cert", kind="uniform", num=100000, m=50, n=50, precision="fp32cert"),
        # The largest LPs of the benchmark: tableaux in device memory.
        dict(name="uniform_500x500_x1000", kind="uniform", num=1000, m=500, n=500, precision="fp64"),
        # Odd mid-size LPs, one workgroup each.
        dict(name="uniform_117x150_x2000_fp32cert", kind="uniform", num=2000, m=117, n=150, precision="fp32cert"),
        # Mixed sizes, two phases, all statuses: a load-balancing workload.
        dict(name="uneven_10-300_x10000", kind="uneven", num=10000, lo=10, hi=300, precision="fp64"),
        dict(name="uneven_10-300_x10000_fp32cert", kind="uneven", num=10000, lo=10, hi=300, precision="fp32cert"),
        # Reachability queries: support functions of one polytope, plain and
        # through the learned warm start.
        dict(name="support_120x40_x100000", kind="support", num=100000, dim=20, facets=80, precision="fp64"),
        dict(name="warm_120x40_x100000_k48", kind="warm", num=100000, k=48),
        # One minibatch of the network's training.
        dict(name="grads_x512", kind="grads", num=512),
        # LPs whose rows and columns differ by many orders of magnitude.
        dict(name="scaled_50x50_x50000", kind="scaled", num=50000, m=50, n=50, precision="fp64"),
        # Template polyhedra: one box and direction per query.
        dict(name="box_n20_x1000000", kind="box", num=1000000, n=20, shared=False, want_x=False),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["uniform", "uniform", "uneven", "support", "warm", "grads", "scaled", "box"])
    precision = rng.choice(["fp64", "fp32cert"])
    if kind == "uniform":
        m, n = _log_int(rng, 3, 500), _log_int(rng, 3, 500)
        most = max(8, min(100000, int(2.5e8 / (m * n))))
        return dict(kind=kind, num=_log_int(rng, 1, most), m=m, n=n, precision=precision)
    if kind == "uneven":
        lo = rng.randint(4, 40)
        hi = rng.randint(lo + 8, 300)
        return dict(kind=kind, num=_log_int(rng, 20, 10000), lo=lo, hi=hi, precision=precision)
    if kind == "support":
        return dict(kind=kind, num=_log_int(rng, 100, 100000), dim=rng.randint(4, 24),
                    facets=rng.randint(40, 80), precision=precision)
    if kind == "warm":
        return dict(kind=kind, num=_log_int(rng, 100, 100000), k=rng.randint(40, 64))
    if kind == "grads":
        return dict(kind=kind, num=_log_int(rng, 16, 4096))
    if kind == "scaled":
        m, n = rng.randint(5, 120), rng.randint(5, 64)
        return dict(kind=kind, num=_log_int(rng, 20, 50000), m=m, n=n, precision=precision)
    return dict(kind=kind, num=_log_int(rng, 1000, 1000000), n=rng.randint(2, 40),
                shared=rng.random() < 0.5, want_x=rng.random() < 0.5)


# ---- inputs -----------------------------------------------------------------

def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _rand(g, lo, hi, *shape):
    return torch.rand(*shape, generator=g, dtype=torch.float64, device="cuda").mul_(hi - lo).add_(lo)


def _uniform(case, seed):
    """A ~ U[1,10], b ~ U[100,1000], c ~ U[1,10], every row <=."""
    N, m, n = case["num"], case["m"], case["n"]
    g = _gen(seed)
    return _rand(g, 1.0, 10.0, N, m, n), _rand(g, 100.0, 1000.0, N, m), _rand(g, 1.0, 10.0, N, n)


def _scaled(case, seed):
    """Uniform LPs with every row and column multiplied by 10^U[-3,3]."""
    A, b, c = _uniform(case, seed)
    g = _gen(seed + 7919)
    rf = torch.pow(10.0, _rand(g, -3.0, 3.0, *b.shape))
    cf = torch.pow(10.0, _rand(g, -3.0, 3.0, *c.shape))
    return A.mul_(rf[:, :, None]).mul_(cf[:, None, :]), b * rf, c * cf


def _dense_batch(A, b, c):
    N, m, n = A.shape
    return lpbatch.DeviceBatch(A.reshape(-1), b.reshape(-1), c.reshape(-1),
                               torch.zeros(N * m, dtype=torch.int8, device="cuda"),
                               np.full(N, m, np.int32), np.full(N, n, np.int32))


def _uneven(case, seed):
    """m, n ~ U{lo..hi}; A ~ N(0,1); 30 % of the rows >= with b ~ U[-50,-1],
    the rest <= with b ~ U[1,100]; c ~ U[-1,10].  5 % of the LPs get the
    infeasible last row x1 + x2 <= -1, another 5 % a zero column with c_j > 0
    (unbounded where feasible).  The sizes belong to the case, the LPs to the
    seed."""
    N, lo, hi = case["num"], case["lo"], case["hi"]
    rng = np.random.default_rng(1002)
    m = rng.integers(lo, hi + 1, N).astype(np.int32)
    n = rng.integers(lo, hi + 1, N).astype(np.int32)
    rng = np.random.default_rng(seed)
    order = rng.permutation(N)
    k = int(round(0.05 * N))
    infeasible, unbounded = order[:k], order[k:2 * k]
    aoff = np.concatenate([[0], np.cumsum(m.astype(np.int64) * n)])
    roff = np.concatenate([[0], np.cumsum(m.astype(np.int64))])
    coff = np.concatenate([[0], np.cumsum(n.astype(np.int64))])
    g = _gen(seed)
    A = torch.randn(int(aoff[-1]), generator=g, dtype=torch.float64, device="cuda")
    ge = torch.rand(int(roff[-1]), generator=g, device="cuda") < 0.3
    b = torch.where(ge, _rand(g, -50.0, -1.0, int(roff[-1])), _rand(g, 1.0, 100.0, int(roff[-1])))
    c = _rand(g, -1.0, 10.0, int(coff[-1]))
    sense = ge.to(torch.int8)
    if k:
        dev = lambda v: torch.from_numpy(np.ascontiguousarray(v, np.int64)).cuda()
        last = roff[infeasible + 1] - 1
        at = np.concatenate([np.arange(aoff[q + 1] - n[q], aoff[q + 1]) for q in infeasible])
        A[dev(at)] = 0.0
        A[dev(aoff[infeasible + 1] - n[infeasible])] = 1.0
        A[dev(aoff[infeasible + 1] - n[infeasible] + 1)] = 1.0
        b[dev(last)] = -1.0
        sense[dev(last)] = 0
        col = np.array([int(rng.integers(0, n[q])) for q in unbounded], np.int64)
        at = np.concatenate([aoff[q] + j + np.arange(m[q], dtype=np.int64) * n[q] for q, j in zip(unbounded, col)])
        A[dev(at)] = 0.0
        c[dev(coff[unbounded] + col)] = 5.0
    return lpbatch.DeviceBatch(A, b, c, sense, m, n), (aoff, roff, coff)


def _directions(g, N, dim):
    d = torch.randn(N, dim, generator=g, dtype=torch.float64, device="cuda")
    return d / d.norm(dim=1, keepdim=True)


def _support(case, seed):
    """The split form of a polytope and one objective per direction."""
    P = workloads.polytope(1003, case.get("facets", 80), case.get("dim", 20))
    A, b = workloads.split_form(P)
    d = _directions(_gen(seed), case["num"], P.dim)
    return A, b, d


def _shared_batch(A, b, d):
    N, (m, n) = int(d.shape[0]), A.shape
    dev = lambda v: torch.from_numpy(np.ascontiguousarray(v)).cuda()
    return lpbatch.DeviceBatch(dev(A.reshape(-1)), dev(b), torch.cat([d, -d], 1).reshape(-1),
                               torch.zeros(m, dtype=torch.int8, device="cuda"),
                               np.full(N, m, np.int32), np.full(N, n, np.int32), shared=True)


def _tight(A, b, d):
    """Tight rows of each direction's optimum (from plain torch)."""
    dA, db = torch.from_numpy(A).cuda(), torch.from_numpy(b).cuda()
    x = _exact_all_le(dA, db, torch.cat([d, -d], 1), shared=True)["x"].reshape(d.shape[0], -1)
    return (db - x @ dA.t() <= 1e-9 * (1.0 + db.abs())).to(torch.uint8)


def _random_params(seed):
    """He-uniform weights and zero biases of the 20-256-256-120 network."""
    g = _gen(seed)
    p = []
    for rows, cols in ((256, 20), (256, 256), (120, 256)):
        r = math.sqrt(6.0 / cols)
        p.append(_rand(g, -r, r, rows * cols))
        p.append(torch.zeros(rows, dtype=torch.float64, device="cuda"))
    return torch.cat(p).float()


def _unpack(p):
    out, o = [], 0
    for shape in ((256, 20), (256,), (256, 256), (256,), (120, 256), (120,)):
        size = math.prod(shape)
        out.append(p[o:o + size].reshape(shape))
        o += size
    return out


def _trained_params(A, b):
    """A network that ranks the tight rows, as a program keeps it: trained on
    20,000 directions of the polytope (Adam, plain torch)."""
    d = _directions(_gen(1203), 20000, 20)
    x, y = d.float(), _tight(A, b, d).float()
    ws = [w.clone().requires_grad_(True) for w in _unpack(_random_params(5))]
    opt = torch.optim.Adam(ws, lr=3e-3)
    pick = _gen(17)
    steps = 300
    for t in range(steps):
        for grp in opt.param_groups:
            grp["lr"] = 3e-3 * 0.5 * (1.0 + math.cos(math.pi * t / steps)) + 1e-5
        i = torch.randint(0, x.shape[0], (2048,), generator=pick, device="cuda")
        h = torch.relu(x[i] @ ws[0].t() + ws[1])
        h = torch.relu(h @ ws[2].t() + ws[3])
        loss = torch.nn.functional.binary_cross_entropy_with_logits(h @ ws[4].t() + ws[5], y[i])
        opt.zero_grad()
        loss.backward()
        opt.step()
    return torch.cat([w.detach().reshape(-1) for w in ws])


def _box(case, seed):
    N, n = case["num"], case["n"]
    g = _gen(seed)
    boxes = 1 if case["shared"] else N
    lo = _rand(g, -10.0, 0.0, boxes, n)
    hi = lo + _rand(g, 0.1, 10.0, boxes, n)
    if case["shared"]:
        lo, hi = lo[0].contiguous(), hi[0].contiguous()
    l = torch.randn(N, n, generator=g, dtype=torch.float64, device="cuda")
    l[torch.rand(N, n, generator=g, device="cuda") < 0.05] = 0.0
    return lo, hi, l


def prepare(case, seed):
    ctx = lpbatch.Context(0)
    kind = case["kind"]
    s = dict(kind=kind, ctx=ctx)
    if kind in ("uniform", "scaled"):
        s["batch"] = _dense_batch(*(_uniform if kind == "uniform" else _scaled)(case, seed))
    elif kind == "uneven":
        s["batch"] = _uneven(case, seed)[0]
    elif kind in ("support", "warm"):
        A, b, d = _support(case, seed)
        s["batch"] = _shared_batch(A, b, d)
        if kind == "warm":
            s["dirs"], s["k"] = d.float(), case["k"]
            ctx.mlp_set_params(_trained_params(A, b))
    elif kind == "grads":
        A, b = workloads.split_form(workloads.polytope(1003))
        d = _directions(_gen(seed), case["num"], 20)
        s["dirs"], s["tight"] = d.float(), _tight(A, b, d)
        ctx.mlp_set_params(_random_params(seed))
    else:
        s["lo"], s["hi"], s["l"] = _box(case, seed)
        s["want_x"] = case["want_x"]
    s["precision"] = PREC[case.get("precision", "fp64")]
    return s


def run(s):
    kind, ctx = s["kind"], s["ctx"]
    if kind == "grads":
        grad, loss = ctx.mlp_grads(s["dirs"], s["tight"])
        return {"grad": grad, "loss": loss}
    if kind == "box":
        value, x = ctx.hyperbox_support(s["lo"], s["hi"], s["l"], want_x=s["want_x"])
        return {"value": value, "x": x}
    if kind == "warm":
        r = warmstart.warm_solve(ctx, s["batch"], s["dirs"], s["k"])
    elif kind == "scaled":
        r = ctx.solve(s["batch"], precision=s["precision"], scaling=4)
    else:
        r = ctx.solve(s["batch"], precision=s["precision"])
    return {"status": r.status, "x": r.x, "obj": r.obj}


def work(case):
    """One read of every input and one write of every output; two operations
    per tableau entry and pivot, with the pivots per LP these distributions
    take (about 0.15 (m + n) / 2 + 1.3 for the uniform LPs, 2.1 (m + n) / 2
    for the uneven ones, 43 for the 120 x 40 support queries)."""
    kind, N = case["kind"], case["num"]
    if kind in ("uniform", "scaled"):
        m, n = case["m"], case["n"]
        pivots = 0.075 * (m + n) + 1.3
        return {"bytes": N * (8.0 * (m * n + m + n) + m + 8 * n + 12), "flops": N * pivots * 2.0 * (m + 1) * (n + 1)}
    if kind == "uneven":
        s, cells = (case["lo"] + case["hi"]) / 2, ((case["lo"] + case["hi"]) / 2) ** 2
        return {"bytes": N * (8.0 * (cells + 2 * s) + s + 8 * s + 12), "flops": N * 2.1 * s * 2.0 * 1.3 * cells}
    if kind in ("support", "warm"):
        dim, facets = case.get("dim", 20), case.get("facets", 80)
        m, n = facets + 2 * dim, 2 * dim
        rows = case.get("k", m)
        extra = 2.0 * (20 * 256 + 256 * 256 + 256 * 120) if kind == "warm" else 0.0
        return {"bytes": N * (8.0 * n + 8 * n + 12 + (80 if kind == "warm" else 0)) + 8.0 * m * (n + 1),
                "flops": N * (2.15 * dim * 2.0 * (rows + 1) * (n + 1) + extra)}
    if kind == "grads":
        return {"bytes": N * (80.0 + 120) + 8.0 * 102008, "flops": 6.0 * N * (20 * 256 + 256 * 256 + 256 * 120)}
    n = case["n"]
    return {"bytes": 8.0 * N * (n * (1 if case["shared"] else 3) + 1 + (n if case["want_x"] else 0)), "flops": 2.0 * N * n}


# ---- the same results from plain torch in 64 bits -----------------------------

def _solve_dense(A, b, c, ge, live_row, live_col):
    """Two-phase simplex on full tableaux, a whole batch at a time.

    A [B,m,n], b [B,m], c [B,n] in 64 bits, ge [B,m] rows that are >=; rows and
    columns outside live_row / live_col are padding.  Returns (status, x):
    0 optimal, 1 infeasible, 2 unbounded; x of the final basis with one step of
    iterative refinement."""
    B, m, n = A.shape
    dev = A.device
    flip = b < 0
    sg = torch.where(flip, -1.0, 1.0).to(torch.float64)
    A0, b0 = A * sg[:, :, None], b * sg
    art = (ge ^ flip) & live_row          # >= after the sign change: surplus and artificial
    ssign = torch.where(art, -1.0, 1.0).to(torch.float64)
    # Columns: n structurals, m slacks / surpluses, right-hand side.  The
    # artificial of a row starts basic and is never priced, so it needs no column.
    T = torch.zeros(B, m + 1, n + m + 1, dtype=torch.float64, device=dev)
    T[:, :m, :n] = A0
    T[:, :m, n:n + m] = torch.diag_embed(ssign)
    T[:, :m, -1] = b0
    status = torch.zeros(B, dtype=torch.int64, device=dev)
    rows = torch.arange(m, device=dev)
    basis = torch.where(art, n + m + rows, n + rows)
    allowed = torch.cat([live_col, live_row], 1)
    eps = 1e-9

    def simplex(T, basis, idx, scale):
        """Pivots LPs idx until each ends; returns those that are unbounded."""
        out = torch.zeros(B, dtype=torch.bool, device=dev)
        for _ in range(40 * (m + n)):
            if idx.numel() == 0:
                break
            d = torch.where(allowed[idx], T[idx, m, :-1], torch.full((), -math.inf, dtype=torch.float64, device=dev))
            best, e = d.max(1)
            go = best > eps * scale[idx]
            idx, e = idx[go], e[go]
            if idx.numel() == 0:
                break
            col = T[idx, :m, e]
            ratio = torch.where(col > eps, T[idx, :m, -1].clamp(min=0) / col, math.inf)
            r, l = ratio.min(1)
            ray = torch.isinf(r)
            out[idx[ray]] = True
            idx, e, l = idx[~ray], e[~ray], l[~ray]
            if idx.numel() == 0:
                break
            prow = T[idx, l] / T[idx, l, e][:, None]
            pcol = T[idx, :, e]
            part = 1 << 27
            step = max(1, part // ((m + 1) * (n + m + 1)))
            if idx.numel() == B:
                for q in range(0, B, step):
                    T[q:q + step].addcmul_(pcol[q:q + step, :, None], prow[q:q + step, None, :], value=-1.0)
            else:
                for q in range(0, idx.numel(), step):
                    i = idx[q:q + step]
                    T[i] = torch.addcmul(T[i], pcol[q:q + step, :, None], prow[q:q + step, None, :], value=-1.0)
            T[idx, l] = prow
            basis[idx, l] = e
        return out

    need = art.any(1)
    one = torch.ones(B, dtype=torch.float64, device=dev)
    if bool(need.any()):
        T[:, m] = torch.where(art[:, :, None], T[:, :m], 0.0).sum(1)
        scale1 = T[:, m, :n].abs().amax(1).clamp(min=1.0)
        simplex(T, basis, need.nonzero()[:, 0], scale1)
        w = torch.where(basis >= n + m, T[:, :m, -1], 0.0).sum(1)
        status[need & (w > 1e-9 * (1 + b.abs().amax(1)))] = 1
    # Phase II; an artificial left basic at zero stays on its row.
    cfull = torch.cat([c, torch.zeros(B, 2 * m, dtype=torch.float64, device=dev)], 1)
    cb = cfull.gather(1, basis)
    T[:, m] = 0.0
    T[:, m, :n] = c
    T[:, m] -= torch.matmul(cb[:, None, :], T[:, :m].contiguous())[:, 0]
    scale2 = c.abs().amax(1).clamp(min=1.0)
    ray = simplex(T, basis, (status == 0).nonzero()[:, 0], torch.maximum(scale2, one))
    status[ray] = 2
    # x_B = B^-1 b, refined: the slack columns of the tableau are B^-1 (by sign).
    inv = T[:, :m, n:n + m] * ssign[:, None, :]
    xb = T[:, :m, -1].clone()
    for _ in range(2):
        full = torch.zeros(B, n + 2 * m, dtype=torch.float64, device=dev)
        full.scatter_(1, basis, xb)
        res = b0 - torch.matmul(A0, full[:, :n, None])[:, :, 0] - ssign * full[:, n:n + m] - full[:, n + m:]
        xb = xb + torch.matmul(inv, res[:, :, None])[:, :, 0]
    full = torch.zeros(B, n + 2 * m, dtype=torch.float64, device=dev)
    full.scatter_(1, basis, xb)
    return status, full[:, :n]


def _pieces(total, cells):
    step = max(1, int(6e9 / (8 * cells)))
    for q in range(0, total, step):
        yield q, min(total, q + step)


def _lp_answer(status, x, c):
    """The binding's outputs: x and c.x where optimal, NaN or infinity elsewhere."""
    ok = status == 0
    obj = (c * x).sum(1)
    nan = torch.full_like(obj, math.nan)
    obj = torch.where(ok, obj, torch.where(status == 2, torch.full_like(obj, math.inf), nan))
    return torch.where(ok[:, None], x, torch.full_like(x, math.nan)), obj


def _exact_all_le(A, b, c, shared=False):
    N, n = c.shape
    m = b.shape[-1]
    xs, objs = [], []
    for q, r in _pieces(N, (m + 1) * (n + m + 1)):
        B = r - q
        Aq = A.expand(B, m, n) if shared else A[q:r]
        bq = b.expand(B, m) if shared else b[q:r]
        no, yes = torch.zeros(B, m, dtype=torch.bool, device=c.device), torch.ones(B, m, dtype=torch.bool, device=c.device)
        status, x = _solve_dense(Aq, bq, c[q:r], no, yes, torch.ones(B, n, dtype=torch.bool, device=c.device))
        x, obj = _lp_answer(status, x, c[q:r])
        xs.append(x)
        objs.append(obj)
    return {"status": None, "x": torch.cat(xs).reshape(-1), "obj": torch.cat(objs)}


def _exact_uneven(case, seed):
    """Padded groups of LPs of similar size."""
    batch, (aoff, roff, coff) = _uneven(case, seed)
    m, n, N = batch.m.astype(np.int64), batch.n.astype(np.int64), batch.num_lps
    x, obj = torch.zeros_like(batch.c), torch.zeros(N, dtype=torch.float64, device="cuda")
    order = np.lexsort((n, (m + 39) // 40))
    step = max(1, N // 16)
    for q in range(0, N, step):
        g = order[q:q + step]
        M, K = int(m[g].max()), int(n[g].max())
        dm, dn, da, dr, dc = (torch.from_numpy(np.ascontiguousarray(v[g], np.int64)).cuda() for v in (m, n, aoff[:-1], roff[:-1], coff[:-1]))
        i, j = torch.arange(M, device="cuda"), torch.arange(K, device="cuda")
        row, col = i[None, :] < dm[:, None], j[None, :] < dn[:, None]
        cell = row[:, :, None] & col[:, None, :]
        at = da[:, None, None] + i[None, :, None] * dn[:, None, None] + j[None, None, :]
        A = torch.where(cell, batch.A[torch.where(cell, at, 0)], 0.0)
        ri, ci = torch.where(row, dr[:, None] + i, 0), torch.where(col, dc[:, None] + j, 0)
        b = torch.where(row, batch.b[ri], 0.0)
        c = torch.where(col, batch.c[ci], 0.0)
        status, xs = _solve_dense(A, b, c, (batch.sense[ri] == 1) & row, row, col)
        xs, o = _lp_answer(status, xs, c)
        x[ci[col]] = xs[col]
        obj[torch.from_numpy(g).cuda()] = o
    return {"status": None, "x": x, "obj": obj}


def _exact_scaled(A, b, c):
    """Solved with rows and columns brought to unit geometric mean first."""
    r, s = torch.zeros_like(b), torch.zeros_like(c)
    E = A.abs().log2()
    for _ in range(4):
        v = E + s[:, None, :]
        r = -torch.round((v.amax(2) + v.amin(2)) / 2)
        v = E + r[:, :, None]
        s = -torch.round((v.amax(1) + v.amin(1)) / 2)
    R, S = torch.exp2(r), torch.exp2(s)
    out = _exact_all_le(A * R[:, :, None] * S[:, None, :], b * R, c * S)
    return {"status": None, "x": out["x"] * S.reshape(-1), "obj": out["obj"]}


def _exact_grads(case, seed):
    A, b = workloads.split_form(workloads.polytope(1003))
    d = _directions(_gen(seed), case["num"], 20)
    y = _tight(A, b, d).double()
    ws = [w.double().clone().requires_grad_(True) for w in _unpack(_random_params(seed))]
    x = d.float().double()
    h = torch.relu(x @ ws[0].t() + ws[1])
    h = torch.relu(h @ ws[2].t() + ws[3])
    loss = torch.nn.functional.binary_cross_entropy_with_logits(h @ ws[4].t() + ws[5], y)
    loss.backward()
    return {"grad": torch.cat([w.grad.reshape(-1) for w in ws]), "loss": loss.detach().reshape(1)}


def exact(case, seed):
    kind = case["kind"]
    if kind == "uniform":
        return _exact_all_le(*_uniform(case, seed))
    if kind == "scaled":
        return _exact_scaled(*_scaled(case, seed))
    if kind == "uneven":
        return _exact_uneven(case, seed)
    if kind in ("support", "warm"):
        A, b, d = _support(case, seed)
        return _exact_all_le(torch.from_numpy(A).cuda(), torch.from_numpy(b).cuda(), torch.cat([d, -d], 1), shared=True)
    if kind == "grads":
        return _exact_grads(case, seed)
    lo, hi, l = _box(case, seed)
    x = torch.where(l < 0, lo, hi)
    return {"value": (l * x).sum(1), "x": x if case["want_x"] else None}
