"""Timed cases of the adaptive FSAI library: the calls a user's program makes, over the range of
sizes, storage types and forms it makes them with.

Matrices are the two families of this repository's tests and benchmark, generated on the GPU:
"lap7", the 7-point operator with constant or log-normal edge coefficients (about 7 entries a
row), and "elast27", the 27-point operator with 3 unknowns per node and log-normal cells
(about 81 entries a row).  Right-hand sides are b = A x with x ~ U(-1, 1); solves run from
x0 = 0 to a residual of 1e-8, setups with eps = 1e-2.
"""
import math

import torch

import paper_2010_14175_amd as af

EPS, RTOL, TAU = 1e-2, 1e-8, 2.0 ** -26


def listed():
    lap = dict(grid="lap7", kmax=5, s=1, g="f64")
    ela = dict(grid="elast27", kmax=10, s=2, g="f64")
    return [
        # one product with a small matrix, as a caller's own iteration makes it (latency)
        dict(name="spmv_elast27_14", kind="spmv", nx=14, ny=15, nz=13, sigma=1.0, **ela),
        # one preconditioner application inside a caller's own iteration, single-precision G
        dict(name="apply_lap7_35", kind="apply", nx=33, ny=27, nz=45, sigma=1.0, **{**lap, "g": "f32"}),
        # a block of eight vectors through a matrix prepared once
        dict(name="spmm8_elast27_61", kind="spmm", nx=61, ny=67, nz=59, sigma=1.0, k=8, **ela),
        # the smallest systems: a setup with the first use of its factor, and a solve with a kept preconditioner
        dict(name="setup_lap7_20", kind="setup", nx=20, ny=20, nz=20, sigma=1.0, **lap),
        dict(name="solve_lap7_20", kind="solve", nx=20, ny=20, nz=20, sigma=0.0, **lap),
        # setup and solve of one GPU's share of the weak-scaling Poisson problem
        dict(name="step_lap7_121", kind="step", nx=121, ny=121, nz=121, sigma=0.0, **lap),
        # the ordinary mechanics workload: its setup, a solve, and eight right-hand sides at once
        dict(name="setup_elast27_64", kind="setup", nx=64, ny=64, nz=64, sigma=1.0, **ela),
        dict(name="solve_elast27_64", kind="solve", nx=64, ny=64, nz=64, sigma=1.0, **ela),
        dict(name="multi8_elast27_43", kind="multi", nx=43, ny=47, nz=41, sigma=1.0, k=8, **ela),
        # many small anisotropic systems together
        dict(name="batch512", kind="batch", nsys=512, side_lo=10, side_hi=40, kmax=5, s=1, g="f64"),
        # a server with mixed requests, single-precision G
        dict(name="serve12", kind="serve", requests=12, n_lo=10000, n_hi=600000, slots=4, g="f32"),
        # the largest single-GPU workload, setup and solve, single-precision G
        dict(name="step_elast27_150", kind="step", nx=150, ny=150, nz=150, sigma=2.0, grid="elast27", kmax=15, s=3, g="f32"),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    kind = rng.choice(["spmv", "apply", "spmm", "setup", "setup", "solve", "solve", "step", "step", "multi", "batch", "serve"])
    if kind == "batch":
        lo = rng.randint(6, 14)
        return dict(kind=kind, nsys=int(_log(rng, 4, 512)), side_lo=lo, side_hi=lo + rng.randint(2, 24), kmax=5, s=1,
                    g=rng.choice(["f64", "f32"]))
    if kind == "serve":
        hi = int(_log(rng, 60000, 600000))
        return dict(kind=kind, requests=rng.randint(3, 12), n_lo=10000, n_hi=hi, slots=rng.choice([2, 4]), g="f32")
    grid = rng.choice(["lap7", "elast27"])
    n = _log(rng, 2e3, 1.8e6)
    if kind == "multi":
        n = _log(rng, 2e3, 4e5)
    side = (n / (3 if grid == "elast27" else 1)) ** (1 / 3)
    nx, ny, nz = (max(3, round(side * rng.uniform(0.8, 1.25))) for _ in range(3))
    kmax, s = (5, 1) if grid == "lap7" else rng.choice([(5, 2), (10, 2), (10, 2), (15, 3)])
    c = dict(kind=kind, grid=grid, nx=nx, ny=ny, nz=nz, kmax=kmax, s=s, g=rng.choice(["f64", "f32"]),
             sigma=rng.choice([1.0, 1.0, 2.0]) if grid == "elast27" or kind == "setup" else rng.choice([0.0, 1.0]))
    if kind in ("spmm", "multi"):
        c["k"] = rng.choice([1, 2, 4, 8])
    return c


# ---- matrices, as padded rows (column -1: no entry) ------------------------------------
def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _shift(idx, mask_dims, shape):
    """idx + the offset (dz, dy, dx), -1 outside the grid."""
    out = torch.full(shape, -1, dtype=torch.int64, device="cuda")
    src, dst = [], []
    for d, m in zip(mask_dims, shape):
        dst.append(slice(max(0, -d), m - max(0, d)))
        src.append(slice(max(0, d), m - max(0, -d)))
    out[tuple(dst)] = idx[tuple(src)]
    return out


def _lap7(nx, ny, nz, sigma, gen, c=(1.0, 1.0, 1.0)):
    """cols, vals [n, 7] in column order; edges carry exp(sigma xi), or the constants c."""
    shape = (nz, ny, nx)

    def edges(d, const):
        e = [nz, ny, nx]
        e[d] += 1
        if sigma == 0.0:
            return torch.full(e, const, dtype=torch.float64, device="cuda")
        return torch.exp(sigma * torch.randn(e, dtype=torch.float64, device="cuda", generator=gen))

    wx, wy, wz = edges(2, c[0]), edges(1, c[1]), edges(0, c[2])
    w = [wz[:-1], wy[:, :-1], wx[:, :, :-1], wx[:, :, 1:], wy[:, 1:], wz[1:]]
    diag = ((w[2] + w[3]) + (w[1] + w[4])) + (w[0] + w[5])
    idx = torch.arange(nx * ny * nz, device="cuda").reshape(shape)
    off = [(-1, 0, 0), (0, -1, 0), (0, 0, -1), (0, 0, 0), (0, 0, 1), (0, 1, 0), (1, 0, 0)]
    cols = torch.stack([_shift(idx, o, shape).reshape(-1) for o in off], 1)
    vals = torch.stack([-w[0], -w[1], -w[2], diag, -w[3], -w[4], -w[5]], -1).reshape(-1, 7)
    return cols, vals


def _elast27(nx, ny, nz, sigma, gen):
    """cols [nodes, 27] (nodes), vals [nodes, 3, 27, 3]: every cell e adds c_e (I_8 - 11'/8) (x) M_e
    with c_e = exp(sigma xi), M_e = I + w w'."""
    shape = (nz, ny, nx)
    r = torch.randn((4, nz + 1, ny + 1, nx + 1), dtype=torch.float64, device="cuda", generator=gen)
    c = torch.exp(sigma * r[0])
    m = {}
    for p in range(3):
        for q in range(p, 3):
            m[p, q] = m[q, p] = c * ((1.0 if p == q else 0.0) + r[1 + p] * r[1 + q])
    idx = torch.arange(nx * ny * nz, device="cuda").reshape(shape)
    cols = torch.empty((nx * ny * nz, 27), dtype=torch.int64, device="cuda")
    vals = torch.empty((nx * ny * nz, 3, 27, 3), dtype=torch.float64, device="cuda")
    o = 0
    for dz in (-1, 0, 1):
        for dy in (-1, 0, 1):
            for dx in (-1, 0, 1):
                cols[:, o] = _shift(idx, (dz, dy, dx), shape).reshape(-1)
                coef = 0.875 if (dx, dy, dz) == (0, 0, 0) else -0.125
                lows = [[0] if d < 0 else [1] if d > 0 else [0, 1] for d in (dz, dy, dx)]
                for p in range(3):
                    for q in range(p, 3):
                        v = None
                        for a in lows[0]:
                            for b in lows[1]:
                                for e in lows[2]:
                                    t = m[p, q][a:a + nz, b:b + ny, e:e + nx]
                                    v = t.clone() if v is None else v.add_(t)
                        vals[:, p, o, q] = (coef * v).reshape(-1)
                        if q > p:
                            vals[:, q, o, p] = vals[:, p, o, q]
                o += 1
    return cols, vals


def _padded(case, gen):
    """The matrix as padded rows (cols [n, w], vals [n, w])."""
    if case["grid"] == "lap7":
        return _lap7(case["nx"], case["ny"], case["nz"], case["sigma"], gen)
    bc, bv = _elast27(case["nx"], case["ny"], case["nz"], case["sigma"], gen)
    nodes = bc.shape[0]
    cols = torch.where(bc >= 0, 3 * bc, -3)[:, None, :, None] + torch.arange(3, device="cuda")
    cols = torch.where(bc[:, None, :, None] >= 0, cols, -1).expand(nodes, 3, 27, 3)
    return cols.reshape(3 * nodes, 81), bv.reshape(3 * nodes, 81)


def _product(cols, vals, x):
    """A x over the padded rows; x of one or several columns."""
    y = torch.empty((cols.shape[0],) + x.shape[1:], dtype=x.dtype, device=x.device)
    for a in range(0, cols.shape[0], 1 << 20):
        c, v = cols[a:a + (1 << 20)], vals[a:a + (1 << 20)]
        for j, xj in enumerate(x.reshape(x.shape[0], -1).unbind(1)):
            s = torch.where(c >= 0, v * xj[c.clamp(min=0)], 0.0).sum(1)
            y.reshape(y.shape[0], -1)[a:a + (1 << 20), j] = s
    return y


def _device_csr(cols, vals):
    keep = cols >= 0
    rp = torch.zeros(cols.shape[0] + 1, dtype=torch.int32, device="cuda")
    rp[1:] = torch.cumsum(keep.sum(1), 0).to(torch.int32)
    return af.DeviceCSR(rp, cols[keep].to(torch.int32), vals[keep].contiguous())


def _vector(n, gen, k=None):
    x = torch.rand((n,) if k is None else (n, k), dtype=torch.float64, device="cuda", generator=gen)
    return x.mul_(2).sub_(1)


def _precision(case):
    return af.F32 if case["g"] == "f32" else af.F64


def _batch(case, seed):
    """(cols, vals, offsets) of the block-diagonal batch: sides and coefficients from the seed."""
    cpu = torch.Generator().manual_seed(seed)
    u = torch.rand((case["nsys"], 5), dtype=torch.float64, generator=cpu)
    span = case["side_hi"] - case["side_lo"] + 1
    # the sides are the same for every seed, spread over their range, so that the work is too
    v = torch.rand((case["nsys"], 3), dtype=torch.float64, generator=torch.Generator().manual_seed(case["nsys"]))
    gen, allc, allv, off = _gen(seed), [], [], [0]
    for k in range(case["nsys"]):
        sides = [case["side_lo"] + min(span - 1, int(t * span)) for t in v[k].tolist()]
        c = [1.0, 1.0, 1.0]
        c[min(2, int(u[k, 4] * 3))] = math.exp(float(u[k, 3]) * math.log(1e3))
        cols, vals = _lap7(*sides, 0.0, gen, c)
        allc.append(torch.where(cols >= 0, cols + off[-1], -1))
        allv.append(vals)
        off.append(off[-1] + cols.shape[0])
    return torch.cat(allc), torch.cat(allv), off


def _requests(case):
    """The requests' matrices: sizes spread over [n_lo, n_hi], the two families in turn."""
    out = []
    for q in range(case["requests"]):
        n = case["n_lo"] * (case["n_hi"] / case["n_lo"]) ** (((5 * q) % case["requests"] + 0.5) / case["requests"])
        grid = "lap7" if q % 2 == 0 else "elast27"
        side = max(4, round((n / (3 if grid == "elast27" else 1)) ** (1 / 3)))
        out.append(dict(grid=grid, nx=side, ny=side, nz=side, sigma=1.0, kmax=5 if grid == "lap7" else 10,
                        s=1 if grid == "lap7" else 2, g=case["g"]))
    return out


# ---- the calls --------------------------------------------------------------------------
def prepare(case, seed):
    gen = _gen(seed)
    st = {"case": case}
    if case["kind"] == "batch":
        cols, vals, off = _batch(case, seed)
        st["offsets"] = off
    elif case["kind"] == "serve":
        st["requests"] = []
        for c in _requests(case):
            cols, vals = _padded(c, gen)
            b = _product(cols, vals, _vector(cols.shape[0], gen))
            st["requests"].append((c, _device_csr(cols, vals), b))
        st["server"] = af.Server(hbm_budget=64 << 30, max_slots=case["slots"], kmax=5, s=1, eps=EPS, rtol=RTOL,
                                 g_prec=_precision(case))
        return st
    else:
        cols, vals = _padded(case, gen)
    n = cols.shape[0]
    A = st["A"] = _device_csr(cols, vals)
    if case["kind"] in ("spmv", "apply", "spmm", "setup"):
        st["x"] = _vector(n, gen, case.get("k") if case["kind"] == "spmm" else None)
    else:
        st["b"] = _product(cols, vals, _vector(n, gen, case.get("k")))
    del cols, vals
    if case["kind"] in ("apply", "solve", "multi"):
        st["P"] = af.setup(A, case["kmax"], case["s"], EPS, g_prec=_precision(case))
    if case["kind"] == "spmm":
        st["M"] = af.PreparedMatrix(A)
    return st


def run(st):
    case, kind = st["case"], st["case"]["kind"]
    if kind == "spmv":
        return {"y": af.spmv(st["A"], st["x"])}
    if kind == "apply":
        return {"z": st["P"].apply(st["x"])}
    if kind == "spmm":
        return {"y": st["M"].spmm(st["x"])}
    if kind == "setup":
        P = af.setup(st["A"], case["kmax"], case["s"], EPS, g_prec=_precision(case))
        psi, steps, reason = P.export_rows()
        z = P.apply(st["x"])
        P.close()
        return {"psi": psi, "steps": steps, "reason": reason, "z": z}
    if kind == "solve":
        x, info = af.pcg_solve(st["A"], st["P"], st["b"], rtol=RTOL)
        return {"x": x, "iters": info.iters}
    if kind == "multi":
        X, infos = af.pcg_solve_multi(st["A"], st["P"], st["b"], rtol=RTOL)
        return {"x": X, "iters": [i.iters for i in infos]}
    if kind == "step":
        P = af.setup(st["A"], case["kmax"], case["s"], EPS, g_prec=_precision(case))
        x, info = af.pcg_solve(st["A"], P, st["b"], rtol=RTOL)
        P.close()
        return {"x": x, "iters": info.iters}
    if kind == "batch":
        P = af.setup_batched(st["A"], st["offsets"], case["kmax"], case["s"], EPS, g_prec=_precision(case))
        x, infos = af.pcg_solve_batched(st["A"], P, st["offsets"], st["b"], rtol=RTOL)
        P.close()
        return {"x": x, "iters": torch.tensor([i.iters for i in infos])}
    srv, xs, iters = st["server"], [], {}
    torch.cuda.current_stream().synchronize()  # the requests run on the server's own streams
    tickets = []
    for c, A, b in st["requests"]:
        xs.append(torch.empty_like(b))
        tickets.append(srv.submit(A, b, xs[-1], kmax=c["kmax"], s=c["s"]))
    while len(iters) < len(tickets):
        for r in srv.poll(wait_ms=1000):
            iters[r.ticket] = r.iters
    return {"x": xs, "iters": [iters[t] for t in tickets]}


# ---- the work ---------------------------------------------------------------------------
def _size(c):
    """(rows, entries) of a grid's matrix."""
    d = (c["nx"], c["ny"], c["nz"])
    if c["grid"] == "lap7":
        n = d[0] * d[1] * d[2]
        return n, 7 * n - 2 * (d[0] * d[1] + d[0] * d[2] + d[1] * d[2])
    return 3 * d[0] * d[1] * d[2], 9 * math.prod(3 * v - 2 for v in d)


def _setup_work(n, nnz, kmax, s, gb):
    """A read and G written once; per row the gradients, and one triangular system per step."""
    m = 1 + kmax * s
    flops = sum(2 * (1 + k * s) * nnz + n * 2 * s * (k * s) ** 2 for k in range(kmax))
    return 12 * nnz + 4 * n + (4 + gb) * n * m, flops


def _solve_work(n, nnz, m, gb, iters, k=1):
    """Every iteration reads A, G and G' once and makes the vector passes of the recurrence."""
    g = n * m
    return iters * (12 * nnz + 2 * (4 + gb) * g + 15 * 8 * n * k), iters * k * (2 * nnz + 4 * g + 12 * n)


def _iterations(c):
    """About as many as the families take: 34 at 20^3 and 148 at 121^3 (7-point), 72 at 64^3."""
    side = (c["nx"] * c["ny"] * c["nz"]) ** (1 / 3)
    return (3.0 if c["grid"] == "lap7" else 2.4) * side ** 0.81


def work(case):
    kind, gb = case["kind"], 4 if case["g"] == "f32" else 8
    if kind == "batch":
        # mean side of the batch, and the iterations of its systems
        side = (case["side_lo"] + case["side_hi"]) / 2
        n = case["nsys"] * side ** 3
        a = _setup_work(n, 6.8 * n, case["kmax"], case["s"], gb)
        b = _solve_work(n, 6.8 * n, 6, gb, 30)
        return {"bytes": a[0] + b[0], "flops": a[1] + b[1]}
    if kind == "serve":
        tot = [work(dict(c, kind="step")) for c in _requests(case)]
        return {"bytes": sum(t["bytes"] for t in tot), "flops": sum(t["flops"] for t in tot)}
    n, nnz = _size(case)
    m, k = 1 + case["kmax"] * case["s"], case.get("k", 1)
    if kind in ("spmv", "spmm"):
        return {"bytes": 12 * nnz + 4 * n + 16 * n * k, "flops": 2 * nnz * k}
    if kind == "apply":
        return {"bytes": 2 * (4 + gb) * n * m + 16 * n, "flops": 4 * n * m}
    a = _setup_work(n, nnz, case["kmax"], case["s"], gb) if kind in ("setup", "step") else (0, 0)
    b = _solve_work(n, nnz, m, gb, _iterations(case), k) if kind in ("solve", "multi", "step") else (0, 0)
    return {"bytes": a[0] + b[0], "flops": a[1] + b[1]}


# ---- the same in plain torch, 64 bits ----------------------------------------------------
def _plain_rows(cols, vals, rows, kmax, s):
    """Rows `rows` of G (Sec. 2 of arXiv 2010.14175): (columns in growth order with -1 where none, the
    row itself last; values; psi)."""
    R = rows.shape[0]
    rcol = rows[:, None]
    col_of_i, val_of_i = cols[rows], vals[rows]
    aii = torch.where(col_of_i == rcol, val_of_i, 0.0).sum(1)
    mem = torch.empty((R, 0), dtype=torch.int64, device=rows.device)
    gm = torch.empty((R, 0), dtype=vals.dtype, device=rows.device)
    gi = aii.rsqrt()
    live = torch.ones(R, dtype=torch.bool, device=rows.device)
    big = cols.shape[0]
    for _ in range(kmax):
        q = torch.cat([rcol, mem], 1)
        g = torch.cat([gi[:, None], gm], 1)
        qc = cols[q.clamp(min=0)]
        ok = (qc >= 0) & (qc < rcol[:, :, None]) & (q >= 0)[:, :, None]
        c = torch.where(ok, qc, big).reshape(R, -1)
        t = torch.where(ok, vals[q.clamp(min=0)] * g[:, :, None], 0.0).reshape(R, -1)
        c, order = torch.sort(c, dim=1, stable=True)
        slot = torch.cumsum(torch.cat([torch.zeros_like(c[:, :1]), (c[:, 1:] != c[:, :-1]).long()], 1), 1)
        v = torch.zeros_like(t).scatter_add_(1, slot, t.gather(1, order)).abs_()
        cc = torch.full_like(c, big).scatter_(1, slot, c)
        v[cc >= big] = -1.0
        for j in range(mem.shape[1]):
            v[cc == mem[:, j:j + 1]] = -1.0
        top = v.amax(1, keepdim=True)
        v[v <= 2.0 ** -40 * top] = -1.0
        new = []
        for _ in range(s):
            top = v.amax(1, keepdim=True)
            pick = torch.where((v >= (1.0 - TAU) * top) & (v > 0), cc, big).amin(1)
            pick = torch.where(live & (pick < big), pick, -1)
            v[cc == pick[:, None]] = -1.0
            new.append(pick)
        new = torch.stack(new, 1)
        live = live & (new[:, 0] >= 0)
        mem = torch.cat([mem, new], 1)
        # the dense system over the members (identity where there is none)
        m = mem.shape[1]
        mc, mv = cols[mem.clamp(min=0)], vals[mem.clamp(min=0)]
        has = mem >= 0
        S = torch.empty((R, m, m), dtype=vals.dtype, device=rows.device)
        for j in range(m):
            S[:, :, j] = torch.where((mc == mem[:, None, j:j + 1]) & has[:, :, None] & has[:, None, j:j + 1], mv, 0.0).sum(2)
        S = S + torch.diag_embed((~has).to(S.dtype))
        ai = torch.where((mc == rcol[:, :, None]) & has[:, :, None], mv, 0.0).sum(2)
        y = -torch.cholesky_solve(ai[:, :, None], torch.linalg.cholesky(S))[:, :, 0]
        psi = aii + (ai * y).sum(1)
        d = psi.rsqrt()
        old = torch.cat([gm, torch.zeros((R, s), dtype=vals.dtype, device=rows.device)], 1)
        gm = torch.where(live[:, None], y * d[:, None], old)
        gi = torch.where(live, d, gi)
        live = live & (psi > EPS * aii)
        if not bool(live.any()):
            break
    return torch.cat([mem, rcol], 1), torch.cat([gm, gi[:, None]], 1), gi ** -2.0


def _plain_factor(cols, vals, kmax, s):
    """G as padded rows with ascending columns (-1 first where a row has fewer); None if it takes long."""
    n, w = cols.shape
    if n * w * (1 + kmax * s) > 1.5e8:
        return None
    step = max(64, int(4e7 / (w * (1 + kmax * s) * 4)))
    parts = []
    for a in range(0, n, step):
        parts.append(_plain_rows(cols, vals, torch.arange(a, min(n, a + step), device=cols.device), kmax, s))
    m = max(p[0].shape[1] for p in parts)
    pad = [(torch.nn.functional.pad(c, (m - c.shape[1], 0), value=-1), torch.nn.functional.pad(v, (m - v.shape[1], 0)))
           for c, v, _ in parts]
    gc, gv = torch.cat([p[0] for p in pad]), torch.cat([p[1] for p in pad])
    gc, order = torch.sort(gc, dim=1)
    return gc, gv.gather(1, order), torch.cat([p[2] for p in parts])


def exact(case, seed):
    kind = case["kind"]
    gen = _gen(seed)
    if kind == "batch":
        cols, _, _ = _batch(case, seed)
        return {"x": _vector(cols.shape[0], gen), "iters": None}
    if kind == "serve":
        xs = []
        for c in _requests(case):
            cols, _ = _padded(c, gen)
            xs.append(_vector(cols.shape[0], gen))
        return {"x": xs, "iters": None}
    cols, vals = _padded(case, gen)
    n = cols.shape[0]
    x = _vector(n, gen, case.get("k") if kind in ("spmm", "multi") else None)
    if kind in ("spmv", "spmm"):
        return {"y": _product(cols, vals, x)}
    if kind in ("solve", "step", "multi"):
        return {"x": x, "iters": None}
    G = _plain_factor(cols, vals, case["kmax"], case["s"])
    if G is None:
        return None
    gc, gv, psi = G
    if case["g"] == "f32":
        gv = gv.float().double()
    t = torch.where(gc >= 0, gv * x[gc.clamp(min=0)], 0.0).sum(1)
    z = torch.zeros_like(x)
    for j in range(gc.shape[1]):
        z.index_add_(0, gc[:, j].clamp(min=0), torch.where(gc[:, j] >= 0, gv[:, j] * t, 0.0))
    return {"psi": psi, "steps": None, "reason": None, "z": z} if kind == "setup" else {"z": z}
