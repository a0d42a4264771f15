"""Performance cases: the solves, batches, served requests and single operators
that a user of the library runs, over the sizes and options it is used with.

A case is a dict of plain values.  `prepare` builds what a program holds before
the call (hierarchies, right-hand sides, a server), `run` makes one pass
through the public entry points, `work` states what a pass cannot do without
and `exact` gives the same outputs in 64-bit arithmetic from plain torch.
"""
import math
import time

import torch

import paper_0904_4152_amd as mg

DEV = "cuda"
F64, F32 = torch.float64, torch.float32
TOLS = (1e-6, 1e-8, 1e-10)
SIDES = (15, 1, 5, 12, 14)  # Dirichlet sides: all, or mixed with free sides


def _solve(name, L, **kw):
    c = {"name": name, "kind": "solve", "L": L, "precision": "f64", "krylov": False,
         "jitter": 0.2, "sides": 15, "tol": 1e-8, "nu": 2, "start": "zero_guess", "rhs": "uniform",
         "coarse": "cholesky", "coarse_level": 1}
    c.update(kw)
    return c


def listed():
    return [
        # the accuracy setting of the paper: one small FP64 solve on the
        # uniform 65 x 65 grid, bound by latency and launches
        _solve("solve_f64_L6", 6, jitter=0.0),
        # a small mixed-precision solve with free (Neumann) sides, a CG
        # coarse grid of level 2 and a vector the caller zeroes
        _solve("solve_mixed_free_L8", 8, precision="mixed", sides=12, start="zeros",
               coarse="cg", coarse_level=2),
        # an ordinary mixed solve, 1025 x 1025 jittered
        _solve("solve_mixed_L10", 10, precision="mixed"),
        # the headline: 4097 x 4097 jittered, Gaussian right-hand side
        _solve("solve_mixed_L12", 12, precision="mixed", rhs="gauss"),
        # the same size in plain FP64
        _solve("solve_f64_L12", 12, rhs="gauss"),
        # CG preconditioned by one FP32 cycle, warm-started as a time loop is
        _solve("solve_pcg_L11", 11, precision="mixed", krylov=True, start="warm"),
        # many independent small problems at once
        {"name": "batch_256", "kind": "batch", "count": 256, "lo": 5, "hi": 9, "tol": 1e-8},
        # a burst of served requests of mixed levels and tolerances
        {"name": "serve_32", "kind": "serve", "count": 32, "lo": 6, "hi": 10},
        # a cycle inside a user's own iteration, V(1,1) in FP64
        {"name": "cycle_f64_L9", "kind": "cycle", "L": 9, "dtype": "f64", "nu": 1, "jitter": 0.2,
         "sides": 15},
        # the band matrix-vector product at full size, in FP32
        {"name": "spmv_f32_L12", "kind": "op", "op": "spmv", "L": 12, "dtype": "f32",
         "jitter": 0.2, "sides": 15},
        # vector steps of a Krylov method around the library's operators
        {"name": "blas_f64_1M", "kind": "blas", "n": (1 << 20) + 3, "dtype": "f64"},
        # the shallow-water prediction step: four 4-band terms, 4096 x 4096
        {"name": "band4_f32_4096", "kind": "band4", "N": 4096, "dtype": "f32", "terms": 4,
         "source": True},
    ]


def draw(rng):
    kind = rng.choices(("solve", "batch", "serve", "cycle", "op", "blas", "band4"),
                       (10, 2, 1, 2, 3, 2, 1))[0]
    jitter = rng.choice((0.0, round(rng.uniform(0.01, 0.25), 3)))
    sides = rng.choice(SIDES[:1] * 2 + SIDES)
    dtype = rng.choice(("f32", "f64"))
    if kind == "solve":
        L = rng.randint(5, 12)
        krylov = rng.random() < 0.25
        coarse = rng.choice(("cholesky", "cholesky", "cg"))
        c = _solve("", L, precision=rng.choice(("f64", "mixed", "mixed")), jitter=jitter,
                   sides=sides, tol=rng.choice(TOLS if L < 12 else TOLS[:2]), krylov=krylov,
                   nu=rng.choice((2, 2, 2, 1, 3)) if L < 11 else 2,
                   start=rng.choice(("zero_guess", "zeros", "warm")),
                   rhs=rng.choice(("uniform", "gauss")), coarse=coarse,
                   coarse_level=rng.choice((2, 3, 4)) if coarse == "cg" else rng.choice((1, 1, 2)))
        del c["name"]
        return c
    if kind == "batch":
        lo = rng.randint(5, 7)
        return {"kind": kind, "count": int(2 ** rng.uniform(1, 8)), "lo": lo,
                "hi": rng.randint(lo, 9), "tol": rng.choice(TOLS)}
    if kind == "serve":
        return {"kind": kind, "count": rng.randint(4, 32), "lo": 6, "hi": rng.randint(7, 10)}
    if kind == "cycle":
        return {"kind": kind, "L": rng.randint(5, 12), "dtype": dtype, "nu": rng.choice((1, 2, 2)),
                "jitter": jitter, "sides": sides}
    if kind == "op":
        return {"kind": kind,
                "op": rng.choice(("spmv", "defect", "defect_norm", "smooth", "restrict",
                                  "prolong")),
                "L": rng.randint(5, 12), "dtype": dtype, "jitter": jitter, "sides": sides}
    if kind == "blas":
        return {"kind": kind, "n": int(2 ** rng.uniform(8, 26)) + rng.randint(0, 5),
                "dtype": dtype}
    return {"kind": kind, "N": rng.randint(65, 4096), "dtype": dtype, "terms": rng.randint(1, 4),
            "source": rng.random() < 0.5}


# ---------------------------------------------------------------- inputs

def _dtype(case):
    return F32 if case["dtype"] == "f32" else F64


def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _randn(n, dtype, g):
    return torch.randn(n, generator=g, device=DEV, dtype=dtype)


def _off_sides(N, sides):
    """1 at the unknowns, 0 at the nodes on the Dirichlet sides."""
    m = torch.ones(N, N, dtype=F64, device=DEV)
    if sides & 1:
        m[:, 0] = 0
    if sides & 2:
        m[:, -1] = 0
    if sides & 4:
        m[0] = 0
    if sides & 8:
        m[-1] = 0
    return m


def _solve_rhs(case, seed):
    N = (1 << case["L"]) + 1
    g = _gen(seed)
    v = _randn(N * N, F64, g) if case["rhs"] == "gauss" else \
        2 * torch.rand(N * N, generator=g, device=DEV, dtype=F64) - 1
    return v * _off_sides(N, case["sides"]).reshape(-1)


def _field(case, seed, salt, level, dtype):
    """A right-hand side or iterate of one level, zero on the Dirichlet sides."""
    N = (1 << level) + 1
    v = _randn(N * N, F64, _gen(seed * 16 + salt)) * _off_sides(N, case["sides"]).reshape(-1)
    return v.to(dtype)


def _batch_spec(case, seed):
    """(level, jitter, geometry seed) of each problem of a batch (the levels
    belong to the case, the grids to the seed)."""
    g = torch.Generator()
    g.manual_seed(4004 + case["count"])
    lv = torch.randint(case["lo"], case["hi"] + 1, (case["count"],), generator=g).tolist()
    g.manual_seed(seed)
    jit = (0.25 * torch.rand(case["count"], generator=g, dtype=F64)).tolist()
    return [(l, j, seed * 1000 + p) for p, (l, j) in enumerate(zip(lv, jit))]


def _level_rows(spec):
    """One buffer per level, a row per problem: its n nodes and one zero, so
    that every row starts on a 16-byte boundary (n is odd)."""
    by = {}
    for l, _, _ in spec:
        by[l] = by.get(l, 0) + 1
    return {"L%d" % l: torch.zeros(k, ((1 << l) + 1) ** 2 + 1, dtype=F64, device=DEV)
            for l, k in sorted(by.items())}


def _batch_rhs(L, seed):
    N = (1 << L) + 1
    v = 2 * torch.rand(N * N, generator=_gen(seed), device=DEV, dtype=F64) - 1
    return v * _off_sides(N, 15).reshape(-1)


def _serve_spec(case, seed):
    """(level, tolerance, jitter, geometry seed, rhs seed) of each request
    (levels and tolerances belong to the case, the rest to the seed)."""
    g = torch.Generator()
    g.manual_seed(5005 + case["count"])
    levels = list(range(case["lo"], case["hi"] + 1))
    p = torch.tensor([1.0 / l for l in levels])  # log-uniform in the level
    li = torch.multinomial(p, case["count"], replacement=True, generator=g).tolist()
    ti = torch.randint(0, 3, (case["count"],), generator=g).tolist()
    g.manual_seed(seed)
    jit = (0.25 * torch.rand(case["count"], generator=g, dtype=F64)).tolist()
    return [(levels[li[r]], TOLS[ti[r]], jit[r], seed * 1000 + r, seed * 1000 + 500 + r)
            for r in range(case["count"])]


def _op_levels(case):
    """Levels of the operator's input and output vectors."""
    L = case["L"]
    return {"restrict": (L, L - 1), "prolong": (L - 1, L)}.get(case["op"], (L, L))


def _band4_inputs(case, seed):
    N, dt = case["N"], _dtype(case)
    n = N * N
    g = _gen(seed)
    offs = [[1, -1, 2, -2], [N, -N, 2 * N, -2 * N], [1, -1, N, -N],
            [N + 1, N - 1, 1 - N, -N - 1]][:case["terms"]]
    bands = [2 * torch.rand(4, n, generator=g, device=DEV, dtype=dt) - 1 for _ in offs]
    v, w, u, s = (_randn(n, dt, g) for _ in range(4))
    return offs, bands, [v, w, u, u][:case["terms"]], u, (s if case["source"] else None)


def prepare(case, seed):
    kind = case["kind"]
    ctx = mg.Context(0)
    if kind == "solve":
        h = mg.Hierarchy(ctx, case["L"], coarse_level=case["coarse_level"],
                         jitter=case["jitter"], seed=seed, dirichlet_sides=case["sides"])
        if case["coarse"] == "cg":
            h.set_coarse_solver(mg.MG_COARSE_CG)
        b = _solve_rhs(case, seed)
        o = mg.default_opts(
            precision=mg.MG_PREC_MIXED if case["precision"] == "mixed" else mg.MG_PREC_FP64,
            rel_tol=case["tol"], nu_pre=case["nu"], nu_post=case["nu"],
            krylov=int(case["krylov"]), zero_guess=int(case["start"] == "zero_guess"))
        x0 = None
        if case["start"] == "warm":  # the solution of a slightly different right-hand side
            x0 = torch.zeros_like(b)
            h.solve(b + 0.1 * b.roll(1) * (b != 0), x0, mg.default_opts(rel_tol=1e-6))
        return {"case": case, "h": h, "b": b, "x": torch.zeros_like(b), "x0": x0, "opts": o}
    if kind == "batch":
        spec = _batch_spec(case, seed)
        hs = [mg.Hierarchy(ctx, l, jitter=j, seed=s) for l, j, s in spec]
        bs = [_batch_rhs(l, s) for l, _, s in spec]
        out = _level_rows(spec)
        row = {l: iter(v) for l, v in out.items()}
        xs = [next(row["L%d" % l])[:-1] for l, _, _ in spec]
        return {"case": case, "hs": hs, "bs": bs, "xs": xs, "out": out,
                "opts": mg.default_opts(precision=mg.MG_PREC_MIXED, rel_tol=case["tol"],
                                        zero_guess=1)}
    if kind == "serve":
        srv = mg.Server(ctx, slots=64, budget_bytes=64 << 30, max_level=11)
        return {"case": case, "srv": srv, "spec": _serve_spec(case, seed)}
    if kind in ("cycle", "op"):
        h = mg.Hierarchy(ctx, case["L"], jitter=case["jitter"], seed=seed,
                         dirichlet_sides=case["sides"])
        dt = _dtype(case)
        li, lo = (case["L"], case["L"]) if kind == "cycle" else _op_levels(case)
        x = _field(case, seed, 1, li, dt)
        return {"case": case, "h": h, "x": x, "b": _field(case, seed, 2, case["L"], dt),
                "x0": x.clone(), "out": _field(case, seed, 3, lo, dt)}
    if kind == "blas":
        g = _gen(seed)
        dt = _dtype(case)
        return {"case": case, "ctx": ctx, "x": _randn(case["n"], dt, g),
                "y": _randn(case["n"], dt, g)}
    offs, bands, vs, u, s = _band4_inputs(case, seed)
    return {"case": case, "ctx": ctx, "offs": offs, "bands": bands, "vs": vs, "u": u, "s": s,
            "out": torch.empty_like(u)}


# ---------------------------------------------------------------- one pass

def _run_op(st):
    case, h = st["case"], st["h"]
    op, L = case["op"], case["L"]
    if op == "spmv":
        h.spmv(L, st["x"], st["out"])
    elif op == "defect":
        h.defect(L, st["b"], st["x"], st["out"])
    elif op == "defect_norm":
        return st["out"], h.defect(L, st["b"], st["x"], st["out"], norm=True)
    elif op == "smooth":
        st["x"].copy_(st["x0"])
        h.smooth(L, st["b"], st["x"], sweeps=2)
        return st["x"]
    elif op == "restrict":
        h.restrict(L, st["x"], st["out"])
    else:
        st["out"].zero_()
        h.prolong(L, st["x"], st["out"])
    return st["out"]


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "solve":
        x = state["x"]
        if case["start"] == "zeros":
            x.zero_()
        elif case["start"] == "warm":
            x.copy_(state["x0"])
        state["h"].solve(state["b"], x, state["opts"])
        return x
    if kind == "batch":
        mg.solve_batch(state["hs"], state["bs"], state["xs"], state["opts"])
        return state["out"]
    if kind == "serve":
        srv = state["srv"]
        tickets = [(srv.submit(L, tol, j, gs, rs, keep_x=True), ((1 << L) + 1) ** 2)
                   for L, tol, j, gs, rs in state["spec"]]
        while srv.info().completed < state.get("served", 0) + len(tickets):
            time.sleep(5e-5)
        state["served"] = state.get("served", 0) + len(tickets)
        xs = []
        for t, n in tickets:
            rc, _, x = srv.poll(t, n)
            while rc == mg.MG_ERR_BUSY:
                time.sleep(5e-5)
                rc, _, x = srv.poll(t, n)
            mg.check(rc)
            xs.append(x)
        return xs
    if kind == "cycle":
        x = state["x"]
        x.copy_(state["x0"])
        state["h"].vcycle(case["L"], state["b"], x, nu_pre=case["nu"], nu_post=case["nu"])
        return x
    if kind == "op":
        return _run_op(state)
    if kind == "blas":
        ctx = state["ctx"]
        ctx.axpy(1e-3, state["x"], state["y"])
        return state["y"], ctx.dot(state["x"], state["y"]), ctx.norm2(state["y"])
    state["ctx"].band4_combine(state["bands"], state["offs"], state["vs"], state["u"],
                               state["out"], s=state["s"])
    return state["out"]


# ---------------------------------------------------------------- work

def _solve_work(L, tol, mixed=True):
    # bands (symmetric: five of nine), b read, x written once; flops: one
    # digit per V(2,2) cycle, four sweeps and a residual each, 4/3 for the
    # coarser levels
    n = ((1 << L) + 1) ** 2
    cycles = math.ceil(-math.log10(tol))
    return 8.0 * 7 * n, 4 / 3 * cycles * (4 * 21 + 2 * 18 + 10) * n


def work(case):
    kind = case["kind"]
    if kind == "solve":
        b, f = _solve_work(case["L"], case["tol"])
        return {"bytes": b, "flops": f}
    if kind == "batch":
        # levels are drawn uniformly
        lv = range(case["lo"], case["hi"] + 1)
        w = [_solve_work(l, case["tol"]) for l in lv]
        k = case["count"] / len(w)
        return {"bytes": k * sum(x[0] for x in w), "flops": k * sum(x[1] for x in w)}
    if kind == "serve":
        lv = range(case["lo"], case["hi"] + 1)
        z = sum(1 / l for l in lv)
        b = f = 0.0
        for l in lv:
            n = ((1 << l) + 1) ** 2
            k = case["count"] / l / z
            # the problem comes from its seeds: only the solution is moved
            b += k * 8.0 * n
            f += k * (_solve_work(l, 1e-8)[1] + 400.0 * 4 / 3 * n)
        return {"bytes": b, "flops": f}
    s = 4 if case["dtype"] == "f32" else 8
    if kind == "cycle":
        n = ((1 << case["L"]) + 1) ** 2
        k = 2 * case["nu"]
        return {"bytes": s * n * (5 * 4 / 3 + 3.0), "flops": 4 / 3 * (21 * k + 28) * n}
    if kind == "op":
        n = ((1 << case["L"]) + 1) ** 2
        streams = {"spmv": 7, "defect": 8, "defect_norm": 8, "smooth": 8, "restrict": 1.25,
                   "prolong": 1.25}[case["op"]]
        flops = {"spmv": 17, "defect": 18, "defect_norm": 20, "smooth": 42, "restrict": 3,
                 "prolong": 3}[case["op"]]
        return {"bytes": float(s * n * streams), "flops": float(flops * n)}
    if kind == "blas":
        # y updated, then x . y and ||y||: two vectors in, one out
        return {"bytes": 3.0 * s * case["n"], "flops": 6.0 * case["n"]}
    n, m = case["N"] ** 2, case["terms"]
    vecs = min(m, 2) + 1  # distinct input vectors
    return {"bytes": float(s * n * (4 * m + vecs + 1 + int(case["source"]))),
            "flops": float(n * (8 * m + int(case["source"])))}


# ---------------------------------------------------------------- 64-bit values
# Plain torch, from the mathematics: bilinear elements with 2 x 2 Gauss points,
# the geometric V-cycle, and (for solves) cycles until the residual stalls.
# Every field has shape (problems, N, N), rows along y.

def _i64(v):
    return v - (1 << 64) if v >= 1 << 63 else v


def _shr(z, k):
    return (z >> k) & ((1 << (64 - k)) - 1)


def _u01(seed, k):
    """SplitMix64 draw k of a seed, as a uniform number of [0, 1)."""
    z = (k + 1) * _i64(0x9E3779B97F4A7C15) + _i64(seed % (1 << 64))
    z = (z ^ _shr(z, 30)) * _i64(0xBF58476D1CE4E5B9)
    z = (z ^ _shr(z, 27)) * _i64(0x94D049BB133111EB)
    return _shr(z ^ _shr(z, 31), 11).to(F64) * 2.0 ** -53


def _grid(L, jitter, seed):
    N = (1 << L) + 1
    h = 1.0 / (N - 1)
    t = torch.arange(N, device=DEV, dtype=F64) * h
    y, x = (v.clone() for v in torch.meshgrid(t, t, indexing="ij"))
    if jitter:
        p = torch.arange(N * N, device=DEV).reshape(N, N)
        inner = _off_sides(N, 15)
        x += (2 * _u01(seed, 2 * p) - 1) * jitter * h * inner
        y += (2 * _u01(seed, 2 * p + 1) - 1) * jitter * h * inner
    return x, y


CORNER = ((0, 0), (1, 0), (1, 1), (0, 1))  # (x, y) of an element's corners in order
REF = ((-1.0, -1.0), (1.0, -1.0), (1.0, 1.0), (-1.0, 1.0))


def _matrix(X, Y, mask):
    """The nine bands {(dj, di): field} on grids X, Y of shape (B, N, N)."""
    B, N, _ = X.shape
    cut = [(slice(cy, N - 1 + cy), slice(cx, N - 1 + cx)) for cx, cy in CORNER]
    cx = [X[:, r, c] for r, c in cut]
    cy = [Y[:, r, c] for r, c in cut]
    A = {(dj, di): torch.zeros_like(X) for dj in (-1, 0, 1) for di in (-1, 0, 1)}
    g = 1 / math.sqrt(3)
    K = {}
    for xi, eta in ((-g, -g), (g, -g), (-g, g), (g, g)):
        dxi = [0.25 * a * (1 + b * eta) for a, b in REF]
        det_ = [0.25 * b * (1 + a * xi) for a, b in REF]
        xx = sum(d * c for d, c in zip(dxi, cx))
        xe = sum(d * c for d, c in zip(det_, cx))
        yx = sum(d * c for d, c in zip(dxi, cy))
        ye = sum(d * c for d, c in zip(det_, cy))
        inv = 1 / (xx * ye - xe * yx)
        G = [ye * p - yx * q for p, q in zip(dxi, det_)]
        H = [xx * q - xe * p for p, q in zip(dxi, det_)]
        for a in range(4):
            for b in range(a, 4):
                v = (G[a] * G[b] + H[a] * H[b]) * inv
                K[a, b] = K[a, b] + v if (a, b) in K else v
    for a in range(4):
        for b in range(4):
            (ax, ay), (bx, by) = CORNER[a], CORNER[b]
            r, c = cut[a]
            A[by - ay, bx - ax][:, r, c] += K[min(a, b), max(a, b)]
    pad = torch.nn.functional.pad(mask, (1, 1, 1, 1))
    for (dj, di), v in A.items():
        v *= mask * pad[1 + dj:1 + dj + N, 1 + di:1 + di + N]
    A[0, 0] += 1 - mask
    return A


def _apply(A, x):
    N = x.shape[-1]
    xp = torch.nn.functional.pad(x, (1, 1, 1, 1))
    y = torch.zeros_like(x)
    for (dj, di), v in A.items():
        y.addcmul_(v, xp[:, 1 + dj:1 + dj + N, 1 + di:1 + di + N])
    return y


def _restrict(d, mask):
    p = torch.nn.functional.pad(d, (1, 1, 1, 1))
    N, e = d.shape[-1], 0.5
    s = torch.zeros_like(d[:, ::2, ::2])
    for dj in (0, 1, 2):
        for di in (0, 1, 2):
            w = e ** (abs(dj - 1) + abs(di - 1))
            s += w * p[:, dj:dj + N:2, di:di + N:2]
    return s * mask


def _prolong(c):
    B, Nc, _ = c.shape
    N = 2 * Nc - 1
    f = torch.zeros(B, N, N, dtype=c.dtype, device=c.device)
    f[:, ::2, ::2] = c
    f[:, ::2, 1::2] = 0.5 * (c[:, :, :-1] + c[:, :, 1:])
    f[:, 1::2] = 0.5 * (f[:, :-1:2] + f[:, 2::2])
    return f


class _Multigrid:
    """Levels coarse..L of one grid, or of a stack of grids of one level."""

    def __init__(self, xs, ys, sides, coarse=1):
        N = xs.shape[-1]
        self.L = (N - 1).bit_length() - 1
        self.coarse = coarse
        self.mask, self.A = {}, {}
        for l in range(coarse, self.L + 1):
            s = 1 << (self.L - l)
            self.mask[l] = _off_sides((1 << l) + 1, sides)
            self.A[l] = _matrix(xs[:, ::s, ::s].contiguous(), ys[:, ::s, ::s].contiguous(),
                                self.mask[l])
        m = ((1 << coarse) + 1) ** 2
        Nc = (1 << coarse) + 1
        cols = []
        for k in range(m):
            e = torch.zeros(m, dtype=F64, device=DEV)
            e[k] = 1
            cols.append(_apply(self.A[coarse], e.reshape(1, Nc, Nc).expand_as(
                self.A[coarse][0, 0]).contiguous()).reshape(-1, m))
        self.inv = torch.linalg.inv(torch.stack(cols, 2).cpu()).to(DEV)

    def cycle(self, l, b, x, nu, omega=0.7):
        if l == self.coarse:
            v = (self.inv * b.reshape(b.shape[0], 1, -1)).sum(2)
            return v.reshape(b.shape)
        A = self.A[l]
        for _ in range(nu):
            x = x + omega * (b - _apply(A, x)) / A[0, 0]
        d = _restrict(b - _apply(A, x), self.mask[l - 1])
        x = x + _prolong(self.cycle(l - 1, d, torch.zeros_like(d), nu))
        for _ in range(nu):
            x = x + omega * (b - _apply(A, x)) / A[0, 0]
        return x

    def solve(self, b):
        x, best = torch.zeros_like(b), math.inf
        for _ in range(60):
            x = self.cycle(self.L, b, x, 2)
            r = float(((b - _apply(self.A[self.L], x)).norm(dim=(1, 2)) /
                       b.norm(dim=(1, 2))).max())
            if r > 0.5 * best:  # down to rounding
                break
            best = r
        return x


def _one(case, seed):
    x, y = _grid(case["L"], case["jitter"], seed)
    return _Multigrid(x[None], y[None], case["sides"])


def _stacked(specs):
    """Solutions of problems (level, jitter, geometry seed, right-hand side),
    all sides Dirichlet, those of one level together."""
    out = [None] * len(specs)
    for l in sorted({s[0] for s in specs}):
        at = [k for k, s in enumerate(specs) if s[0] == l]
        grids = [_grid(l, specs[k][1], specs[k][2]) for k in at]
        m = _Multigrid(torch.stack([g[0] for g in grids]), torch.stack([g[1] for g in grids]), 15)
        N = (1 << l) + 1
        x = m.solve(torch.stack([specs[k][3].reshape(N, N) for k in at]))
        for k, v in zip(at, x):
            out[k] = v.reshape(-1)
    return out


def _serve_rhs(L, seed):
    N = (1 << L) + 1
    u = _u01(seed, torch.arange(N * N, device=DEV))
    return (2 * u - 1) * _off_sides(N, 15).reshape(-1)


def _exact_op(case, seed):
    op, L = case["op"], case["L"]
    dt = _dtype(case)
    li, _ = _op_levels(case)
    N = (1 << li) + 1
    x = _field(case, seed, 1, li, dt).to(F64).reshape(1, N, N)
    if op == "restrict":
        return _restrict(x, _off_sides((1 << (L - 1)) + 1, case["sides"])).reshape(-1)
    if op == "prolong":
        return _prolong(x).reshape(-1)
    gx, gy = _grid(L, case["jitter"], seed)
    A = _matrix(gx[None], gy[None], _off_sides(N, case["sides"]))
    if dt == F32:  # the FP32 operators work on the bands rounded to FP32
        A = {k: v.to(F32).to(F64) for k, v in A.items()}
    if op == "spmv":
        return _apply(A, x).reshape(-1)
    b = _field(case, seed, 2, L, dt).to(F64).reshape(1, N, N)
    if op == "smooth":
        for _ in range(2):
            x = x + 0.7 * (b - _apply(A, x)) / A[0, 0]
        return x.reshape(-1)
    d = (b - _apply(A, x)).reshape(-1)
    return d if op == "defect" else (d, float(d.norm()))


def exact(case, seed):
    kind = case["kind"]
    if kind == "solve":
        N = (1 << case["L"]) + 1
        return _one(case, seed).solve(_solve_rhs(case, seed).reshape(1, N, N)).reshape(-1)
    if kind == "batch":
        spec = _batch_spec(case, seed)
        xs = _stacked([(l, j, s, _batch_rhs(l, s)) for l, j, s in spec])
        out = _level_rows(spec)
        row = {l: iter(v) for l, v in out.items()}
        for (l, _, _), x in zip(spec, xs):
            next(row["L%d" % l])[:-1] = x
        return out
    if kind == "serve":
        return _stacked([(l, j, gs, _serve_rhs(l, rs))
                         for l, _, j, gs, rs in _serve_spec(case, seed)])
    if kind == "cycle":
        N, dt = (1 << case["L"]) + 1, _dtype(case)
        b, x = (_field(case, seed, k, case["L"], dt).to(F64).reshape(1, N, N) for k in (2, 1))
        return _one(case, seed).cycle(case["L"], b, x, case["nu"]).reshape(-1)
    if kind == "op":
        return _exact_op(case, seed)
    if kind == "blas":
        g = _gen(seed)
        dt = _dtype(case)
        x, y = _randn(case["n"], dt, g).to(F64), _randn(case["n"], dt, g).to(F64)
        y = y + 1e-3 * x
        return y, float((x * y).sum()), float(y.norm())
    offs, bands, vs, u, s = _band4_inputs(case, seed)
    n = u.numel()
    out = u.to(F64, copy=True)  # u may be one of vs
    for o4, bd, v in zip(offs, bands, vs):
        for k, o in enumerate(o4):
            lo, hi = max(0, -o), min(n, n - o)
            out[lo:hi] += bd[k, lo:hi].to(F64) * v[lo + o:hi + o].to(F64)
    return out + s.to(F64) if s is not None else out
