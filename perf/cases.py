"""Cases of the performance measurement of libtrg: what a user of the library
has it do, through its public entry points, from the smallest call to the
largest that ends within two seconds.

Five kinds of case:

* ``solve``        one whole HOTRG run: the Ising tensor, every coarse-graining
                   step of the lattice L^d, then ln Z/V, E, M and the step
                   records (what a scan over couplings does at each point);
* ``step``         steps of one steady-state run whose legs have reached Dcut
                   (what a long run spends its time on), HOTRG or ATRG;
* ``batch``        the same for several HOTRG runs stepped together, as the
                   solve server does;
* ``join``         the block-spin contraction of a bond dimension whose whole
                   step takes too long to repeat, as one product of a slice;
* ``observables``  ln Z/V, E, M and the degeneracy indicator X of a run.

Mixed precision is used for long steps and joins; whole solves run in FP64,
because a run of many steps near the transition amplifies the rounding of the
mixed joins.  The tensors of mixed steps are taken in FP32, the type of what
those joins deliver.  The pieces of ATRG are taken by modulus: the network is
invariant under a sign of every leg index, which rounding picks.
"""
import math
import random

import numpy as np
import torch

import paper_1911_12954_amd as trg

#: planes of a join operand per precision: how many, and of which type
PLANES = {"fp64": (1, torch.float64), "fp32": (1, torch.float32), "bf16x3": (2, torch.bfloat16),
          "bf16x6": (3, torch.bfloat16)}


# ------------------------------------------------------------------- cases ---
def listed():
    return [
        # Monitoring of a run: after a step the scan reads ln Z/V, E, M and X
        # (the bisection of the transition does it at every coupling).  Pure latency.
        {"name": "observables_4d_dcut6", "kind": "observables", "d": 4, "dcut": 6},
        # 2D study at a moderate lattice: small joins, Gram matrices of order 196 in
        # the selection eigensolver, latency of many small launches.
        {"name": "solve_2d_dcut14_L64", "kind": "solve", "d": 2, "dcut": 14, "L": 64, "impure": "E"},
        # The small 4D run (Dcut 4, 16^4, E and M): sixteen steps whose joins are
        # negligible; launches and the small eigenproblems count.
        {"name": "solve_4d_dcut4_L16", "kind": "solve", "d": 4, "dcut": 4, "L": 16, "impure": "EM"},
        # The solve server: eight Dcut-6 runs of one lane in shared launches, one sweep
        # over the four axes, in the server's mixed precision.
        {"name": "batch_dcut6_x8_bf16x6", "kind": "batch", "dcut": 6, "runs": 8, "steps": 4, "precision": "bf16x6"},
        # A run that follows E and M in FP32 joins: five joins a step.
        {"name": "step_dcut6_fp32_em", "kind": "step", "method": "hotrg", "dcut": 6, "steps": 2, "precision": "fp32",
         "impure": "EM"},
        # FP64 reference run at an odd bond dimension (K = 7^5: ragged in every tile).
        {"name": "step_dcut7_fp64", "kind": "step", "method": "hotrg", "dcut": 7, "steps": 2, "precision": "fp64",
         "impure": ""},
        # The headline mixed path at the largest bond dimension whose step ends in time.
        {"name": "step_dcut8_bf16x6", "kind": "step", "method": "hotrg", "dcut": 8, "steps": 2, "precision": "bf16x6",
         "impure": ""},
        # The Dcut = 10 join: one value of the outer leg x0 (10^4 rows, padded) against
        # as many rows of the other site, the whole K = 10^5.
        {"name": "join_dcut10_bf16x6", "kind": "join", "precision": "bf16x6", "M": 10112, "N": 10112, "K": 100000},
        {"name": "join_dcut10_fp64", "kind": "join", "precision": "fp64", "M": 10112, "N": 10112, "K": 100000},
        # The fast mixed path, at the Dcut = 9 join (K = 9^5 padded).
        {"name": "join_dcut9_bf16x3", "kind": "join", "precision": "bf16x3", "M": 13312, "N": 13312, "K": 59072},
        # ATRG at the bond dimension of the beta scan, one step.
        {"name": "atrg_dcut24", "kind": "step", "method": "atrg", "dcut": 24, "steps": 1, "precision": "fp64",
         "impure": "", "z2": False},
        # ATRG at a serving bond dimension in the symmetric (Z2) mode that the
        # transition bracket uses, two steps.
        {"name": "atrg_dcut10_z2", "kind": "step", "method": "atrg", "dcut": 10, "steps": 2, "precision": "fp64",
         "impure": "", "z2": True},
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    case = _draw(rng)
    if case["kind"] != "join" and not case.get("z2"):
        case["h"] = round(10.0 ** rng.uniform(-3.0, -2.0), 6)
    return case


def _draw(rng):
    kind = rng.choice(["observables", "solve", "solve", "batch", "step", "step", "join", "join", "atrg", "atrg"])
    if kind == "observables":
        d = rng.choice([2, 3, 4])
        return {"kind": kind, "d": d, "dcut": _log_int(rng, 2, {2: 24, 3: 10, 4: 7}[d])}
    if kind == "solve":
        d = rng.choice([2, 2, 3, 4])
        if d == 2:
            return {"kind": kind, "d": 2, "dcut": _log_int(rng, 4, 20), "L": 2 ** rng.randint(2, 6),
                    "impure": rng.choice(["", "E"])}
        if d == 3:
            return {"kind": kind, "d": 3, "dcut": _log_int(rng, 2, 10), "L": 2 ** rng.randint(1, 3),
                    "impure": rng.choice(["", "E", "EM"])}
        return {"kind": kind, "d": 4, "dcut": _log_int(rng, 2, 6), "L": 2 ** rng.randint(1, 3),
                "impure": rng.choice(["", "EM"])}
    if kind == "batch":
        dcut = rng.choice([4, 5, 6])
        return {"kind": kind, "dcut": dcut, "runs": _log_int(rng, 2, 8 if dcut == 6 else 24), "steps": rng.randint(1, 4),
                "precision": rng.choice(["fp64", "fp32", "bf16x3", "bf16x6"])}
    if kind == "step":
        dcut = rng.choice([5, 6, 7, 8])
        precision = rng.choice(["fp64", "fp32", "bf16x3", "bf16x6"])
        if dcut == 8:
            precision = rng.choice(["bf16x3", "bf16x6"])
        return {"kind": "step", "method": "hotrg", "dcut": dcut, "steps": rng.randint(1, 2 if dcut == 8 else 4),
                "precision": precision, "impure": rng.choice(["", "M", "EM"]) if dcut <= 6 else ""}
    if kind == "join":
        precision = rng.choice(["fp64", "fp32", "bf16x3", "bf16x6"])
        tm, tn, tk = (256, 256, 32) if precision == "bf16x3" else (128, 128, 16 if precision == "fp64" else 32)
        M, N = (t * _log_int(rng, 1, 10240 // t) for t in (tm, tn))
        return {"kind": kind, "precision": precision, "M": M, "N": N, "K": tk * _log_int(rng, 4, 100000 // tk)}
    # between 6 and 9 the cut splits a multiplet of the lattice symmetry, and
    # rounding picks the kept member
    dcut = rng.choice([4, 5, _log_int(rng, 10, 20), _log_int(rng, 10, 20)])
    z2 = rng.random() < 0.3
    # oversampling and power iterations over the range in which f no longer depends on them
    return {"kind": "step", "method": "atrg", "dcut": dcut, "steps": 1 if dcut > 10 else rng.randint(1, 2),
            "precision": "fp64", "impure": "" if z2 or dcut > 10 else rng.choice(["", "E"]), "z2": z2,
            "rsvd_p": rng.randint(2 * dcut, 5 * dcut), "rsvd_q": rng.randint(dcut, 2 * dcut)}


# ------------------------------------------------------------------ inputs ---
def _coupling(case, seed, i=0):
    """(beta, h) of the i-th run: near the transition of the 4D model, spread
    around it in 2D and 3D."""
    r = random.Random("%d/%d" % (seed, i))
    lo, hi = {2: (0.36, 0.50), 3: (0.19, 0.25), 4: (0.1490, 0.1505)}[case.get("d", 4)]
    beta = r.uniform(lo, hi)
    return beta, (0.0 if case.get("z2") else case.get("h", 1e-3))


def _ramp(d):
    """Steps after which every leg of a run has reached its bond dimension."""
    return {2: 10, 3: 6, 4: 4}[d]


def _context(case, seed, i=0):
    beta, h = _coupling(case, seed, i)
    cfg = dict(dcut=case["dcut"], precision=case.get("precision", "fp64"), impure=tuple(case.get("impure", "")))
    if case.get("method") == "atrg":
        cfg.update(method="atrg", z2=case["z2"], seed=seed & 0xffff, rsvd_p=case.get("rsvd_p", 0),
                   rsvd_q=case.get("rsvd_q", 0))
    return trg.trg_init_ising(beta, h, case.get("d", 4), **cfg)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "join":
        return _prepare_join(case, seed)
    if kind == "solve":
        return {"case": case, "seed": seed}
    if kind == "observables":
        case = dict(case, impure="EM")
    ctxs = [_context(case, seed, i) for i in range(case.get("runs", 1))]
    d = case.get("d", 4)
    for n in range(_ramp(d)):
        if kind == "batch":
            trg.trg_hotrg_step_batch(ctxs, n % d, case["dcut"])
        elif case.get("method") == "atrg":
            ctxs[0].atrg_step(n % d, case["dcut"])
        else:
            ctxs[0].hotrg_step(n % d, case["dcut"])
    for c in ctxs:
        c.sync()
    return {"case": case, "ctxs": ctxs, "n": _ramp(d)}


def _prepare_join(case, seed):
    """Operands as the step builds them: rows of an FP64 matrix whose columns
    decay over four decades (a normalised site tensor times isometries), in
    the planes of the join precision."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    planes, dtype = PLANES[case["precision"]]

    def operand(rows):
        out = torch.empty((planes, rows, case["K"]), dtype=dtype, device="cuda")
        scale = torch.exp(-9.2 * torch.rand(case["K"], generator=g, device="cuda"))
        for r0 in range(0, rows, 1024):
            x = torch.randn((min(1024, rows - r0), case["K"]), generator=g, device="cuda") * scale
            if planes == 1:
                out[0, r0:r0 + x.shape[0]] = x.to(dtype) if dtype == torch.float32 else x.double() * (1.0 / 3.0)
            else:
                for p in range(planes):
                    out[p, r0:r0 + x.shape[0]] = x.to(dtype)
                    x = x - out[p, r0:r0 + x.shape[0]].float()
        return out

    C = torch.empty((case["M"], case["N"]), dtype=torch.float64 if case["precision"] == "fp64" else torch.float32,
                    device="cuda")
    return {"case": case, "A": operand(case["M"]), "B": operand(case["N"]), "C": C}


# --------------------------------------------------------------------- run ---
def _tensors(ctx, case):
    dtype = np.float64 if case["precision"] == "fp64" else np.float32
    return [ctx.tensor(w).astype(dtype, copy=False) for w in range(1 + len(case.get("impure", "")))]


def _records(ctx):
    """ln c_n and the discarded weights of every step."""
    log = ctx.step_log()
    return {"ln_c": np.array([r.ln_c for r in log]), "eps": np.array([r.eps for r in log])}


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "join":
        A, B, C = state["A"], state["B"], state["C"]
        M, N, K = case["M"], case["N"], case["K"]
        trg.trg_gemm(case["precision"], A.data_ptr(), B.data_ptr(), C.data_ptr(), M, N, K, K, K, N, False,
                     torch.cuda.current_stream().cuda_stream)
        return C
    if kind == "solve":
        ctx = _context(case, state["seed"])
        ctx.run(case["L"])
        out = {"f": ctx.free_energy(), "log": _records(ctx)}
        if "E" in case["impure"]:
            out["E"] = ctx.impure_energy()
        if "M" in case["impure"]:
            out["M"] = ctx.impure_magnetization()
        ctx.close()
        return out
    ctxs, d = state["ctxs"], case.get("d", 4)
    if kind == "observables":
        c = ctxs[0]
        return [c.free_energy(), c.impure_energy(), c.impure_magnetization()] + [c.indicator_x(a) for a in range(d)]
    for _ in range(case["steps"]):
        axis = state["n"] % d
        state["n"] += 1
        if kind == "batch":
            trg.trg_hotrg_step_batch(ctxs, axis, case["dcut"])
        elif case["method"] == "atrg":
            ctxs[0].atrg_step(axis, case["dcut"])
        else:
            ctxs[0].hotrg_step(axis, case["dcut"])
    if case.get("method") == "atrg":
        c = ctxs[0]
        out = {"f": c.free_energy(), "sigma": c.atrg_spectrum().copy(), "GH": [np.abs(x) for x in c.factors()]}
        if case["impure"]:
            out["E"] = c.impure_energy()
        return out
    return {"f": [c.free_energy() for c in ctxs], "T": [t for c in ctxs for t in _tensors(c, case)]}


# -------------------------------------------------------------------- work ---
def _dims_flow(d, dcut, steps, start=0):
    """Leg dimensions before each of `steps` steps, the first being number `start`."""
    dims, out = [2] * d, []
    for n in range(start + steps):
        if n >= start:
            out.append((n % d, list(dims)))
        dims = [x if a == n % d else min(x * x, dcut) for a, x in enumerate(dims)]
    return out, dims


def _hotrg_work(d, dcut, steps, start, nimp):
    flops = nbytes = 0.0
    flow, _ = _dims_flow(d, dcut, steps, start)
    for mu, dims in flow:
        others = [a for a in range(d) if a != mu]
        pre, post = others[:(len(others) + 1) // 2], others[(len(others) + 1) // 2:]
        new = {a: min(dims[a] ** 2, dcut) for a in others}
        m = dims[mu] * math.prod(dims[a] ** 2 for a in post) * math.prod(new[a] for a in pre)
        k = dims[mu] * math.prod(dims[a] ** 2 for a in pre)
        flops += 2.0 * m * m * k * (1 + 2 * nimp)
        size_old = math.prod(x * x for x in dims)
        size_new = dims[mu] ** 2 * math.prod(new[a] ** 2 for a in others)
        nbytes += 8.0 * (size_old + size_new) * (1 + nimp)
    return flops, nbytes


def work(case):
    kind = case["kind"]
    if kind == "join":
        planes, dtype = PLANES[case["precision"]]
        el = planes * torch.empty(0, dtype=dtype).element_size()
        M, N, K = case["M"], case["N"], case["K"]
        return {"bytes": float((M + N) * K * el + M * N * (8 if case["precision"] == "fp64" else 4)),
                "flops": 2.0 * M * N * K}
    d, D = case.get("d", 4), case["dcut"]
    if kind == "observables":
        # the diagonals that the four traces read, three tensors, and the open legs of X
        n = float(min(D, 2 ** _ramp(d))) ** d
        return {"bytes": 8.0 * n * (3 + d * D), "flops": n * (3 + d * D)}
    if kind == "solve":
        flops, nbytes = _hotrg_work(d, D, d * int(math.log2(case["L"])), 0, len(case["impure"]))
        return {"bytes": nbytes, "flops": flops}
    if case.get("method") == "atrg":
        # per swap: 2 q + 2 products of 4 D^{d+2} r flops each and their
        # orthonormalisations; two contractions of 2 D^{2d+1} each; pieces read and written
        q, r = case.get("rsvd_q", 2 * D), D + case.get("rsvd_p", 4 * D)
        terms = 1 + 2 * len(case["impure"])
        swap = (2 * q + 2) * (4.0 * D ** (d + 2) * r + 2.0 * D ** d * r * r)
        return {"bytes": 8.0 * 4 * D ** (d + 1) * terms * case["steps"],
                "flops": terms * (swap + 4.0 * D ** (2 * d + 1)) * case["steps"]}
    flops, nbytes = _hotrg_work(d, D, case["steps"], _ramp(d), len(case.get("impure", "")))
    n = case.get("runs", 1)
    return {"bytes": nbytes * n, "flops": flops * n}


# ------------------------------------------------------------------- exact ---
# HOTRG in plain torch FP64 on named axes, written from the definition: the
# two-site environments of every transverse axis, their leading eigenvectors
# (degenerate eigenspaces in the basis of their projector), the block-spin
# contraction, the norm.
def _ising(d, beta, h):
    n = np.zeros((2,) * (2 * d), dtype=np.int64)
    for ax in range(2 * d):
        n += np.arange(2).reshape([2 if a == ax else 1 for a in range(2 * d)])
    ch, sh = math.cosh(beta), math.sinh(beta)
    base = 2.0 * ch ** (0.5 * (2 * d - n)) * sh ** (0.5 * n)
    g = np.where(n % 2 == 0, math.cosh(beta * h), math.sinh(beta * h))
    gp = np.where(n % 2 == 0, math.sinh(beta * h), math.cosh(beta * h))
    slope = 0.5 * (2 * d - n) * math.tanh(beta) + 0.5 * n / math.tanh(beta)
    return base * g, base * (slope * g + h * gp), base * gp


def _environment(T, l1, l2):
    X = torch.movedim(T, (l1, l2), (0, 1))
    n1, n2 = X.shape[0], X.shape[1]
    X = X.reshape(n1 * n2, -1)
    return (X @ X.T).reshape(n1, n2, n1, n2)


def _isometry(T, mu, nu, k, window):
    sides = []
    for side in (0, 1):
        P, Q = _environment(T, 2 * mu + 1, 2 * nu + side), _environment(T, 2 * mu, 2 * nu + side)
        i, a = P.shape[0], P.shape[1]
        G = P.permute(1, 3, 0, 2).reshape(a * a, i * i) @ Q.permute(0, 2, 1, 3).reshape(i * i, a * a)
        G = G.reshape(a, a, a, a).permute(0, 2, 1, 3).reshape(a * a, a * a).cpu().numpy()
        w, v = np.linalg.eigh(0.5 * (G + G.T))
        w, v = w[::-1], v[:, ::-1]
        sides.append((np.maximum(w[k:], 0.0).sum(), w, v))
    eps = [x[0] for x in sides]
    _, w, v = sides[0] if sides[0][0] < (1.0 - 1e-10) * sides[1][0] else sides[1]
    U, lo, n = np.zeros((len(w), k)), 0, len(w)
    while lo < k:
        hi = lo + 1
        while hi < n and w[hi - 1] - w[hi] <= window * max(w[0], 0.0):
            hi += 1
        Pr = v[:, lo:hi] @ v[:, lo:hi].T
        for j in range(lo, min(hi, k)):
            dg = np.diag(Pr)
            r = int(np.nonzero(dg >= (1.0 - 1e-9) * dg.max())[0][0])
            U[:, j] = Pr[:, r] / math.sqrt(Pr[r, r])
            Pr = Pr - np.outer(U[:, j], U[:, j])
        lo = hi
    a = T.shape[2 * nu]
    return torch.from_numpy(U).to(T.device).reshape(a, a, k), eps


def _contract(X1, X2, mu, U):
    """sum over the joined leg of X1 (forward mu) and X2 (backward mu), every
    transverse pair compressed by its isometry."""
    d = X1.ndim // 2
    others = [a for a in range(d) if a != mu]
    pre, post = others[:(len(others) + 1) // 2], others[(len(others) + 1) // 2:]
    # axes by name: site 1 (o, i, a_nu, A_nu), site 2 (i, p, b_nu, B_nu); capitals are forward legs
    n1 = [("o", "i") if a == mu else ("a%d" % a, "A%d" % a) for a in range(d)]
    n2 = [("i", "p") if a == mu else ("b%d" % a, "B%d" % a) for a in range(d)]
    n1, n2 = [x for y in n1 for x in y], [x for y in n2 for x in y]

    def times(X, names, u, unames, over):
        X = torch.tensordot(X, u, ([names.index(x) for x in over], [unames.index(x) for x in over]))
        return X, [x for x in names if x not in over] + [x for x in unames if x not in over]

    for s in pre:
        X1, n1 = times(X1, n1, U[s], ["a%d" % s, "b%d" % s, "K%d" % s], ["a%d" % s])
        X2, n2 = times(X2, n2, U[s], ["A%d" % s, "B%d" % s, "L%d" % s], ["B%d" % s])
    X1, n1 = times(X1, n1, X2, n2, [x for x in n1 if x in n2])
    for r in post:
        X1, n1 = times(X1, n1, U[r], ["a%d" % r, "b%d" % r, "K%d" % r], ["a%d" % r, "b%d" % r])
        X1, n1 = times(X1, n1, U[r], ["A%d" % r, "B%d" % r, "L%d" % r], ["A%d" % r, "B%d" % r])
    order = [x for a in range(d) for x in (("o", "p") if a == mu else ("K%d" % a, "L%d" % a))]
    return X1.permute([n1.index(x) for x in order]).contiguous()


def _ref_run(case, seed, steps, i=0):
    """(tensors, ln Z/V, [(ln c_n, discarded weights)]) after `steps` steps of the i-th run of the case."""
    d, D, impure = case.get("d", 4), case["dcut"], case.get("impure", "")
    mixed = case.get("precision", "fp64") != "fp64"
    beta, h = _coupling(case, seed, i)
    T, SE, SM = (torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in _ising(d, beta, h))
    ts = [T] + [{"E": SE, "M": SM}[x] for x in impure]
    c = float(ts[0].norm())
    ts, acc, log = [t / c for t in ts], math.log(c), []
    for n in range(steps):
        mu, T = n % d, ts[0]
        window = 1e-6 if mixed and n else 1e-10
        U, eps = {}, np.zeros((d, 2))
        for a in range(d):
            if a != mu:
                U[a], eps[a] = _isometry(T, mu, a, min(T.shape[2 * a] ** 2, D), window)
        new = [_contract(T, T, mu, U)] + [0.5 * (_contract(S, T, mu, U) + _contract(T, S, mu, U)) for S in ts[1:]]
        c = float(new[0].norm())
        ts = [t / c for t in new]
        acc += 2.0 ** -(n + 1) * math.log(c)
        log.append((math.log(c), eps))
    return ts, acc + 2.0 ** -steps * math.log(_trace(ts[0])), log


def _partial(T, axis):
    for a in reversed(range(T.ndim // 2)):
        if a != axis:
            T = torch.diagonal(T, 0, 2 * a, 2 * a + 1).sum(-1)
    return T


def _trace(T):
    return float(torch.trace(_partial(T, 0)))


def exact(case, seed):
    kind = case["kind"]
    if kind == "join":
        s = _prepare_join(case, seed)
        A, B = (sum(s[x][p].double() for p in range(s[x].shape[0])) for x in ("A", "B"))
        return A @ B.T
    if case.get("method") == "atrg":
        return None  # a randomised algorithm with its own trial matrices: minutes in plain numpy
    d = case.get("d", 4)
    if kind == "observables":
        (T, SE, SM), f, _ = _ref_run(dict(case, impure="EM"), seed, _ramp(d))
        out = [f, -_trace(SE) / _trace(T), _trace(SM) / _trace(T)]
        for a in range(d):
            M = _partial(T, a)
            out.append(float(torch.trace(M) ** 2 / torch.trace(M @ M)))
        return out
    if kind == "solve":
        ts, f, log = _ref_run(case, seed, d * int(math.log2(case["L"])))
        out = {"f": f, "log": {"ln_c": np.array([x for x, _ in log]), "eps": np.array([x for _, x in log])}}
        for x, S in zip(case["impure"], ts[1:]):
            out[x] = (-1.0 if x == "E" else 1.0) * _trace(S) / _trace(ts[0])
        return out
    runs = [_ref_run(case, seed, _ramp(d) + case["steps"], i) for i in range(case.get("runs", 1))]
    # the basis of a mixed step's tensor hangs on the rounding of its joins: no value for it
    mixed = case["precision"] != "fp64"
    return {"f": [r[1] for r in runs], "T": [None if mixed else t for r in runs for t in r[0]]}
