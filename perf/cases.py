"""Performance cases: what a user of the library has it do, at the sizes the
repository's own workloads, tests and benchmark use.

A case is a dict of plain values. `prepare` makes the inputs on the GPU from
a seed, with the handles a user's program keeps (the matrix, its tuned
kernels, the polynomial); `run` is one pass through the public entry points.
`exact` gives the same outputs in 64 bits from plain torch and numpy.

Kinds:
  apply  p(A)v or phi(A)v of a fixed root list (one chain of sparse products)
  setup  the polynomial of degree d from one GMRES(d) cycle
  solve  setup + PP-GMRES(m) solve of A x = b (the benchmark's time-to-solution)
  grad   x = A(vals)^-1 b and its gradients with respect to vals and b
  batch  many independent systems x several right-hand sides, setup + solve
Matrices:
  box2 / box3  convection-diffusion, 5- / 7-point stencil with constant coefficients
  var2         the 5-point stencil with every row scaled on its own (coefficients that vary in space)
  bihar        the 13-point biharmonic stencil plus u_xxx
  rand         k random off-diagonal columns per row, diagonally dominant
"""

import math

import numpy as np
import torch

import paper_1911_07065_amd as pp
from workloads import CSR

DTYPES = {"fp64": torch.float64, "fp32": torch.float32, "bf16": torch.bfloat16}


def listed():
    return [
        # the smallest system the tests and the smoke run use: every launch counts
        {"name": "apply_box2_50_fp64", "kind": "apply", "matrix": "box2", "nx": 50, "ny": 50, "nz": 1, "conv": 1.0,
         "op": "phi", "d": 25, "pairs": 3, "dtype": "fp64"},
        # one preconditioner application on the grid of the differentiable 2-D workload
        {"name": "apply_box2_1024_fp64", "kind": "apply", "matrix": "box2", "nx": 1024, "ny": 1024, "nz": 1,
         "conv": 20.0, "op": "phi", "d": 50, "pairs": 0, "dtype": "fp64"},
        # the operator of the benchmark's inner cycles: phi(A)v at 128^3, degree 40, FP32
        {"name": "apply_box3_128_fp32", "kind": "apply", "matrix": "box3", "nx": 128, "ny": 128, "nz": 128,
         "conv": 10.0, "op": "phi", "d": 40, "pairs": 2, "dtype": "fp32"},
        # the solution update p(A)y in FP64 on a box with odd, unequal sides
        {"name": "apply_box3_odd_fp64", "kind": "apply", "matrix": "box3", "nx": 201, "ny": 150, "nz": 97,
         "conv": 5.0, "op": "p", "d": 40, "pairs": 2, "dtype": "fp64"},
        # the biharmonic example at its full size and degree
        {"name": "apply_bihar_200_fp64", "kind": "apply", "matrix": "bihar", "nx": 200, "ny": 200, "nz": 1,
         "conv": 1.0, "op": "phi", "d": 200, "pairs": 0, "dtype": "fp64"},
        # the random sparse workload at its full size and degree, FP32 inner cycles
        {"name": "apply_rand_1e6_fp32", "kind": "apply", "matrix": "rand", "nx": 1000000, "ny": 1, "nz": 1, "k": 16,
         "conv": 0.0, "op": "phi", "d": 100, "pairs": 48, "dtype": "fp32"},
        # the reduced-storage form on a smaller scattered matrix
        {"name": "apply_rand_25e4_bf16", "kind": "apply", "matrix": "rand", "nx": 250007, "ny": 1, "nz": 1, "k": 16,
         "conv": 0.0, "op": "p", "d": 30, "pairs": 14, "dtype": "bf16"},
        # coefficients that vary in space: no constant stencil to exploit
        {"name": "apply_var2_600_fp64", "kind": "apply", "matrix": "var2", "nx": 600, "ny": 431, "nz": 1, "conv": 5.0,
         "op": "p", "d": 30, "pairs": 2, "dtype": "fp64"},
        # the polynomial of the benchmark's plain FP64 form
        {"name": "setup_box3_128_fp64", "kind": "setup", "matrix": "box3", "nx": 128, "ny": 128, "nz": 128,
         "conv": 10.0, "d": 40, "basis": "fp64"},
        # the benchmark's headline, solved to the tolerance that the differentiable solves ask for
        {"name": "solve_box3_128_fp32", "kind": "solve", "matrix": "box3", "nx": 128, "ny": 128, "nz": 128,
         "conv": 10.0, "d": 40, "m": 50, "basis": "fp32", "inner": "fp32", "tol": 1e-12},
        # differentiation through the solve: forward and adjoint
        {"name": "grad_box2_512_fp64", "kind": "grad", "matrix": "box2", "nx": 512, "ny": 512, "nz": 1, "conv": 20.0,
         "d": 50, "m": 50, "inner": "fp64", "tol": 1e-12},
        # many systems of different sizes in lockstep, several right-hand sides each
        {"name": "batch_48x4_fp32", "kind": "batch", "count": 48, "lo": 64, "hi": 256, "rhs": 4, "conv": 50.0, "d": 20,
         "m": 50, "inner": "fp32", "tol": 1e-12},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: the listed kinds and matrices, sizes over the listed ranges."""
    what = rng.choice(["box2", "box2", "box3", "box3", "bihar", "rand", "var2", "setup", "solve", "grad", "batch"])
    # FP32 stencil chains are drawn as phi(A)v, what FP32 cycles apply at every step
    dtype = rng.choice(["fp64", "fp32"])
    c = {"kind": "apply", "matrix": what, "ny": 1, "nz": 1, "conv": round(rng.uniform(0.0, 20.0), 3),
         "op": "phi" if dtype == "fp32" else rng.choice(["p", "phi"]), "pairs": rng.randint(0, 3), "dtype": dtype}
    if what == "box2":
        n = _log(rng, 24, 1024)
        return {**c, "nx": n, "ny": max(24, int(n * rng.uniform(0.6, 1.0))), "d": rng.randint(12, 60)}
    if what == "box3":
        s = [_log(rng, 20, 200) for _ in range(3)]
        while s[0] * s[1] * s[2] > 3_000_000:
            s = [max(20, int(0.9 * v)) for v in s]
        return {**c, "nx": s[0], "ny": s[1], "nz": s[2], "d": rng.randint(12, 48)}
    if what == "bihar":
        n = rng.randint(40, 200)
        return {**c, "nx": n, "ny": n, "d": rng.randint(40, 200), "dtype": "fp64"}
    if what == "rand":
        d = rng.randint(20, 100)
        return {**c, "nx": _log(rng, 20_000, 1_000_000), "k": rng.randint(6, 16), "d": d, "pairs": rng.randint(d // 3, d // 2),
                "dtype": rng.choice(["fp64", "fp32", "bf16"])}
    if what == "var2":
        return {**c, "nx": rng.randint(60, 700), "ny": rng.randint(60, 700), "d": rng.randint(12, 50)}
    if what == "setup":
        return {"kind": "setup", "matrix": "box3", "nx": rng.randint(30, 128), "ny": rng.randint(30, 128),
                "nz": rng.randint(30, 128), "conv": round(rng.uniform(5.0, 15.0), 3), "d": rng.randint(10, 40), "basis": "fp64"}
    if what == "solve":
        n = rng.randint(24, 128)
        return {"kind": "solve", "matrix": "box3", "nx": n, "ny": rng.randint(24, n), "nz": rng.randint(24, n),
                "conv": round(rng.uniform(5.0, 15.0), 3), "d": rng.randint(15, 40), "m": 50, "basis": "fp32", "inner": "fp32",
                "tol": 1e-12}
    if what == "grad":
        n = rng.randint(48, 512)
        return {"kind": "grad", "matrix": "box2", "nx": n, "ny": n, "nz": 1, "conv": round(rng.uniform(10.0, 30.0), 3),
                "d": rng.randint(30, 50), "m": 50, "inner": "fp64", "tol": 1e-12}
    return {"kind": "batch", "count": _log(rng, 4, 48), "lo": 64, "hi": rng.randint(80, 256), "rhs": rng.choice([1, 2, 4]),
            "conv": 50.0, "d": rng.randint(12, 20), "m": 50, "inner": "fp32", "tol": 1e-12}


# ---------------------------------------------------------------------------
# matrices, roots and vectors
# ---------------------------------------------------------------------------

def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _normal(g, *shape):
    return torch.randn(*shape, generator=g, dtype=torch.float64, device="cuda")


def _coef(case, seed, axes):
    """Convection coefficient per axis: the case's value within a tenth, from the seed."""
    r = np.random.default_rng(seed)
    return [case["conv"] * float(r.uniform(0.9, 1.1)) for _ in range(axes)]


def _pack(cols, vals, keep):
    counts = keep.sum(dim=1)
    rowptr = torch.zeros(cols.shape[0] + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(counts, 0, out=rowptr[1:])
    return rowptr.to(torch.int32), cols[keep].to(torch.int32), vals.expand(cols.shape)[keep].contiguous()


def _axis(m, c):
    """(lower, upper) neighbour of one axis: -u'' + c u', scaled by h^2."""
    h = 1.0 / (m + 1)
    return -1.0 - 0.5 * c * h, -1.0 + 0.5 * c * h


def _csr(case, seed):
    """(rowptr, colind, val) of the case's matrix on the GPU, columns ascending."""
    nx, ny, nz = case["nx"], case["ny"], case["nz"]
    n = nx * ny * nz
    i = torch.arange(n, device="cuda")
    m = case["matrix"]
    if m in ("box2", "box3", "var2"):
        sides = [nx, ny, nz][: 3 if m == "box3" else 2]
        coef = _coef(case, seed, len(sides))
        slots, stride = [(0, 2.0 * len(sides), torch.ones(n, dtype=torch.bool, device="cuda"))], 1
        for s, c in zip(sides, coef):
            lo, up = _axis(s, c)
            at = (i // stride) % s
            slots += [(-stride, lo, at > 0), (stride, up, at < s - 1)]
            stride *= s
        slots.sort(key=lambda t: t[0])
        cols = torch.stack([i + t[0] for t in slots], dim=1)
        vals = torch.tensor([t[1] for t in slots], dtype=torch.float64, device="cuda")[None, :]
        if m == "var2":
            vals = vals * (0.5 + 0.5 * torch.rand(n, 1, generator=_gen(seed + 77), dtype=torch.float64, device="cuda"))
        return _pack(cols, vals, torch.stack([t[2] for t in slots], dim=1))
    if m == "bihar":
        h = _coef(case, seed, 1)[0] / (nx + 1)
        st = {(0, 0): -20.0}
        for a, b in ((1, 0), (-1, 0), (0, 1), (0, -1)):
            st[a, b], st[2 * a, 2 * b] = 8.0, -1.0
        for a in (1, -1):
            for b in (1, -1):
                st[a, b] = -2.0
        for a, v in ((-2, -0.5), (-1, 1.0), (1, -1.0), (2, 0.5)):
            st[a, 0] += h * v
        x, y = i % nx, i // nx
        slots = sorted((b * nx + a, v, a, b) for (a, b), v in st.items())
        cols = torch.stack([i + t[0] for t in slots], dim=1)
        keep = torch.stack([(x + t[2] >= 0) & (x + t[2] < nx) & (y + t[3] >= 0) & (y + t[3] < ny) for t in slots], dim=1)
        return _pack(cols, torch.tensor([t[1] for t in slots], dtype=torch.float64, device="cuda")[None, :], keep)
    # rand: one column in each of k equal parts of [0, n), never the diagonal
    k, g = case["k"], _gen(seed + 77)
    w = n // k
    off = (torch.rand(n, k, generator=g, device="cuda", dtype=torch.float64) * w).long().clamp_(max=w - 1)
    cols = off + torch.arange(k, device="cuda")[None, :] * w
    cols = torch.where(cols == i[:, None], torch.where(off > 0, cols - 1, cols + 1), cols)
    vals = _normal(g, n, k)
    cols = torch.cat([cols, i[:, None]], dim=1)
    vals = torch.cat([vals, 1.05 * vals.abs().sum(dim=1, keepdim=True)], dim=1)
    cols, at = torch.sort(cols, dim=1)
    rowptr = torch.arange(n + 1, device="cuda", dtype=torch.int64) * (k + 1)
    return rowptr.to(torch.int32), cols.reshape(-1).to(torch.int32), torch.gather(vals, 1, at).reshape(-1).contiguous()


def _roots(case):
    """d roots over the matrix's spectrum: Chebyshev points of its interval with
    a little room above (or a circle's around a scattered matrix's spectrum),
    the last `pairs` * 2 of them joined into conjugate pairs."""
    d, pairs = case["d"], case["pairs"]
    if case["matrix"] == "rand":
        mean = 1.05 * case["k"] * math.sqrt(2.0 / math.pi)
        rad = 1.3 * math.sqrt(case["k"])
        t = (np.arange(pairs) + 0.5) * math.pi / pairs
        up = mean + rad * np.exp(1j * t)
        real = mean + rad * np.linspace(-0.8, 0.8, d - 2 * pairs) if d > 2 * pairs else np.zeros(0)
        return np.concatenate([real.astype(complex), np.stack([up, up.conj()], axis=1).reshape(-1)])
    hi = 1.05 * {"box2": 8.0, "var2": 8.0, "box3": 12.0, "bihar": -64.0}[case["matrix"]]
    lo = 4.0 * hi / (d * d)
    x = 0.5 * (hi + lo) - 0.5 * (hi - lo) * np.cos((np.arange(d) + 0.5) * math.pi / d)
    r = x.astype(complex)
    for p in range(min(pairs, d // 2)):
        a, b = x[d - 2 * p - 2], x[d - 2 * p - 1]
        r[d - 2 * p - 2] = complex(0.5 * (a + b), 0.5 * abs(b - a))
        r[d - 2 * p - 1] = r[d - 2 * p - 2].conjugate()
    return r


def _vector(case, seed):
    n = case["nx"] * case["ny"] * case["nz"]
    return _normal(_gen(seed), n)


def _systems(case, seed):
    """(side, convection coefficient) of each system of a batch: the sides are
    the case's (one per system, spread over its range), the coefficients the seed's."""
    count, r = case["count"], np.random.default_rng(seed)
    sides = np.random.default_rng(count).permutation(np.linspace(case["lo"], case["hi"], count).round().astype(int))
    return [(int(s), float(a)) for s, a in zip(sides, r.uniform(0.0, case["conv"], count))]


def prepare(case, seed):
    if case["kind"] == "batch":
        systems = _systems(case, seed)
        csrs = []
        for s, a in systems:
            rp, ci, va = _csr({"matrix": "box2", "nx": s, "ny": s, "nz": 1, "conv": 0.0}, 0)
            # convection along x, as in the batched workload
            rows = torch.repeat_interleave(torch.arange(s * s, device="cuda"), (rp[1:] - rp[:-1]).long())
            step = ci.long() - rows
            lo, up = _axis(s, a)
            va[step == -1], va[step == 1] = lo, up
            csrs.append(CSR(s * s, rp.cpu().numpy(), ci.cpu().numpy(), va.cpu().numpy()))
        B = pp.Batch(csrs)
        g = _gen(seed)
        b = B.interleave(_normal(g, case["rhs"], B.n) / math.sqrt(B.n))
        v0 = _normal(g, B.n)
        for prec in ("fp32", "fp64"):
            B.tune(case["rhs"], prec)
        return {"case": case, "B": B, "b": b, "v0": v0}
    rp, ci, va = _csr(case, seed)
    M = pp.Matrix(rp, ci, va)
    v = _vector(case, seed)
    s = {"case": case, "M": M}
    if case["kind"] == "apply":
        M.tune(case["dtype"])
        s.update(v=v.to(DTYPES[case["dtype"]]), poly=pp.poly_from_roots(_roots(case)))
        s["out"] = torch.empty_like(s["v"])
    elif case["kind"] == "setup":
        M.tune(case["basis"])
        s.update(v0=v)
    elif case["kind"] == "solve":
        for prec in {case["basis"], case["inner"], "fp64"}:
            M.tune(prec)
        s.update(v0=_normal(_gen(seed + 1), v.numel()), b=v / torch.linalg.norm(v))
    else:
        M.tune(case["inner"])
        s.update(poly=pp.setup(M, _normal(_gen(seed + 1), v.numel()), case["d"]),
                 vals=va.clone().requires_grad_(True), b=(v / torch.linalg.norm(v)).requires_grad_(True),
                 target=_normal(_gen(seed + 2), v.numel()))
    return s


def run(state):
    case = state["case"]
    if case["kind"] == "apply":
        return pp.apply(state["poly"], state["M"], state["v"], case["op"], out=state["out"])
    if case["kind"] == "setup":
        return pp.setup(state["M"], state["v0"], case["d"], basis=case["basis"]).roots("leja")
    if case["kind"] == "solve":
        poly = pp.setup(state["M"], state["v0"], case["d"], basis=case["basis"])
        x, _ = pp.solve(poly, state["M"], state["b"], tol=case["tol"], m=case["m"], inner=case["inner"])
        return x
    if case["kind"] == "grad":
        x = pp.pp_solve_fn(state["vals"], state["b"], state["M"], state["poly"], tol=case["tol"], m=case["m"],
                           inner=case["inner"])
        dvals, db = torch.autograd.grad(0.5 * torch.sum((x - state["target"]) ** 2), (state["vals"], state["b"]))
        return {"x": x.detach(), "dvals": dvals, "db": db}
    polys = state["B"].setup(state["v0"], case["d"])
    x, _ = state["B"].solve(polys, state["b"], case["rhs"], tol=case["tol"], m=case["m"], inner=case["inner"])
    return x


def work(case):
    """Bytes: the matrix (values and column indices as the caller gives them)
    and the input vectors read once, the outputs written once. Operations: the
    sparse products and updates that the degree asks for; for the solves one
    application of phi and p, the least a preconditioned solve can do."""
    if case["kind"] == "batch":
        n = sum(s * s for s, _ in _systems(case, 0))
        nnz, R, d = 5 * n, case["rhs"], case["d"]
        return {"bytes": 12 * nnz + 4 * n + 8 * n + 16 * n * R, "flops": 2 * d * (2 * nnz + 3 * n) * (R + 1)}
    n = case["nx"] * case["ny"] * case["nz"]
    per = {"box2": 5, "var2": 5, "box3": 7, "bihar": 13, "rand": case.get("k", 0) + 1}[case["matrix"]]
    nnz, d = n * per, case["d"]
    matrix, chain = 12 * nnz + 4 * n, d * (2 * nnz + 3 * n)
    if case["kind"] == "apply":
        return {"bytes": matrix + 2 * n * DTYPES[case["dtype"]].itemsize, "flops": chain}
    if case["kind"] == "setup":
        return {"bytes": matrix + 8 * n, "flops": d * 2 * nnz + 2 * n * d * d}
    if case["kind"] == "solve":
        return {"bytes": matrix + 24 * n, "flops": d * 2 * nnz + 2 * n * d * d + 2 * chain}
    return {"bytes": matrix + 8 * nnz + 32 * n, "flops": 4 * chain}


# ---------------------------------------------------------------------------
# the same in 64 bits, without the library
# ---------------------------------------------------------------------------

def _leja(r):
    """Units (real roots and +imag members of pairs) in Leja order."""
    u = np.array(sorted((z for z in r if z.imag >= 0), key=lambda z: (z.real, z.imag)))
    out, logs = [], np.zeros(u.size)
    left = np.ones(u.size, dtype=bool)
    k = int(np.argmax(np.abs(u)))
    for _ in range(u.size):
        out.append(u[k])
        left[k] = False
        with np.errstate(divide="ignore"):
            logs += np.log(np.abs(u - u[k]))
            if u[k].imag != 0:
                logs += np.log(np.abs(u - np.conj(u[k])))
        if left.any():
            k = int(np.argmax(np.where(left, logs, -np.inf)))
    return out


def _product(case, seed):
    rp, ci, va = _csr(case, seed)
    n = rp.numel() - 1
    A = torch.sparse_csr_tensor(rp.long(), ci.long(), va, size=(n, n))
    return lambda x: (A @ x[:, None])[:, 0]


def _sine(m, c, transpose):
    """T = W diag(lam) V of one axis of the stencil, W V = I."""
    lo, up = _axis(m, c)
    if transpose:
        lo, up = up, lo
    i = torch.arange(1, m + 1, dtype=torch.float64, device="cuda")
    Q = math.sqrt(2.0 / (m + 1)) * torch.sin(math.pi / (m + 1) * i[:, None] * i[None, :])
    g = (lo / up) ** (0.5 * (i - 0.5 * (m + 1)))
    lam = 2.0 - 2.0 * math.sqrt(lo * up) * torch.cos(math.pi / (m + 1) * i)
    return g[:, None] * Q, Q / g[None, :], lam


def _box_product(sides, coef, transpose):
    """The constant-coefficient box stencil (or its transpose) on a grid."""
    pairs = [_axis(m, c) for m, c in zip(sides, coef)]
    shape = list(reversed(sides))

    def product(x):
        x = x.reshape(shape)
        y = 2.0 * len(sides) * x
        for k, (lo, up) in enumerate(pairs):
            if transpose:
                lo, up = up, lo
            dim, m = len(sides) - 1 - k, sides[k]
            y.narrow(dim, 1, m - 1).add_(x.narrow(dim, 0, m - 1), alpha=lo)
            y.narrow(dim, 0, m - 1).add_(x.narrow(dim, 1, m - 1), alpha=up)
        return y.reshape(-1)

    return product


def _box_solve(sides, coef, b, transpose=False):
    """The solution of a constant-coefficient box stencil's system (or its
    transpose's) by sine transforms along every axis, refined."""
    ax = [_sine(m, c, transpose) for m, c in zip(sides, coef)]
    shape = list(reversed(sides))
    lam = 0.0
    for k, (_, _, l) in enumerate(ax):
        lam = lam + l.reshape([-1 if j == len(sides) - 1 - k else 1 for j in range(len(sides))])

    def along(t, k, W):
        dim = len(sides) - 1 - k
        return torch.movedim(torch.tensordot(W, t, dims=([1], [dim])), 0, dim)

    def solve(r):
        t = r.reshape(shape)
        for k, (_, V, _) in enumerate(ax):
            t = along(t, k, V)
        t = t / lam
        for k, (W, _, _) in enumerate(ax):
            t = along(t, k, W)
        return t.reshape(-1)

    product, x = _box_product(sides, coef, transpose), solve(b)
    for _ in range(4):
        x = x + solve(b - product(x))
    return x


def exact(case, seed):
    kind = case["kind"]
    if kind == "batch":
        R, systems = case["rhs"], _systems(case, seed)
        b = _normal(_gen(seed), R, sum(s * s for s, _ in systems))
        b = b / math.sqrt(b.shape[1])
        out, at = torch.empty_like(b), 0
        for s, a in systems:
            for r in range(R):
                out[r, at: at + s * s] = _box_solve([s, s], [a, 0.0], b[r, at: at + s * s])
            at += s * s
        return out.t().contiguous().reshape(-1)
    A, v = _product(case, seed), _vector(case, seed)
    if kind == "apply":
        v = v.to(DTYPES[case["dtype"]]).double()
        prod, p = v.clone(), torch.zeros_like(v)
        for z in _leja(_roots(case)):
            if z.imag == 0:
                p += prod / z.real
                prod = prod - A(prod) / z.real
            else:
                t = (2.0 * z.real * prod - A(prod)) / (z.real ** 2 + z.imag ** 2)
                p += t
                prod = prod - A(t)
        return p if case["op"] == "p" else v - prod
    if kind == "setup":
        d = case["d"]
        H, V = np.zeros((d + 1, d)), torch.zeros(d + 1, v.numel(), dtype=torch.float64, device="cuda")
        V[0] = v / torch.linalg.norm(v)
        for j in range(d):
            w = A(V[j])
            for _ in range(2):
                h = V[: j + 1] @ w
                w = w - h @ V[: j + 1]
                H[: j + 1, j] += h.cpu().numpy()
            H[j + 1, j] = float(torch.linalg.norm(w))
            V[j + 1] = w / H[j + 1, j]
        f = np.linalg.solve(H[:d].T, np.eye(d)[:, -1])
        G = H[:d].copy()
        G[:, -1] += H[d, d - 1] ** 2 * f
        out = []
        for z in _leja(np.linalg.eigvals(G)):
            out += [z] if z.imag == 0 else [z, z.conjugate()]
        return np.array(out, dtype=complex)
    sides = [case["nx"], case["ny"], case["nz"]][: 3 if case["matrix"] == "box3" else 2]
    coef = _coef(case, seed, len(sides))
    b = v / torch.linalg.norm(v)
    x = _box_solve(sides, coef, b)
    if kind == "solve":
        return x
    rp, ci, va = _csr(case, seed)
    rows = torch.repeat_interleave(torch.arange(v.numel(), device="cuda"), (rp[1:] - rp[:-1]).long())
    lam = _box_solve(sides, coef, x - _normal(_gen(seed + 2), v.numel()), transpose=True)
    return {"x": x, "dvals": -lam[rows] * x[ci.long()], "db": lam}
