"""The work a user of the library has it do, as timed cases.

A case names one call (or one solve) through the binding, with its sizes:

* ``filter``: one Chebyshev filter pass, ``chfsi_filter`` -- the path's hot
  loop -- on a dense, complex Hermitian, grid, Bloch grid or CSR operator, in
  FP64, FP32 or BF16, by the residual filter (Algorithm 3) or, in FP64, the
  plain one (Algorithm 2);
* ``rr``: one Rayleigh-Ritz step on a filtered block, ``chfsi_rayleigh_ritz``;
* ``solve``: a full eigensolve from a random start, ``chfsi_solve``.

Inputs are what such a call meets inside a solve.  Dense and Hermitian states
are Ritz pairs and residuals of a few passes of a plain torch subspace
iteration (no library code): about half-way through a solve for FP64; for the reduced precisions the residuals of
the slowest columns are cut to the size that they have late in a solve, whose
last passes these are.
Grid states are blocks of well-centred orbitals (an LCAO start) with their
Rayleigh quotients and residuals, the residuals scaled to a late pass.
"""
import math

import numpy as np
import torch

import paper_2503_22652_amd as P
import workloads as wl
from workloads import gpu as wg

PREC = {"fp64": P.PREC_FP64, "fp32": P.PREC_FP32, "bf16": P.PREC_BF16}
F64 = torch.float64


def listed():
    return [
        # the benchmark's pencil: one FP32 filter pass, 256 wanted of 320
        dict(name="dense_fp32_8192x320", kind="filter", op="dense", prec="fp32", method="r",
             n=8192, b=320, degree=20),
        # the smallest pencil of the serving stream (k = 26 wanted): latency and launches
        dict(name="dense_fp32_512x48", kind="filter", op="dense", prec="fp32", method="r",
             n=512, b=48, degree=20),
        # a serving-stream size in BF16 products; its block (k = 205 wanted, 1.25 k rounded
        # up to 16) is no multiple of a large tile
        dict(name="dense_bf16_4096x272", kind="filter", op="dense", prec="bf16", method="r",
             n=4096, b=272, degree=20),
        # the plain filter, the FP64 baseline, at an odd size and block
        dict(name="dense_fp64_plain_3001x77", kind="filter", op="dense", prec="fp64", method="c",
             n=3001, b=77, degree=16),
        # a k-point problem in dense form, complex Hermitian, FP32 products
        dict(name="hermitian_fp32_2048x144", kind="filter", op="hermitian", prec="fp32",
             method="r", n=2048, b=144, degree=20),
        # the 128^3 grid pencil with BF16-stored blocks (a column panel of the benchmark's block)
        dict(name="grid_bf16_128x160", kind="filter", op="grid", prec="bf16", method="r",
             nx=128, ny=128, nz=128, b=160, degree=30),
        # a ragged grid, FP32
        dict(name="grid_fp32_60x52x44x33", kind="filter", op="grid", prec="fp32", method="r",
             nx=60, ny=52, nz=44, b=33, degree=20),
        # a grid pencil at a wave vector, BF16-stored blocks, 48 complex vectors
        dict(name="bloch_bf16_64x48", kind="filter", op="bloch", prec="bf16", method="r",
             nx=64, ny=64, nz=64, b=48, degree=30),
        # an assembled finite-element pencil in CSR form, FP32
        dict(name="csr_fp32_64x64", kind="filter", op="csr", prec="fp32", method="r",
             nx=64, ny=64, nz=64, b=64, degree=20),
        # the benchmark's Rayleigh-Ritz step (two thirds of a BF16 solve)
        dict(name="rr_dense_8192x320", kind="rr", op="dense", n=8192, b=320, degree=20),
        # Rayleigh-Ritz of a grid pencil: tall blocks, FP64 Gram products and rotation
        dict(name="rr_grid_64x300", kind="rr", op="grid", nx=64, ny=64, nz=64, b=300, degree=20),
        # one request of the serving stream: N = 1024, 5% wanted, FP32, cold start, to 1e-8
        dict(name="solve_dense_fp32_1024x80", kind="solve", op="dense", prec="fp32", n=1024, b=80,
             degree=20),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _grid(rng, lo, hi):
    return dict(nx=_log(rng, lo, hi), ny=_log(rng, lo, hi), nz=_log(rng, lo, hi))


def draw(rng):
    what = rng.choice(["dense", "dense", "dense", "plain", "hermitian", "grid", "grid", "bloch",
                       "csr", "rr_dense", "rr_grid", "solve"])
    prec = rng.choice(["fp64", "fp32", "fp32", "bf16", "bf16"])
    degree = rng.randint(16, 24)
    if what == "solve":
        n = _log(rng, 400, 2500)
        return dict(kind="solve", op="dense", prec=rng.choice(["fp32", "bf16", "fp64"]), n=n,
                    b=_block(n), degree=20)
    if what in ("dense", "plain", "rr_dense"):
        n = _log(rng, 400, 6000)
        b = max(8, min(384, int(n * rng.uniform(0.015, 0.07))))
        if what == "rr_dense":
            return dict(kind="rr", op="dense", n=n, b=b, degree=degree)
        if what == "plain":
            return dict(kind="filter", op="dense", prec="fp64", method="c", n=n, b=b, degree=degree)
        return dict(kind="filter", op="dense", prec=prec, method="r", n=n, b=b, degree=degree)
    if what == "hermitian":
        n = _log(rng, 300, 2600)
        return dict(kind="filter", op="hermitian", prec=prec, method="r", n=n,
                    b=max(6, int(n * rng.uniform(0.02, 0.06))), degree=degree)
    if what == "rr_grid":
        return dict(kind="rr", op="grid", b=rng.randint(40, 260), degree=degree, **_grid(rng, 32, 64))
    if what == "bloch":
        return dict(kind="filter", op="bloch", prec=prec, method="r", b=rng.randint(4, 40),
                    degree=degree, **_grid(rng, 20, 64))
    if what == "csr":
        return dict(kind="filter", op="csr", prec=prec, method="r", b=rng.randint(5, 64),
                    degree=degree, **_grid(rng, 20, 60))
    return dict(kind="filter", op="grid", prec=prec, method="r", b=rng.randint(8, 100),
                degree=degree, **_grid(rng, 24, 100))


def _block(n):
    """The serving stream's block: 5% wanted, 1.25 times that, rounded up to 16."""
    k = math.ceil(0.05 * n)
    return math.ceil(1.25 * k / 16) * 16


def _wanted(b):
    return max(1, int(0.8 * b))


# ---------------------------------------------------------------------------
# plain torch in 64 bits: operators, Rayleigh-Ritz, the two filters
# ---------------------------------------------------------------------------
def _filter_scalars(lmin, lmax, lT):
    e, c = (lmax - lT) / 2.0, (lmax + lT) / 2.0
    return e, c, e / (lmin - c)


def _residual_filter(op_A, d, X, lam, R, p, bounds):
    """Algorithm 3 on (rows, columns) blocks; d: D^{-1} as a column, or None."""
    e, c, s1 = _filter_scalars(*bounds)
    RX, RY = torch.zeros_like(R), (s1 / e) * R
    LX, LY = torch.ones_like(lam), (s1 / e) * (lam - c)
    s = s1
    for _ in range(2, p + 1):
        s2 = 1.0 / (2.0 / s1 - s)
        a, bb, cc = 2.0 * s2 / e, -2.0 * s2 * c / e, -s * s2
        new = op_A(RY if d is None else d * RY)
        new.mul_(a).add_(RY, alpha=bb).add_(RX, alpha=cc).add_(R * (a * LY))
        RX, RY = RY, new
        LX, LY = LY, a * LY * lam + bb * LY + cc * LX
        s = s2
    return (RY if d is None else d * RY) + X * LY


def _plain_filter(op_A, d, X, p, bounds):
    e, c, s1 = _filter_scalars(*bounds)
    V, W = X, (s1 / e) * (d * op_A(X) - c * X)
    s = s1
    for _ in range(2, p + 1):
        s2 = 1.0 / (2.0 / s1 - s)
        V, W = W, (2.0 * s2 / e) * (d * op_A(W) - c * W) - s * s2 * V
        s = s2
    return W


def _torch_rr(op_A, op_B, Y):
    """(Ritz values, Ritz vectors, residuals); each vector's sign makes its largest share of Y positive."""
    AY, BY = op_A(Y), op_B(Y)
    G = Y.mH @ BY
    s = torch.diagonal(G).real.rsqrt()
    G = s[:, None] * (G + G.mH) * s[None, :] / 2
    H = Y.mH @ AY
    H = s[:, None] * (H + H.mH) * s[None, :] / 2
    L = torch.linalg.cholesky(G)
    H = torch.linalg.solve_triangular(L, H, upper=False)
    H = torch.linalg.solve_triangular(L, H.mH, upper=False)
    w, E = np.linalg.eigh(((H + H.mH) / 2).cpu().numpy())   # small: faster on the host
    w, E = torch.from_numpy(w).to(Y.device), torch.from_numpy(E).to(Y.device)
    if not E.is_complex():
        E = E * torch.sign(E.gather(0, E.abs().argmax(0, keepdim=True)))
    T = s[:, None] * torch.linalg.solve_triangular(L.mH, E, upper=True)
    X = Y @ T
    return w, X, AY @ T - (BY @ T) * w


def _policy(lam, lmax, lT=None):
    """The library's own bounds: from the block's Ritz values, with lT given by the caller or their largest."""
    lo, hi = float(lam.min()), float(lam.max())
    return lo - 0.05 * (hi - lo), lmax, hi if lT is None else lT


def _col(X):
    """Column-major copy (the library's block layout)."""
    return X.mT.contiguous().mT


def _mass_1d(U, dim, ph):
    if ph is None:
        return (torch.roll(U, -1, dim) + torch.roll(U, 1, dim)).mul_(1 / 6).add_(U, alpha=2 / 3)
    return (torch.roll(U, -1, dim) * ph + torch.roll(U, 1, dim) * ph.conjugate()).mul_(1 / 6).add_(U, alpha=2 / 3)


def _grid_ops(shape, V, k):
    """A = 1/2 K + 1/2 (V M + M V) and B = M on (rows, columns) blocks, factor by
    factor: the 1D stiffness is 6 (1 - M1)."""
    nz, ny, nx = shape
    ph = [None if k is None else complex(math.cos(t), math.sin(t)) for t in (k or (0, 0, 0))]
    step = max(1, (1 << 31) // (8 * nx * ny * nz * (1 if k is None else 2)))

    def mass(U):
        return _mass_1d(_mass_1d(_mass_1d(U, 3, ph[0]), 2, ph[1]), 1, ph[2])

    def apply_A(U):
        ux = _mass_1d(U, 3, ph[0])
        kx = (U - ux).mul_(6)
        uxy = _mass_1d(ux, 2, ph[1])
        c = _mass_1d(kx, 2, ph[1]).add_((ux - uxy).mul_(6))
        m = _mass_1d(uxy, 1, ph[2])
        out = _mass_1d(c, 1, ph[2]).add_((uxy - m).mul_(6))
        return out.add_(V * m).add_(mass(V * U)).mul_(0.5)

    def on_columns(f):
        def g(X):
            Y = torch.empty_like(X.mT.contiguous())
            for j in range(0, X.shape[1], step):
                U = X[:, j:j + step].mT.reshape(-1, nz, ny, nx)
                Y[j:j + step] = f(U).reshape(U.shape[0], -1)
            return Y.mT
        return g

    return on_columns(apply_A), on_columns(mass)


# ---------------------------------------------------------------------------
# states
# ---------------------------------------------------------------------------
def _dense_pencil(case, seed):
    """A solve has guard columns beyond its wanted (low) eigenvalues; one pass on its own has a
    block that spans all the low ones, so that every column of a late state has converged."""
    n, cplx = case["n"], case["op"] == "hermitian"
    make = wg.hermitian_problem if cplx else wg.dense_problem
    A, B, dinv, _ = make(n, math.ceil(0.05 * n) if case["kind"] == "solve" else case["b"], seed)
    # a bound of the spectrum of B^{-1} A: largest of A over smallest of B (D >= 1/2, 5% off it)
    return A, B, dinv, 10.0 / (0.95 * 0.5) + 0.1


def _dense_state(case, seed, target, cut=math.inf):
    """Ritz pairs and residuals of a subspace iteration stopped at a max residual `target` or after
    eight passes; residuals longer than `cut` are scaled to that length.  The pencil has exactly b
    negative eigenvalues (those of A, by inertia), so lT = 0 once they are found."""
    A, B, dinv, lmax = _dense_pencil(case, seed)
    n, b = case["n"], case["b"]
    g = torch.Generator(device="cuda").manual_seed(int(seed) + 1)
    Y = torch.randn(n, b, dtype=A.dtype, device="cuda", generator=g)

    def op_A(X):
        return A @ X

    def op_B(X):
        return B @ X

    d = dinv[:, None]
    lam, X, R = _torch_rr(op_A, op_B, Y)
    for _ in range(8):
        if float(torch.linalg.vector_norm(R, dim=0).max()) < target:
            break
        Y = _residual_filter(op_A, d, X, lam, R, 20, _policy(lam, lmax, max(0.0, float(lam.max()))))
        lam, X, R = _torch_rr(op_A, op_B, Y)
    R = R * (cut / torch.linalg.vector_norm(R, dim=0)).clamp_(max=1.0)
    return dict(A=A, B=B, dinv=dinv, lmax=lmax, op_A=op_A, op_B=op_B, lam=lam, X=_col(X), R=_col(R),
                bounds=_policy(lam, lmax, max(0.0, float(lam.max()))))


K_BLOCH = (0.3, -0.7, 1.1)


def _grid_state(case, seed):
    """Orbitals (s, px, py, pz with their own widths along each axis) in Gaussian wells,
    sorted by their Rayleigh quotients, and their residuals at a late pass's size."""
    shape = (case["nz"], case["ny"], case["nx"])
    n, b = shape[0] * shape[1] * shape[2], case["b"]
    k = K_BLOCH if case["op"] == "bloch" else None
    wells = max(1, (b + 3) // 4)
    rng = np.random.default_rng(int(seed))
    centres = rng.uniform(0, 1, (wells, 3)) * np.array(shape[::-1])
    depth, width = rng.uniform(1, 5, wells), rng.uniform(2, 4, wells)
    axis_width = rng.uniform(1.2, 2.6, (wells, 3))
    ax = [torch.arange(m, dtype=F64, device="cuda") for m in shape[::-1]]

    def off(d, c):                       # signed periodic offset from a centre along axis d
        L = shape[::-1][d]
        return torch.remainder(ax[d] - c + L / 2, L) - L / 2

    V = torch.zeros(shape, dtype=F64, device="cuda")
    X = torch.empty((b, n), dtype=F64 if k is None else torch.complex128, device="cuda")
    for w in range(wells):
        g = [off(d, centres[w, d]) for d in range(3)]
        e = [torch.exp(-g[d] ** 2 / (2 * width[w] ** 2)) for d in range(3)]
        V -= depth[w] * e[2][:, None, None] * e[1][None, :, None] * e[0][None, None, :]
        s = [torch.exp(-g[d] ** 2 / (2 * axis_width[w, d] ** 2)) for d in range(3)]
        for o in range(min(4, b - 4 * w)):
            f = [s[d] * g[d] if o == d + 1 else s[d] for d in range(3)]
            X[4 * w + o] = (f[2][:, None, None] * f[1][None, :, None] * f[0][None, None, :]).reshape(-1)
    op_A, op_B = _grid_ops(shape, V, k)
    X = X.mT
    BX = op_B(X)
    s = (X.conj() * BX).sum(0).real.rsqrt()
    X, BX = X * s, BX * s
    AX = op_A(X)
    lam = (X.conj() * AX).sum(0).real
    lam, at = torch.sort(lam)
    X = _col(X[:, at])
    lmax = 23.0
    if case["kind"] == "rr":
        return dict(V=V, shape=shape, op_A=op_A, op_B=op_B, Y=X, lmax=lmax, k=k)
    AX = AX[:, at]
    BX = BX[:, at]
    R = _col((AX - BX * lam).mul_(1e-8 if case["prec"] == "bf16" else 1e-5))
    return dict(V=V, shape=shape, op_A=op_A, op_B=op_B, lam=lam, X=X, R=R, dinv=None, lmax=lmax,
                bounds=_policy(lam, lmax), k=k)


def _csr_of_grid(shape, V):
    """The grid pencil's A assembled: 27 entries a row, sorted by column."""
    nz, ny, nx = shape
    cA, cM = 0.5 * wl.tensor_stencil_27("stiffness"), wl.tensor_stencil_27("mass")
    idx = torch.arange(nz * ny * nx, device="cuda").reshape(shape)
    cols, vals = [], []
    for dz in (-1, 0, 1):
        for dy in (-1, 0, 1):
            for dx in (-1, 0, 1):
                sh = (-dz, -dy, -dx)
                cols.append(torch.roll(idx, sh, (0, 1, 2)).reshape(-1))
                v = float(cA[dz + 1, dy + 1, dx + 1]) + 0.5 * float(cM[dz + 1, dy + 1, dx + 1]) * (
                    V + torch.roll(V, sh, (0, 1, 2)))
                vals.append(v.reshape(-1))
    cols, at = torch.sort(torch.stack(cols, 1), 1)
    vals = torch.stack(vals, 1).gather(1, at)
    n = cols.shape[0]
    return (torch.arange(n + 1, dtype=torch.int64, device="cuda") * 27,
            cols.reshape(-1).to(torch.int32), vals.reshape(-1).contiguous())


def _state(case, seed):
    if case["op"] in ("dense", "hermitian"):
        if case["kind"] == "rr":
            s = _dense_state(case, seed, 1e-2)
            s["Y"] = _col(_residual_filter(s["op_A"], s["dinv"][:, None], s["X"], s["lam"], s["R"],
                                           case["degree"], s["bounds"]))
            return s
        if case.get("method") == "c":    # an early pass: a random block
            A, B, dinv, lmax = _dense_pencil(case, seed)
            g = torch.Generator(device="cuda").manual_seed(int(seed) + 1)
            X = torch.randn(case["b"], case["n"], dtype=F64, device="cuda", generator=g).mT
            return dict(A=A, B=B, dinv=dinv, lmax=lmax, op_A=lambda Z: A @ Z, X=X, lam=None, R=None,
                        bounds=(-2.2, lmax, 0.4))
        return _dense_state(case, seed, *{"fp64": (1e-2,), "fp32": (1e-4, 3e-4),
                                          "bf16": (1e-6, 1e-5)}[case["prec"]])
    return _grid_state(case, seed)


def _params(case, lmax, **more):
    return P.make_params(_wanted(case["b"]), case["b"], case["degree"], filter_prec=PREC[case.get("prec", "fp64")],
                         method=P.METHOD_CHFSI if case.get("method") == "c" else P.METHOD_RCHFSI,
                         lambda_max=lmax, **more)


def prepare(case, seed):
    if case["kind"] == "solve":
        A, B, dinv, _ = _dense_pencil(case, seed)
        prm = P.make_params(math.ceil(0.05 * case["n"]), case["b"], case["degree"], max_iter=60, tol=1e-8,
                            method=P.METHOD_RCHFSI, filter_prec=PREC[case["prec"]], seed=int(seed) % 100003,
                            init_random=1)
        ctx = P.chfsi_create(P.dense_operator(A), P.dense_operator(B), dinv, prm, keep=(A, B, dinv))
        return dict(kind="solve", ctx=ctx, X=P.colmajor_empty(case["n"], case["b"]), wanted=math.ceil(0.05 * case["n"]))
    s = _state(case, seed)
    prm = _params(case, s["lmax"])
    if case["op"] == "dense":
        A, B, keep = P.dense_operator(s["A"]), P.dense_operator(s["B"]), (s["A"], s["B"], s["dinv"])
    elif case["op"] == "hermitian":
        A, B, keep = P.hermitian_operator(s["A"]), P.hermitian_operator(s["B"]), (s["A"], s["B"], s["dinv"])
    elif case["op"] == "csr":
        keep = _csr_of_grid(s["shape"], s["V"])
        n = keep[0].numel() - 1
        A, B = P.csr_operator(n, *keep), None
    else:
        V = s["V"].reshape(-1).contiguous()
        keep = (V,)
        A = P.stencil_operator(s["shape"], 0.5 * wl.tensor_stencil_27("stiffness"),
                               coef_mass=wl.tensor_stencil_27("mass"), field=V, field_mode=2, bloch=s["k"])
        B = P.stencil_operator(s["shape"], wl.tensor_stencil_27("mass"), bloch=s["k"])
    ctx = P.chfsi_create(A, B, s.get("dinv"), prm, keep=keep)
    if case["kind"] == "rr":
        Y = s["Y"]
        return dict(kind="rr", ctx=ctx, Y=Y, X=torch.empty_like(Y.mT).mT, R=torch.empty_like(Y.mT).mT)
    lam = None if s["lam"] is None else s["lam"].cpu().numpy()
    return dict(kind="filter", ctx=ctx, X=s["X"], lam=lam, R=s["R"], Yp=torch.empty_like(s["X"].mT).mT,
                bounds=s["bounds"])


def run(state):
    ctx = state["ctx"]
    if state["kind"] == "filter":
        P.chfsi_filter(ctx, state["X"], state["lam"], state["R"], state["Yp"], *state["bounds"])
        return state["Yp"].mT
    if state["kind"] == "rr":
        ritz, norms = P.chfsi_rayleigh_ritz(ctx, state["Y"], state["X"], state["R"])
        return {"ritz": np.array(ritz), "norms": np.array(norms), "X": state["X"].mT, "R": state["R"].mT}
    # the wanted pairs: the block's other columns are guards that a solve leaves unconverged
    _, ev, _, _ = P.chfsi_solve(ctx, state["X"])
    w = state["wanted"]
    return {"values": np.array(ev[:w]), "X": state["X"].mT[:w]}


def exact(case, seed):
    if case["kind"] == "solve":
        A, B, _, _ = _dense_pencil(case, seed)
        L = torch.linalg.cholesky(B)
        H = torch.linalg.solve_triangular(L, torch.linalg.solve_triangular(L, A, upper=False).mT, upper=False)
        w = np.linalg.eigvalsh(((H + H.mT) / 2).cpu().numpy())
        return {"values": w[:math.ceil(0.05 * case["n"])], "X": None}   # vectors: defined up to sign
    s = _state(case, seed)
    if case["kind"] == "rr":
        lam, X, R = _torch_rr(s["op_A"], s["op_B"], s["Y"])
        # vectors and their residuals are defined up to sign
        return {"ritz": lam, "norms": torch.linalg.vector_norm(R, dim=0), "X": None, "R": None}
    d = None if s["dinv"] is None else s["dinv"][:, None]
    if case.get("method") == "c":
        return _plain_filter(s["op_A"], d, s["X"], case["degree"], s["bounds"]).mT
    out = torch.empty_like(s["X"].mT.contiguous())
    step = max(1, (1 << 31) // (16 * s["X"].shape[0]))       # a few columns at a time: they are independent
    for j in range(0, out.shape[0], step):
        c = slice(j, j + step)
        out[c] = _residual_filter(s["op_A"], d, s["X"][:, c], s["lam"][c], s["R"][:, c], case["degree"],
                                  s["bounds"]).mT
    return out


def work(case):
    b, p = case["b"], case["degree"]
    if case["op"] in ("dense", "hermitian"):
        n = case["n"]
        c = 4 if case["op"] == "hermitian" else 1              # real products in a complex one
        el = 16 if case["op"] == "hermitian" else 8
        product, operator = 2.0 * c * n * n * b, el * n * n
    else:
        n = case["nx"] * case["ny"] * case["nz"]
        c = 2 if case["op"] == "bloch" else 1
        el = 8 * c
        # stiffness and two mass applications, by offset classes: ~40 operations a point;
        # an assembled row has 27 products
        product, operator = (54.0 if case["op"] == "csr" else 40.0) * c * n * b, 8.0 * n
        if case["op"] == "csr":
            operator = 27.0 * 12 * n
    block = float(el) * n * b
    if case["kind"] == "filter":
        blocks = 2 if case["method"] == "c" else 3
        steps = p if case["method"] == "c" else p - 1
        return {"bytes": operator + blocks * block, "flops": steps * product}
    # Rayleigh-Ritz: two products, two symmetric Grams, the rotation, the small eigenproblem
    rr = 2 * product + 4.0 * n * b * b + 10.0 * b ** 3
    if case["kind"] == "rr":
        return {"bytes": 2 * operator + 3 * block, "flops": rr}
    passes = 9                                                # a cold solve of the serving stream
    return {"bytes": 2 * operator + block, "flops": passes * ((p - 1) * product + rr)}
