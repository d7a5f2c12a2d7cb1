"""GPU parity of the FP64 products at the edges of their tiles: column tiles of 16,
32 and 64, 64-row tiles, 16-deep k-slices, odd sizes and leading dimensions (16-byte
loads at 8-byte alignment, rows repeated past an edge), and the narrow Gram products
with many k-splits.  Bars: FP64 columns within G u sqrt(K p) of their own norm
(tests/parity.py), Ritz values to 1e-11 of the largest.
"""
import numpy as np
import pytest
import scipy.linalg as sla

import workloads as wl
from oracle import filters, rr
from parity import assert_columns

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2503_22652_amd as P  # noqa: E402

SIZES = [(1, 1), (2, 1), (17, 3), (63, 16), (64, 17), (65, 32), (130, 33), (257, 47), (401, 77),
         (500, 100)]


def _dense(n, seed=3):
    rng = np.random.default_rng(seed)
    G = rng.standard_normal((n, n))
    return (G + G.T) / (2 * np.sqrt(n)), rng.uniform(0.5, 1.5, n)


def _padded(M, pad):
    """Column-major device copy with leading dimension rows + pad."""
    n, b = M.shape
    buf = torch.zeros((b, n + pad), dtype=torch.float64, device="cuda")
    buf[:, :n] = torch.from_numpy(np.ascontiguousarray(M.T))
    return buf, buf.t()[:n]


@pytest.mark.parametrize("n,b", SIZES)
@pytest.mark.parametrize("pad", [0, 3])
@pytest.mark.parametrize("method", [P.METHOD_CHFSI, P.METHOD_RCHFSI])
def test_fp64_filter_product_edges(method, pad, n, b):
    A, d = _dense(n)
    keep, Ad = _padded(A, pad)
    op = P.dense_operator(Ad)
    op.ld = n + pad
    dd = torch.from_numpy(d).cuda()
    prm = P.make_params(b, b, 4, method=method, filter_prec=P.PREC_FP64, lambda_max=2.6)
    ctx = P.chfsi_create(op, None, dd, prm, keep=(keep, dd))
    X, R = wl.random_block(n, b, 1), wl.random_block(n, b, 2)
    lam, bounds = np.linspace(-1.5, -1.0, b), (-1.6, 2.6, 0.2)
    Y = P.colmajor_empty(n, b)
    kx, Xd = _padded(X, pad)
    kr, Rd = _padded(R, pad)
    Xd, Rd = (P.to_colmajor(X), P.to_colmajor(R)) if b == 1 else (Xd, Rd)
    print("fp64 product", n, b, "pad", pad, "method", method, flush=True)
    P.chfsi_filter(ctx, Xd, lam, Rd, Y, *bounds)
    torch.cuda.synchronize()
    if method == P.METHOD_CHFSI:
        ref = filters.chebyshev_filter(lambda Z: d[:, None] * (A @ Z), X, 4, *bounds)
    else:
        ref = filters.residual_filter(filters.dense_op(A), filters.diag_op(d), X, lam, R, 4, *bounds)
        ref = ref[0] if isinstance(ref, tuple) else ref
    assert_columns(Y.cpu().numpy(), ref, np.linalg.norm(ref, axis=0), "fp64", 4, n, f"n {n} b {b}")


@pytest.mark.parametrize("n,b", [(700, 48), (1003, 81), (1601, 144), (1300, 16)])
def test_fp64_product_odd_splits(n, b):
    """Sizes whose plans take split counts that are no powers of two, with a short last
    k range."""
    test_fp64_filter_product_edges(P.METHOD_RCHFSI, 3, n, b)


@pytest.mark.parametrize("n,b", [(2065, 129), (2305, 130), (4111, 191)])
def test_fp64_gram_many_splits(n, b):
    """Blocks of 128 <= b <= 640 with n >= 16 b: odd k ranges over up to 64 splits."""
    rng = np.random.default_rng(4)
    lam = np.sort(rng.uniform(-1, 4, n))
    A = np.diag(lam)
    Ad = P.to_colmajor(A)
    prm = P.make_params(b, b, 4, filter_prec=P.PREC_FP64, lambda_max=4.5)
    ctx = P.chfsi_create(P.dense_operator(Ad), None, None, prm, keep=(Ad,))
    Yh = wl.random_block(n, b, 5)
    Yd = P.to_colmajor(Yh)
    X, R = P.colmajor_empty(n, b), P.colmajor_empty(n, b)
    print("fp64 gram", n, b, flush=True)
    w, norms = P.chfsi_rayleigh_ritz(ctx, Yd, X, R)
    Q, _ = np.linalg.qr(Yh)
    ref = sla.eigvalsh(Q.T @ (lam[:, None] * Q))
    assert np.abs(np.array(w) - ref).max() <= 1e-11 * np.abs(ref).max()
    Xh = X.cpu().numpy()
    assert np.abs(Xh.T @ Xh - np.eye(b)).max() <= 1e-11
    Rh = lam[:, None] * Xh - Xh * np.array(w)
    assert np.abs(R.cpu().numpy() - Rh).max() <= 1e-11
