"""GPU parity of the dense filter product on bfloat16 matrix instructions (FP32
operands in three parts, or bfloat16 ones) at the edges of its tiles and slices.

One launch below a size, split-K over workgroups and a reduction above it; 32-row
and 32-column tiles, 32-deep k-slices (BF16: 64 to a stage), column tiles of up
to 160, complex operators as two k-segments.  A degree of 4 chains three products:
the first packs its right operand itself, the others read what the step before
left.  Bars as for the other filters (tests/parity.py): each column's error against
the oracle is at most G u sqrt(K p) of its residual part, K = n (complex: 2 n).
"""
import numpy as np
import pytest

import workloads as wl
from oracle import filters, rr
from parity import assert_columns, prec_name, residual_part

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2503_22652_amd as P  # noqa: E402

DEG = 4
# (n, b): one element past and short of tiles, slices and stages; odd leading
# dimensions; all in one launch a step
SIZES = [(20, 1), (31, 4), (32, 32), (33, 31), (64, 33), (65, 2), (127, 16), (129, 65), (700, 100),
         (1300, 163), (1281, 321)]


def _case(n, b, prec, cplx, scale=1.0, seed=9):
    """A random symmetric (Hermitian) A of norm ~2, a random block with small Ritz-like values."""
    rng = np.random.default_rng(seed)
    G = rng.standard_normal((n, n)) + (1j * rng.standard_normal((n, n)) if cplx else 0)
    A = (G + G.conj().T) / (2 * np.sqrt(n) * (np.sqrt(2) if cplx else 1))
    d = rng.uniform(0.5, 1.5, n)
    make = wl.random_block_complex if cplx else wl.random_block
    X, R = make(n, b, seed + 1), make(n, b, seed + 2) * scale
    lam = np.linspace(-1.5, -1.0, b)
    bounds = (-1.6, 2.6, 0.2)
    cm = P.to_colmajor_complex if cplx else P.to_colmajor
    Ad, dd = cm(A), torch.from_numpy(d).cuda()
    op = (P.hermitian_operator if cplx else P.dense_operator)(Ad)
    prm = P.make_params(b, b, DEG, method=P.METHOD_RCHFSI, filter_prec=prec, lambda_max=bounds[1])
    ctx = P.chfsi_create(op, None, dd, prm, keep=(Ad, dd))
    return A, d, X, R, lam, bounds, ctx, cm


@pytest.mark.parametrize("n,b", SIZES)
@pytest.mark.parametrize("cplx", [False, True], ids=["real", "complex"])
@pytest.mark.parametrize("prec", [P.PREC_FP32, P.PREC_BF16])
def test_filter_product_edges(prec, cplx, n, b):
    b = min(b, n)
    A, d, X, R, lam, bounds, ctx, cm = _case(n, b, prec, cplx)
    Y = (P.colmajor_empty_complex if cplx else P.colmajor_empty)(n, b)
    print("filter product", "complex" if cplx else "real", n, b, prec_name(prec), flush=True)
    P.chfsi_filter(ctx, cm(X), lam, cm(R), Y, *bounds)
    torch.cuda.synchronize()
    ref, RY, _ = filters.residual_filter(filters.dense_op(A), filters.diag_op(d), X, lam, R, DEG,
                                         *bounds, return_parts=True)
    assert_columns(Y.cpu().numpy(), ref, residual_part(RY, d), prec_name(prec), DEG,
                   (2 if cplx else 1) * n, f"product n {n} b {b}")


@pytest.mark.parametrize("n,b", [(96, 20), (1300, 163)])
@pytest.mark.parametrize("scale", [1e-28, 1e25])
def test_filter_product_fp32_scale(scale, n, b):
    """The three parts of a value keep its 24 bits at any scale at which they are normal numbers."""
    A, d, X, R, lam, bounds, ctx, cm = _case(n, b, P.PREC_FP32, False, scale)
    Y = P.colmajor_empty(n, b)
    print("filter product scale", scale, n, b, flush=True)
    X0 = np.zeros_like(X)
    P.chfsi_filter(ctx, cm(X0), lam, cm(R), Y, *bounds)
    torch.cuda.synchronize()
    ref, RY, _ = filters.residual_filter(filters.dense_op(A), filters.diag_op(d), X0, lam, R, DEG,
                                         *bounds, return_parts=True)
    assert_columns(Y.cpu().numpy(), ref, residual_part(RY, d), "fp32", DEG, n, f"scale {scale}")


@pytest.mark.parametrize("n,b", [(96, 20), (1300, 163)])
def test_filter_product_non_finite_stays_in_its_column(n, b):
    """A NaN or an infinity in one column of the block leaves the others as they were."""
    A, d, X, R, lam, bounds, ctx, cm = _case(n, b, P.PREC_FP32, False)
    Y0, Y1 = P.colmajor_empty(n, b), P.colmajor_empty(n, b)
    P.chfsi_filter(ctx, cm(X), lam, cm(R), Y0, *bounds)
    R[5, 3], R[7, 11] = np.nan, np.inf
    P.chfsi_filter(ctx, cm(X), lam, cm(R), Y1, *bounds)
    torch.cuda.synchronize()
    a, c = Y0.cpu().numpy(), Y1.cpu().numpy()
    good = [j for j in range(b) if j not in (3, 11)]
    assert np.array_equal(a[:, good], c[:, good])
    assert not np.isfinite(c[:, 3]).any() and not np.isfinite(c[:, 11]).any()


@pytest.mark.parametrize("n,b", [(33, 31), (129, 65), (700, 100), (1281, 321)])
@pytest.mark.parametrize("splits", [1, 3])
@pytest.mark.parametrize("cplx", [False, True], ids=["real", "complex"])
@pytest.mark.parametrize("prec", [P.PREC_FP32, P.PREC_BF16])
def test_filter_product_edges_two_launches(monkeypatch, prec, cplx, splits, n, b):
    """The path of large products (k-splits and a reduction) at ragged sizes."""
    monkeypatch.setenv("CHFSI_FILTER_GEMM_SPLITS", str(splits))
    test_filter_product_edges(prec, cplx, n, b)


@pytest.mark.parametrize("n,b,prec", [(3000, 255, P.PREC_FP32), (3000, 540, P.PREC_BF16)])
def test_filter_product_large_by_rule(prec, n, b):
    """Past the size from which a step is two launches."""
    test_filter_product_edges(prec, False, n, b)


@pytest.mark.parametrize("n,b,cplx", [(1893, 157, False), (1893, 80, True), (2090, 127, False)])
@pytest.mark.parametrize("prec", [P.PREC_FP32, P.PREC_BF16])
def test_filter_product_two_column_tiles(prec, n, b, cplx):
    """One launch with two column tiles a workgroup: a last pair whose second tile lies
    past the packed columns (160 of 192), and one that ends at them."""
    test_filter_product_edges(prec, cplx, n, b)
