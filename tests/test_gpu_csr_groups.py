"""GPU parity of the CSR residual filter's blocks in 16-byte column groups (two FP64,
four FP32 or eight BF16 columns) against the oracle: columns that do not fill a group,
row tiles of 64 with a remainder, few tiles (columns split over workgroups), ragged rows
and empty ones, a leading dimension past n for the residuals, and degree 1 (no step).
Bounds of tests/parity.py with K = the longest row.
"""
import numpy as np
import pytest
import scipy.sparse as sp

import workloads as wl
from oracle import filters
from parity import assert_columns, prec_name, residual_part

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2503_22652_amd as P  # noqa: E402

BOUNDS = (-4.5, 9.0, -2.0)


def _matrix(n, seed=12):
    rng = np.random.default_rng(seed)
    m = max(1, 2 * n)
    G = sp.coo_matrix((rng.uniform(-0.4, 0.4, m), (rng.integers(0, n, m), rng.integers(0, n, m))),
                      shape=(n, n)).tocsr()
    A = (G + G.T + sp.diags(np.where(np.arange(n) % 5 == 3, 0.0, rng.uniform(-1, 3, n)))).tocsr()
    A.eliminate_zeros()                              # some rows end up short or empty
    A.sort_indices()
    return A, rng.uniform(0.5, 1.5, n)


@pytest.mark.parametrize("n,b", [(1, 1), (3, 2), (63, 3), (64, 4), (65, 5), (129, 7), (200, 8),
                                 (257, 9), (400, 17), (1000, 33), (70000, 10)])
@pytest.mark.parametrize("deg", [1, 5])
@pytest.mark.parametrize("prec", [P.PREC_FP64, P.PREC_FP32, P.PREC_BF16])
def test_csr_group_edges(prec, deg, n, b):
    A, d = _matrix(n)
    rp, ci = torch.from_numpy(A.indptr.astype(np.int64)).cuda(), torch.from_numpy(A.indices).cuda()
    va, dd = torch.from_numpy(A.data).cuda(), torch.from_numpy(d).cuda()
    op = P.csr_operator(n, rp, ci, va)
    prm = P.make_params(b, b, deg, method=P.METHOD_RCHFSI, filter_prec=prec, lambda_max=BOUNDS[1])
    ctx = P.chfsi_create(op, None, dd, prm, keep=(rp, ci, va, dd))
    X, R = wl.random_block(n, b, 1), wl.random_block(n, b, 2)
    lam = np.linspace(-4.0, -2.5, b)
    Rd = torch.zeros((b, n + 3), dtype=torch.float64, device="cuda")
    Rd[:, :n] = torch.from_numpy(np.ascontiguousarray(R.T))
    Rd = Rd.t()[:n] if b > 1 else P.to_colmajor(R)
    Y = P.colmajor_empty(n, b)
    print("csr groups", n, b, prec_name(prec), "degree", deg, flush=True)
    P.chfsi_filter(ctx, P.to_colmajor(X), lam, Rd, Y, *BOUNDS, degree=deg)
    torch.cuda.synchronize()
    ref, RY, _ = filters.residual_filter(lambda V: A @ V, filters.diag_op(d), X, lam, R, deg, *BOUNDS,
                                         return_parts=True)
    scale = np.linalg.norm(ref, axis=0) if prec == P.PREC_FP64 else residual_part(RY, d)
    assert_columns(Y.cpu().numpy(), ref, scale, prec_name(prec), deg,
                   max(1, int(np.diff(A.indptr).max())), f"csr n {n} b {b}")
