"""GPU parity of the CholQR factorisation at the edges of its 16-row tiles: blocks of
up to 128 vectors are factored and inverted by one workgroup (64- and 128-row
variants), larger ones in 64-row blocks with a last block of any size.  Bars: a
random block's Gram matrix is well conditioned, so orthonormality and residuals hold to
1e-11 and Ritz values to 1e-11 of the largest; a repeated or scaled-down column has to
end in the same subspace as the oracle's.
"""
import numpy as np
import pytest
import scipy.linalg as sla

import workloads as wl

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2503_22652_amd as P  # noqa: E402

BLOCKS = [1, 2, 15, 16, 17, 33, 48, 63, 64, 65, 79, 80, 81, 112, 127, 128, 129, 145, 193]


def _ritz(b, Yh, lam):
    n = len(lam)
    Ad = P.to_colmajor(np.diag(lam))
    prm = P.make_params(b, b, 4, filter_prec=P.PREC_FP64, lambda_max=4.5)
    ctx = P.chfsi_create(P.dense_operator(Ad), None, None, prm, keep=(Ad,))
    Yd, X, R = P.to_colmajor(Yh), P.colmajor_empty(n, b), P.colmajor_empty(n, b)
    w, _ = P.chfsi_rayleigh_ritz(ctx, Yd, X, R)
    return np.array(w), X.cpu().numpy(), R.cpu().numpy()


@pytest.mark.parametrize("b", BLOCKS)
def test_cholesky_tile_edges(b):
    n = 457
    lam = np.sort(np.random.default_rng(6).uniform(-1, 4, n))
    Yh = wl.random_block(n, b, 7) * np.logspace(-3, 3, b)      # scaled out before factoring
    print("cholesky", b, flush=True)
    w, X, R = _ritz(b, Yh, lam)
    Q, _ = np.linalg.qr(Yh)
    ref = sla.eigvalsh(Q.T @ (lam[:, None] * Q))
    assert np.abs(w - ref).max() <= 1e-11 * np.abs(ref).max()
    assert np.abs(X.T @ X - np.eye(b)).max() <= 1e-11
    assert np.abs(R - (lam[:, None] * X - X * w)).max() <= 1e-11


@pytest.mark.parametrize("b,j", [(17, 16), (64, 40), (80, 3), (80, 79), (128, 100), (150, 149)])
def test_cholesky_breakdown_keeps_the_span(b, j):
    """A column that repeats column 0 breaks a pivot in tile j / 16; the block is read
    again from the untouched Gram matrix, and the other columns' span is kept."""
    n = 457
    lam = np.sort(np.random.default_rng(6).uniform(-1, 4, n))
    Yh = wl.random_block(n, b, 8)
    if j:
        Yh[:, j] = Yh[:, 0]
    print("cholesky breakdown", b, j, flush=True)
    w, X, _ = _ritz(b, Yh, lam)
    assert np.abs(X.T @ X - np.eye(b)).max() <= 1e-8
    Q, _ = np.linalg.qr(np.delete(Yh, j, axis=1))
    assert np.abs(Q - X @ (X.T @ Q)).max() <= 1e-7
