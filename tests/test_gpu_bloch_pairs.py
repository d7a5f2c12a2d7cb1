"""GPU: the Bloch correction kernels take 2, 4, 8 or 16 column pairs a thread, by the
number of workgroups.  Every column's arithmetic is the same whatever its block, so a
filter of many columns (4, 8 and 16 pairs a thread, with a ragged last chunk) has to give
the bits of the same filter on slices of 10 columns (2 a thread, which the oracle tests
cover); fused path (nx a multiple of 4) and in-place correction (nx = 10).
"""
import numpy as np
import pytest

import workloads as wl

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2503_22652_amd as P  # noqa: E402

K, LMAX = (0.3, -0.7, 1.1), 18.5


def _filter(op, V, X, lam, R, prec):
    n, b = X.shape
    prm = P.make_params(b, b, 4, method=P.METHOD_RCHFSI, filter_prec=prec, lambda_max=LMAX)
    ctx = P.chfsi_create(op, None, None, prm, keep=(V,))
    Y = P.colmajor_empty_complex(n, b)
    P.chfsi_filter(ctx, P.to_colmajor_complex(X), lam, P.to_colmajor_complex(R), Y, -1.0, LMAX, 4.0,
                   degree=4)
    torch.cuda.synchronize()
    return Y.cpu().numpy()


# 21 and 23 blocks of 256 boundary points: 4, 8 and 16 pairs at these widths
@pytest.mark.parametrize("shape", [(30, 30, 32), (50, 42, 10)])
@pytest.mark.parametrize("b", [51, 101, 219])
@pytest.mark.parametrize("prec", [P.PREC_FP64, P.PREC_BF16])
def test_wide_blocks_have_the_bits_of_narrow_ones(prec, b, shape):
    V, _ = wl.gaussian_wells(shape, 3, np.random.default_rng(8))
    Vd = torch.from_numpy(np.ascontiguousarray(V).reshape(-1)).cuda()
    op = P.stencil_operator(shape, 0.5 * wl.tensor_stencil_27("stiffness"),
                            coef_mass=wl.tensor_stencil_27("mass"), field=Vd, field_mode=2, bloch=K)
    n = int(np.prod(shape))
    X, R = wl.random_block_complex(n, b, 3), wl.random_block_complex(n, b, 4)
    lam = np.linspace(-0.5, 3.5, b)
    print("bloch pairs", shape, b, prec, flush=True)
    wide = _filter(op, Vd, X, lam, R, prec)
    assert np.all(np.isfinite(wide))
    for j in range(0, b, 50):
        part = slice(j, min(j + 10, b))
        np.testing.assert_array_equal(wide[:, part],
                                      _filter(op, Vd, X[:, part], lam[part], R[:, part], prec))
