"""GPU parity of the z-marching grid kernels over row lengths and plane counts: rows
that 4, 2 or only 1 point per thread divide (odd rows, 3 to 128 points; 129 goes to
the scalar kernel), y tiles of unequal height, and planes cut into ranges with a
short last one (few columns: 3 to 41 planes).  Real and Bloch, every field mode.
Bars as for the other grid tests (tests/parity.py).
"""
import numpy as np
import pytest

import workloads as wl
from oracle import filters, rr, stencil
from parity import GRID_TERMS, assert_columns, prec_name, residual_part

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2503_22652_amd as P  # noqa: E402

SHAPES = [(3, 3, 3), (5, 7, 9), (41, 5, 7), (6, 5, 14), (23, 19, 22), (5, 6, 127), (4, 3, 129), (4, 5, 130)]
LMAX = 18.5
K = (0.3, -0.7, 1.1)


def _problem(shape, mode, k=None, seed=8):
    V, _ = wl.gaussian_wells(shape, 3, np.random.default_rng(seed))
    cA, cB = 0.5 * wl.tensor_stencil_27("stiffness"), wl.tensor_stencil_27("mass")
    if k is None:
        ops = stencil.make_ops(cA, cB, V, shape, mode)
    else:
        ops = stencil.make_ops_bloch(cA, cB, V, shape, mode, k)
    Vd = torch.from_numpy(np.ascontiguousarray(V).reshape(-1)).cuda()
    opA = P.stencil_operator(shape, cA, coef_mass=cB, field=Vd, field_mode=mode, bloch=k)
    return (*ops, opA, P.stencil_operator(shape, cB, bloch=k), Vd)


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("mode", [0, 1, 2])
@pytest.mark.parametrize("prec", [P.PREC_FP64, P.PREC_FP32, P.PREC_BF16])
@pytest.mark.parametrize("k", [None, K], ids=["real", "bloch"])
def test_residual_filter_rows(k, prec, mode, shape):
    apply_A, apply_B, opA, opB, Vd = _problem(shape, mode, k)
    n, b, deg = int(np.prod(shape)), 5, 6
    cx = k is not None
    cm = P.to_colmajor_complex if cx else P.to_colmajor
    prm = P.make_params(b, b, deg, filter_prec=prec, lambda_max=LMAX)
    ctx = P.chfsi_create(opA, opB, None, prm, keep=(Vd,))
    make = wl.random_block_complex if cx else wl.random_block
    X, R = make(n, b, 4), make(n, b, 5)
    lam, bounds = np.linspace(-5.0, 0.0, b), (-5.5, LMAX, 0.5)
    Y = (P.colmajor_empty_complex if cx else P.colmajor_empty)(n, b)
    print("grid rows", shape, "mode", mode, prec_name(prec), "bloch" if cx else "real", flush=True)
    P.chfsi_filter(ctx, cm(X), lam, cm(R), Y, *bounds)
    torch.cuda.synchronize()
    ref, RYp, _ = filters.residual_filter(apply_A, filters.identity_op(), X, lam, R, deg, *bounds,
                                          return_parts=True)
    scale = np.linalg.norm(ref, axis=0) if prec == P.PREC_FP64 else residual_part(RYp)
    assert_columns(Y.cpu().numpy(), ref, scale, prec_name(prec), deg, GRID_TERMS, f"rows {shape}")


@pytest.mark.parametrize("shape", SHAPES[1:])
def test_plain_filter_and_rayleigh_ritz_rows(shape):
    apply_A, apply_B, opA, opB, Vd = _problem(shape, 2)
    n, b = int(np.prod(shape)), 6
    print("grid rows, plain filter and Rayleigh-Ritz", shape, flush=True)
    prm = P.make_params(b, b, 4, method=P.METHOD_CHFSI, lambda_max=LMAX)
    ctx = P.chfsi_create(opA, opB, None, prm, keep=(Vd,))
    X, Y = wl.random_block(n, b, 3), P.colmajor_empty(n, b)
    bounds = (-6.0, LMAX, 0.5)
    P.chfsi_filter(ctx, P.to_colmajor(X), None, None, Y, *bounds)
    torch.cuda.synchronize()
    ref = filters.chebyshev_filter(apply_A, X, 4, *bounds)
    assert_columns(Y.cpu().numpy(), ref, np.linalg.norm(ref, axis=0), "fp64", 4, GRID_TERMS, "plain")
    Xd, Rd = P.colmajor_empty(n, b), P.colmajor_empty(n, b)
    ritz, norms = P.chfsi_rayleigh_ritz(ctx, P.to_colmajor(X), Xd, Rd)
    o = rr.rayleigh_ritz(X, apply_A, apply_B)
    np.testing.assert_allclose(ritz, o["lam"], atol=1e-11 * np.abs(o["lam"]).max())
    np.testing.assert_allclose(norms, o["resnorm"], rtol=1e-7)
    Xh = Xd.cpu().numpy()
    np.testing.assert_allclose(Rd.cpu().numpy(), apply_A(Xh) - apply_B(Xh) * np.asarray(ritz)[None, :],
                               atol=1e-11)
