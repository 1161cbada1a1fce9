"""The fused passes (double and single layer in one) against the oracle.

Solves reach this pass only behind their own residual checks, where a small
error of its float sums would cost iterations and fail nothing.  A stopped GMRES
shows one product: from an initial guess x0 the first iterate minus x0 is a
multiple d of the residual b - A x0, and the second minus x0 lies in the span of
d and A d, with A the product under test (double, or float pairs: one
correction solve of the iterative refinement).  So on sampled rows the double
product is held to b - A x0 ~ d, and both to that span, with A d from the oracle:
what a fit of the one or two coefficients leaves is the error of the product,
relative to the largest A d, and keeps the bars of the layer sums (1e-12 in
double, 3e-6 in float).  Sizes of 2 to 85 tiles: every cut of a tile pair into
parts, near pairs evaluated once for both directions, and the one-direction
passes of the same plan.

The residual passes (the right-hand side's single layer and the operator's
double layer, Laplace and Stokes, in double) end the mixed coupled solves, which
converge on what they return: at the smoke check's tolerances (1e-12, 1e-11)
the oracle's residuals of both equations on sampled rows stay below 1e-9 of the
right-hand sides.
"""
import numpy as np
import pytest
import torch

from gpu_check import TOL32, TOL64, dev
from oracle import oracle as O
from test_gpu_plan_lifetime import cube_sphere
from workloads import fields

pytestmark = pytest.mark.gpu

MU, K, ALPHA = 1.3, 1e-2, 1.0
U = np.array([0.2, -0.5, 0.8])


@pytest.fixture(scope="module")
def sd():
    import paper_2110_10749_amd as sd
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    return sd


def product(geo, beta, v, rows):
    """Abar_S v + V[beta P_tau v] on the rows"""
    flux = float((geo.w * (geo.n * v).sum(axis=0)).sum()) / geo.area
    return (O.stokes_apply(geo, MU, O.SDLS, v, rows) + flux * geo.n[:, rows]
            + O.stokes_apply(geo, MU, O.SSL, beta * O.tangential(geo.n, v), rows))


def left_over(target, columns, scale_column):
    """What the best fit of target by the columns leaves, relative to the last one's part in it."""
    A = np.stack([c.ravel() for c in columns], axis=1)
    c = np.linalg.lstsq(A, target.ravel(), rcond=None)[0]
    return float(np.max(np.abs(target.ravel() - A @ c)) / (abs(c[scale_column]) * np.max(np.abs(A[:, scale_column]))))


SIZES = [7, 16, 24, 32, 40, 53, 60]


@pytest.mark.parametrize("symmetric", [True, False])
@pytest.mark.parametrize("m", SIZES)
def test_slip_product(sd, m, symmetric):
    x, w = cube_sphere(m)
    N, delta = x.shape[1], 3.0 * 2.0 / m
    geo, beta = O.Geometry(x, x, w, delta), O.Params(MU, K, ALPHA).beta
    rows = np.arange(0, N, max(1, N // 61))
    plan = sd.Plan(dev(x), dev(x), dev(w), delta, max_restart=4)
    plan.set_symmetric(symmetric)
    x0 = fields.random_vector(N, m) + fields.smooth_vector(x, m)
    zero = dev(np.zeros(N))
    for prec, tol in (("fp64", TOL64), ("mixed", TOL32)):
        d = []
        for it in (1, 2):
            opts = dict(prec=prec, tol_gmres=1e-14, restart=4, maxit_gmres=it, mixed_mode="refine", refine_max=1,
                        tol_mixed=1e-12)
            u, _ = sd.stokes_solve(plan, MU, K, ALPHA, U, zero, u=dev(x0), opts=opts)
            d.append(u.cpu().numpy() - x0)
        residual = U[:, None] - product(geo, beta, x0, rows)
        e1 = left_over(residual, [d[0][:, rows]], 0)
        e2 = left_over(d[1][:, rows], [d[0][:, rows], product(geo, beta, d[0], rows)], 1)
        print(f"N={N} symmetric={symmetric} {prec}: residual {e1:.1e}, product {e2:.1e}", flush=True)
        assert e1 < TOL64 and e2 < tol
    plan.close()


@pytest.mark.parametrize("m", SIZES)
def test_residual_sums_of_mixed_coupled_solves(sd, m):
    x, w = cube_sphere(m)
    N, delta = x.shape[1], 3.0 * 2.0 / m
    geo = O.Geometry(x, x, w, delta)
    rows = np.arange(0, N, max(1, N // 97))
    plan = sd.Plan(dev(x), dev(x), dev(w), delta)
    p, u, _, info = sd.ddm_solve(plan, MU, K, ALPHA, U, opts=dict(prec="mixed", tol_gmres=1e-12, tol_ddm=1e-11))
    assert info["converged"]
    r1, b1, r2, b2 = O.coupled_residual(geo, O.Params(MU, K, ALPHA), U, p.cpu().numpy(), u.cpu().numpy(), rows)
    e1 = float(np.sqrt(np.mean((r1 - r1.mean()) ** 2) / np.mean(b1 ** 2)))  # up to the completion's constant
    e2 = float(np.sqrt(np.mean(r2 ** 2) / np.mean(b2 ** 2)))
    print(f"N={N}: Darcy {e1:.1e}, Stokes {e2:.1e}, {info}", flush=True)
    assert e1 < 1e-9 and e2 < 1e-9
    plan.close()
