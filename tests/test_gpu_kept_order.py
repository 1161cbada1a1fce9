"""Sums whose order of additions is an invariant keep their bits.

The inexact interface products of an FP64 coupled solve make its result, within
tol_ddm, a function of every rounding of the pair sums and of the Gram-Schmidt
sums, so these keep their order: the far-only symmetric set with one-direction
near pairs, near_split_body (four waves to a near unit, by sources or by units)
as near_body, dev_cgs2 as the separate kernels of the steps past 64 columns,
dev_dot_host as dev_dot.  golden/kept_order.json holds digests of the results of
the plain forms (one wave to a near unit, every Gram-Schmidt operation a launch
of its own, sums reduced on the device); the library has to reproduce them bit
for bit.  The inputs are exact (integer cube cells, quotients, square roots).

    python tests/test_gpu_kept_order.py > tests/golden/kept_order.json

records the digests of the library that it finds.
"""
import hashlib
import json
import os
import sys

import numpy as np
import pytest
import torch

from gpu_check import dev
from test_gpu_plan_lifetime import cube_sphere

pytestmark = pytest.mark.gpu

GOLDEN = os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden", "kept_order.json")
E = [0.0, 0.6, 0.8]
PRECS = ("fp64", "mixed")
LAYERS = ("sl", "dl_raw", "dl_sub")


def density(shape, seed):
    return dev(np.random.default_rng(seed).integers(-2**20, 2**20, size=shape) / 2.0**20)


def digest(t):
    a = np.ascontiguousarray(t.cpu().numpy() if isinstance(t, torch.Tensor) else np.asarray(t, dtype=np.float64))
    assert np.all(np.isfinite(a))
    return [hashlib.sha256(a.tobytes()).hexdigest()[:32], float(a.ravel()[0]).hex()]


def allocation_free_sums(sd, m, width):
    """eight splits: near units shared by sources (up to 9.2 of them to a split on average, and in
    float), or in double with more than ten (10.01 at m = 60, delta = 1/m, to 24) by units"""
    x, w = cube_sphere(m)
    X, W, u = dev(x), dev(w), density(x.shape, m)
    return {f"{layer} {prec}": digest(sd.stokes_layer_apply_noalloc(X, X, W, width / m, 1.3, layer, u, prec=prec))
            for layer in LAYERS for prec in PRECS}


def one_direction_sums(sd, m, width):
    """near units shared by sources (up to n = 4056 here), or a wave to each (from n = 4374 on)"""
    x, w = cube_sphere(m)
    plan = sd.Plan(dev(x), dev(x), dev(w), width / m, max_restart=1)
    plan.set_symmetric(False)
    q, u = density(w.shape, m), density(x.shape, m + 1)
    out = {}
    for layer in LAYERS:
        for prec in PRECS:
            out[f"laplace {layer} {prec}"] = digest(sd.laplace_layer_apply(plan, layer, q, prec=prec))
            out[f"stokes {layer} {prec}"] = digest(sd.stokes_layer_apply(plan, 1.3, layer, u, prec=prec))
    plan.close()
    return out


def one_direction_solves(sd, m):
    """Krylov steps short of and past 64 columns (tight tolerance, strong slip), and restarted ones"""
    x, w = cube_sphere(m)
    plan = sd.Plan(dev(x), dev(x), dev(w), 6.0 / m, max_restart=100)
    plan.set_symmetric(False)
    v, out = density(w.shape, m), {}
    for restart in (100, 20):
        opts = dict(restart=restart, tol_gmres=1e-13, maxit_gmres=90)
        p, info = sd.darcy_solve(plan, 1.0, 1e-2, 1.0, v, opts=opts)
        out[f"darcy restart {restart}"] = digest(p) + [info["gmres_iters"]]
        u, info = sd.stokes_solve(plan, 1.0, 1e-5, 1.0, E, p, opts=opts)
        out[f"stokes restart {restart}"] = digest(u) + [info["gmres_iters"]]
    plan.close()
    return out


def coupled_solves(sd, m):
    x, w = cube_sphere(m)
    plan = sd.Plan(dev(x), dev(x), dev(w), 6.0 / m, max_restart=80)
    out = {}
    for name, opts in (("default", {}), ("no recycling", dict(recycle=0)), ("restart 12", dict(restart=12)),
                       ("restart 80, tight", dict(restart=80, tol_gmres=1e-13, tol_ddm=1e-12))):
        p, u, drag, info = sd.ddm_solve(plan, 1.0, 1e-2, 1.0, E, opts=opts)
        out[name] = digest(p) + digest(u) + digest(drag) + [info["gmres_iters"]]
    plan.close()
    return out


def adjoints(sd, m):
    x, w = cube_sphere(m)
    plan = sd.Plan(dev(x), dev(x), dev(w), 6.0 / m)
    p, u, _, _ = sd.ddm_solve(plan, 1.0, 1e-2, 1.0, E)
    gx, gk, ga, info = sd.ddm_adjoint(plan, 1.0, 1e-2, 1.0, E, p, u, E)
    plan.close()
    return {"gradient": digest(gx) + digest([gk, ga]) + [info["gmres_iters"]]}


CASES = {}
for _m, _width in ((4, 6), (10, 6), (20, 6), (28, 9), (30, 9), (45, 2), (45, 6), (60, 1), (60, 6), (72, 4)):
    CASES[f"allocation-free sums m={_m} delta={_width}/m"] = (allocation_free_sums, _m, _width)
for _m, _width in ((10, 6), (20, 6), (26, 6), (27, 6), (40, 3)):
    CASES[f"one-direction sums m={_m} delta={_width}/m"] = (one_direction_sums, _m, _width)
for _m in (10, 27):
    CASES[f"one-direction solves m={_m}"] = (one_direction_solves, _m)
for _m in (8, 14, 20, 27, 40):
    CASES[f"coupled solves m={_m}"] = (coupled_solves, _m)
for _m in (8, 14, 27):
    CASES[f"adjoint m={_m}"] = (adjoints, _m)


@pytest.fixture(scope="module")
def golden():
    with open(GOLDEN) as f:
        return json.load(f)


@pytest.mark.parametrize("case", CASES)
def test_kept_order(case, golden):
    import paper_2110_10749_amd as sd
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    f, *args = CASES[case]
    got = f(sd, *args)
    differ = {k: (v, golden[case][k]) for k, v in got.items() if v != golden[case][k]}
    assert set(got) == set(golden[case]) and not differ


if __name__ == "__main__":
    import paper_2110_10749_amd as sd
    result = {}
    for case, (f, *args) in CASES.items():
        print(case, file=sys.stderr, flush=True)
        result[case] = f(sd, *args)
    json.dump(result, sys.stdout, indent=0)
