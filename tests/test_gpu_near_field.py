"""One-direction near field of small surfaces, four waves to a target unit.

The waves share each near unit of a split (up to ten units on average, and in
float), or take four units at a time (double, more than ten).  Allocation-free
Stokes sums (eight splits) of nodes scattered over the unit sphere with a
smoothing length of 0.25, so that a split holds less than one unit up to
thirteen, the last unit full or ragged; every layer kind in both precisions
against the oracle on sampled rows (1e-12 in double; in float 3e-6, and the
coordinate-rounding bound 4 eps32 / delta^2 for the raw double layer) and
against the plan's one-direction sums (the same pairs in other splits: 1e-12).
"""
import math

import numpy as np
import pytest
import torch

from gpu_check import EPS32, LAYERS, TOL32, TOL64, dev, relerr
from oracle import oracle as O
from workloads import fields

pytestmark = pytest.mark.gpu

DELTA = 0.25


@pytest.mark.parametrize("N", [1, 64, 65, 300, 1601, 4400, 12000, 12033])
def test_near_units_shared_by_waves(N):
    import paper_2110_10749_amd as sd
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    x = np.random.default_rng(N).normal(size=(3, N))
    x /= np.linalg.norm(x, axis=0)
    w = np.full(N, 4 * math.pi / N)
    X, W, u = dev(x), dev(w), fields.random_vector(N, 3)
    geo = O.Geometry(x, x, w, DELTA)
    rows = np.arange(0, N, max(1, N // 61))
    plan = sd.Plan(X, X, W, DELTA)
    plan.set_symmetric(False)
    for name, _, kind in LAYERS:
        ref = O.stokes_apply(geo, 1.3, kind, u, rows)
        for prec in ("fp64", "mixed"):
            a = sd.stokes_layer_apply_noalloc(X, X, W, DELTA, 1.3, name, dev(u), prec=prec).cpu().numpy()
            b = sd.stokes_layer_apply(plan, 1.3, name, dev(u), prec=prec).cpu().numpy()
            e, eo = relerr(a, b), relerr(a[:, rows], ref)
            print(f"N={N} {name} {prec}: vs plan {e:.1e}, vs oracle {eo:.1e}", flush=True)
            assert np.all(np.isfinite(a)) and e < 1e-12
            tol = TOL64 if prec == "fp64" else max(TOL32, 4 * EPS32 / DELTA**2 if name == "dl_raw" else 0.0)
            assert eo < tol
    plan.close()
