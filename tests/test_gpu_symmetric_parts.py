"""Symmetric passes where their work lists change shape.

A tile pair is cut into 16, 8, 4, 2 or 1 parts by the number of tiles (and by
the room for partial slots), with the last tile full or ragged, a tile alone,
and with near and far unit pairs inside the near tile pairs.  Nodes scattered
over the unit sphere, delta = 3 mean spacings: every layer kind in both
precisions against the one-direction sums on every row (the same pairs added
in another order: 1e-13 in double; in float both add blocks of 16 float terms
into doubles, 3e-7) and against the oracle on sampled rows (1e-12 in double;
in float 3e-6, and the coordinate-rounding bound 4 eps32 / delta^2 for the raw
double layer).
"""
import math

import numpy as np
import pytest
import torch

from gpu_check import EPS32, LAYERS, TOL32, TOL64, dev, relerr
from oracle import oracle as O
from workloads import fields

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sd():
    import paper_2110_10749_amd as sd
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    return sd


@pytest.mark.parametrize("N", [256, 257, 1280, 2816, 2817, 5633, 8192, 11521, 16128, 16129, 23040, 23041])
def test_symmetric_passes_at_the_list_edges(sd, N):
    x = np.random.default_rng(N).normal(size=(3, N))
    x /= np.linalg.norm(x, axis=0)
    w = np.full(N, 4 * math.pi / N)
    delta = 3 * math.sqrt(4 * math.pi / N)
    plan = sd.Plan(dev(x), dev(x), dev(w), delta)
    geo = O.Geometry(x, x, w, delta)
    rows = np.arange(0, N, max(1, N // 61))
    q, u = fields.random_scalar(N, 1), fields.random_vector(N, 2)
    for name, lk, sk in LAYERS:
        for prec in ("fp64", "mixed"):
            out = []
            for sym in (False, True):
                plan.set_symmetric(sym)
                out.append((sd.laplace_layer_apply(plan, name, dev(q), prec=prec).cpu().numpy(),
                            sd.stokes_layer_apply(plan, 1.3, name, dev(u), prec=prec).cpu().numpy()))
            (dl, ds), (gl, gs) = out
            e = relerr(gl, dl), relerr(gs, ds)
            eo = (relerr(gl[rows], O.laplace_apply(geo, lk, q, rows)),
                  relerr(gs[:, rows], O.stokes_apply(geo, 1.3, sk, u, rows)))
            print(f"N={N} {name} {prec}: vs one-direction {e[0]:.1e} {e[1]:.1e}, vs oracle {eo[0]:.1e} {eo[1]:.1e}",
                  flush=True)
            assert max(e) < (1e-13 if prec == "fp64" else 3e-7)
            tol = TOL64 if prec == "fp64" else TOL32
            if prec == "mixed" and name == "dl_raw":
                tol = max(TOL32, 4 * EPS32 / delta**2)
            assert max(eo) < tol
    plan.close()
