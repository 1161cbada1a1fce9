"""Staging sorts any order of the same nodes into one order.

Nodes on distinct cells of the 1024^3 Morton grid have distinct keys, so the
staged order, and with it every bit of a layer sum, must not depend on the
order in which they are given.  Sizes on both sides of what one wave, one
block and the one, two and three merged steps of the sorting network hold.
Non-finite and out-of-range data are refused at every size.
"""
import numpy as np
import pytest
import torch

from gpu_check import dev
from workloads import fields

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sd():
    import paper_2110_10749_amd as sd
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    return sd


def nodes(N):
    rng = np.random.default_rng(N)
    cell = np.unique(rng.integers(0, 1024, size=(2 * N + 64, 3)), axis=0)
    cell = cell[rng.permutation(len(cell))[:N]]
    cell[0] = 0
    if N > 1:
        cell[1] = 1023  # the box is the grid: a node's cell is its coordinate
    cell = np.unique(cell, axis=0)
    return np.ascontiguousarray(cell[rng.permutation(len(cell))].T.astype(np.float64))


@pytest.mark.parametrize("N", [1, 63, 500, 520, 4100, 8192, 8200, 16390, 32770, 65540, 131080])
def test_the_given_order_of_the_nodes_does_not_matter(sd, N):
    x = nodes(N)
    n = x.shape[1]
    nr = fields.random_vector(n, 2)
    w = np.random.default_rng(3).uniform(0.5, 1.0, size=n) / n
    q = fields.random_scalar(n, 4)
    out = []
    for order in (np.arange(n), np.random.default_rng(5).permutation(n)):
        plan = sd.Plan(dev(x[:, order]), dev(nr[:, order]), dev(w[order]), 40.0, max_restart=1)
        r = np.empty(n)
        r[order] = sd.laplace_layer_apply(plan, "dl_sub", dev(q[order])).cpu().numpy()
        out.append(r)
        plan.close()
    assert np.all(np.isfinite(out[0])) and np.array_equal(out[0], out[1])


@pytest.mark.parametrize("N", [1, 300, 20000])
def test_bad_node_data_is_refused(sd, N):
    x, nr, w = fields.point_cloud(N, seed=1)
    for what, value, code in [("x", np.nan, sd.binding.ERR_NONFINITE), ("x", -np.inf, sd.binding.ERR_NONFINITE),
                              ("x", 2e15, sd.binding.ERR_ARG), ("n", np.inf, sd.binding.ERR_NONFINITE),
                              ("w", np.nan, sd.binding.ERR_NONFINITE)]:
        a = {"x": x.copy(), "n": nr.copy(), "w": w.copy()}
        a[what].reshape(-1)[-1] = value
        with pytest.raises(sd.SdbieError) as e:
            sd.Plan(dev(a["x"]), dev(a["n"]), dev(a["w"]), 0.1)
        assert e.value.code == code
    with pytest.raises(sd.SdbieError) as e:
        sd.Plan(dev(x), dev(nr), dev(0.0 * w), 0.1)
    assert e.value.code == sd.binding.ERR_ARG
