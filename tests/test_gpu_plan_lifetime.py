"""Destroying a plan after a solve is host work only, and solves from many threads
do not share the host memory they read their scalars from.

sdbie_plan_destroy must not wait for the device (other plans' and other
programs' streams may be busy) and must be allowed while a stream is being
captured: the collector may destroy a plan at any time.  Solves of more threads
at once than the library keeps host blocks for, each on a plan and a stream of
its own, give the bits of the same solves one after the other.
"""
import threading

import numpy as np
import pytest
import torch

from gpu_check import dev
from workloads import fields

pytestmark = pytest.mark.gpu

E = [0.0, 0.6, 0.8]


@pytest.fixture(scope="module")
def sd():
    import paper_2110_10749_amd as sd
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    return sd


def cube_sphere(m):
    """6 m^2 nodes of the unit sphere: the cells of a cube's faces, projected."""
    c = 2.0 * np.arange(m) - (m - 1)
    a, b = (v.ravel() for v in np.meshgrid(c, c, indexing="ij"))
    f = np.full(a.shape, float(m))
    k = np.concatenate([np.stack(t) for t in ((f, a, b), (-f, b, a), (a, f, b), (b, -f, a), (a, b, f), (b, a, -f))],
                       axis=1)
    r = np.sqrt(k[0] * k[0] + k[1] * k[1] + k[2] * k[2])
    return k / r, 4.0 * m / (r * r * r)


def solved_plan(sd, m):
    x, w = cube_sphere(m)
    plan = sd.Plan(dev(x), dev(x), dev(w), 3.0 / m)
    sd.darcy_solve(plan, 1.0, 1e-2, 1.0, dev(fields.smooth_scalar(x, 1)))
    torch.cuda.synchronize()
    return plan


def test_destroying_a_plan_does_not_wait_for_other_streams(sd):
    plan = solved_plan(sd, 10)
    a = torch.randn(8192, 8192, device="cuda", dtype=torch.bfloat16)
    out = torch.empty_like(a)
    torch.mm(a, a, out=out)
    torch.cuda.synchronize()
    side, done = torch.cuda.Stream(), torch.cuda.Event()
    with torch.cuda.stream(side):
        for _ in range(300):  # a few hundred milliseconds of work
            torch.mm(a, a, out=out)
        done.record()
    assert not done.query()
    plan.close()
    waited = done.query()
    torch.cuda.synchronize()
    assert not waited, "sdbie_plan_destroy waited for another stream"


def test_destroying_a_plan_while_a_stream_is_captured(sd):
    plan, keep = solved_plan(sd, 10), solved_plan(sd, 12)
    q = dev(fields.random_scalar(keep.n, 3))
    ref = sd.laplace_layer_apply(keep, "dl_sub", q)
    out = torch.zeros_like(ref)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        sd.laplace_layer_apply(keep, "dl_sub", q, out=out)
        plan.close()
    for _ in range(3):
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, ref)
    keep.close()


def test_solves_of_many_threads_have_their_own_host_memory(sd):
    sizes = [4 + k % 6 for k in range(20)]
    plans, vn, ref = [], [], []
    for k, m in enumerate(sizes):
        x, w = cube_sphere(m)
        plans.append(sd.Plan(dev(x), dev(x), dev(w), 3.0 / m))
        vn.append(dev(fields.smooth_scalar(x, k)))
        ref.append(sd.stokes_solve(plans[-1], 1.0, 1e-2, 1.0, E, vn[-1])[0])
    torch.cuda.synchronize()
    start, out, err = threading.Barrier(len(sizes)), [None] * len(sizes), []

    def work(k):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                start.wait(30)
                for _ in range(3):
                    out[k] = sd.stokes_solve(plans[k], 1.0, 1e-2, 1.0, E, vn[k])[0]
                torch.cuda.current_stream().synchronize()
        except Exception as e:  # reported by the main thread
            err.append(e)

    threads = [threading.Thread(target=work, args=(k,)) for k in range(len(sizes))]
    for t in threads:
        t.start()
    for t in threads:
        t.join(60)
    assert not err and not any(t.is_alive() for t in threads)
    for k, p in enumerate(plans):
        assert torch.equal(out[k], ref[k])
        p.close()
