"""The periodic halo columns of a state that a recorded graph finds.

A fused step of populations reads halo columns and does not refresh them where
the kernel before it wrote them.  A recorded one finds whatever state is there
when it is replayed, and an eager one whatever a replay left: each kernel that
fills the state has to fill its halos, the collision of the split path too.
"""

import pytest

from helpers import gpu_available
from paper_1703_00186_amd import workload

pytestmark = pytest.mark.gpu

if gpu_available():
    import torch
    from paper_1703_00186_amd.lb import LB

FORMS = [dict(regularize=0), dict(regularize=0, layout="soa"), dict(precision="fp32s")]
SPLIT = ["split", "split_lds", "split_wide", "split_mfma"]
SHAPES = [(6, 6), (7, 70), (50, 300)]  # every column an edge, one that is none, several tiles


def make(shape, **kw):
    return LB(*shape, *workload.rt_fields(*shape, seed=4)[:4], g=(1e-3, -2e-3), **kw)


def kernels(form):
    return [k for k in SPLIT if k != "split_mfma" or form.get("precision", "fp64") == "fp64"]


@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("ybc", ["walls", "periodic"])
@pytest.mark.parametrize("shape", SHAPES)
def test_fused_graph_after_split_steps(shape, ybc, form):
    """Recorded with valid halos, replayed on what a split step left."""
    a, b = (make(shape, ybc=ybc, **form) for _ in range(2))
    g = a.capture(2)
    b.step(2)
    for kernel in kernels(form):
        for lb in (a, b):
            lb.set_params(kernel=kernel)
            lb.step(1)
            lb.set_params(kernel="fused")
        g.replay()
        b.set_state(b.get_state())  # which refreshes the halos
        b.step(2)
        assert torch.equal(a.get_state(), b.get_state()), kernel


@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("ybc", ["walls", "periodic"])
@pytest.mark.parametrize("shape", SHAPES)
def test_fused_steps_after_a_split_graph(shape, ybc, form):
    """A replayed split step between eager fused ones."""
    a, b = (make(shape, ybc=ybc, **form) for _ in range(2))
    for kernel in kernels(form):
        a.set_params(kernel=kernel)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            a.step(1)
        a.set_params(kernel="fused")
        for _ in range(2):
            a.step(2)
            g.replay()
            a.step(2)
            b.step(2)
            b.set_params(kernel=kernel)
            b.step(1)
            b.set_params(kernel="fused")
            b.set_state(b.get_state())
            b.step(2)
            assert torch.equal(a.get_state(), b.get_state()), kernel


def test_collision_of_coefficients_fills_the_halos():
    """lb_collide on the scratch that a regularized step left, as coefficients."""
    for kernel in SPLIT:
        a, b = (make((50, 70)) for _ in range(2))
        for lb in (a, b):
            lb.step(4)
            lb.set_params(kernel=kernel)
            lb.collide()
            lb.set_params(kernel="fused", regularize=0)
        g = torch.cuda.CUDAGraph()
        torch.cuda.synchronize()
        with torch.cuda.graph(g):  # recorded as steps of a state with halos
            a.set_params(regularize=0)
            a.step(2)
        c = make((50, 70), regularize=0)
        c.set_state(b.get_state())
        c.step(2)
        g.replay()
        assert torch.equal(a.get_state(), c.get_state()), kernel
