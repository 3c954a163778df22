"""Two steps per launch from stored populations equal single steps in every bit,
on states that stay finite at every extent: a weak gravity, so that the tallest
hydrostatic column neither overflows nor underflows.  The sizes lie on both
sides of every line of the rule, as in test_gpu_two_steps.py."""

import pytest

from helpers import gpu_available
from paper_1703_00186_amd import workload

pytestmark = pytest.mark.gpu

if gpu_available():
    import torch
    from paper_1703_00186_amd.lb import LB

FORMS = [{"regularize": 0}, {"precision": "fp32s"}, {"precision": "fp32s_f32sum"},
         {"precision": "fp32s", "regularize": 0}]
SMALL = [(6, 6), (9, 59), (64, 48), (170, 170), (200, 170)]
LARGE = {0: [(280, 280), (1400, 57), (6, 16000)], 1: [(14003, 57), (6, 140000), (2001, 404)]}


@pytest.mark.parametrize("ybc", ["walls", "periodic"])
@pytest.mark.parametrize("form", range(len(FORMS)))
def test_equals_single_steps(form, ybc):
    kw = FORMS[form]
    for lx, ly in SMALL + LARGE[int("precision" in kw)]:
        f = workload.rt_fields(lx, ly, g=1e-6, seed=4)[:4]
        a, b = (LB(lx, ly, *f, ybc=ybc, g=(5e-7, -1e-6), **kw) for _ in range(2))
        for n in (5, 10, 7):
            a.step(n)
            for _ in range(n):
                b.step(1)
            state = a.get_state()
            assert bool(state.isfinite().all()), (lx, ly, n)
            assert torch.equal(state, b.get_state()), (lx, ly, n)
        assert torch.equal(a.get_scratch(), b.get_scratch()), (lx, ly)
