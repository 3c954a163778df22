"""Steps of lattices that stay in the Infinity Cache store into it, smaller and
larger ones stream: the same results on both sides of each line, for every
storage form.  The sizes straddle the lines (bytes of one buffer: 21 MB and
156 MB for the stored populations, 36 MB and 135 MB for FP64 coefficients).
"""

import numpy as np
import pytest

import oracle
from helpers import gpu_available
from paper_1703_00186_amd import workload

pytestmark = pytest.mark.gpu

if gpu_available():
    import torch
    from paper_1703_00186_amd.lb import LB


# (form, lattice): below, between and above the lines
CASES = [({"regularize": 0}, (101, 640)), ({"regularize": 0}, (149, 640)),
         ({"regularize": 0}, (901, 640)),
         ({"precision": "fp32c"}, (201, 640)), ({"precision": "fp32c"}, (249, 640)),
         ({"precision": "fp32c"}, (1709, 640)),
         ({"precision": "fp32l"}, (249, 640)), ({"precision": "fp32s"}, (249, 640)),
         ({"precision": "fp32s"}, (1709, 640)),
         ({}, (401, 640)), ({}, (479, 640)), ({}, (1811, 640))]


@pytest.mark.parametrize("layout", ["column", "soa"])
@pytest.mark.parametrize("kw,shape", CASES)
def test_step_matches_oracle(kw, shape, layout):
    lx, ly = shape
    fields = workload.rt_fields(lx, ly, seed=5)[:4]
    lb = LB(lx, ly, *fields, g=(1e-3, -2e-3), layout=layout, **kw)
    f = lb.populations().cpu().numpy()
    lb.step(3)
    got = lb.populations().cpu().numpy()
    p = oracle.Params(tau=0.7, gx=1e-3, gy=-2e-3, t_bottom=1.5, t_top=0.5,
                      regularize=kw.get("regularize", 1), ybc=0)
    ref = oracle.run(f, p, 3)
    # FP64: roundings of some hundred operations; FP32: two roundings a step of
    # each stored deviation (and the FP32 collision's), relative to the largest
    tol = 1e-13 if "precision" not in kw else 3 * 8 * 2.0 ** -24
    assert np.abs(got - ref).max() <= tol * np.abs(ref).max()
