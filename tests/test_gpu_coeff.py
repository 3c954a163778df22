"""The coefficient form of the FP64 state (15 Hermite coefficients per site)
against the 37 stored populations.

A lattice that has just been given its populations steps from those; one that
has stepped before steps from its coefficients.  Both must agree bit for bit,
and with the CPU oracle to FP64 rounding, for every tile the sweep kernels
are launched with (1 to 4 columns per wave, 56 rows per wave: the sizes
sit on both sides of a tile and have ragged ends), and so must two steps made
in one launch.  Changing the collision,
the split stages, replacing the state of a recorded graph and reading the
scratch buffer have to find the state whatever form it is in.
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


def host(t):
    torch.cuda.synchronize()
    return t.detach().cpu().numpy()


def make(lx, ly, **kw):
    f = workload.rt_fields(lx, ly, seed=21)[:4]
    kw.setdefault("g", (1e-3, -2e-3))
    return LB(lx, ly, *f, **kw), f


def params(**kw):
    base = dict(tau=0.7, gx=1e-3, gy=-2e-3, t_bottom=1.5, t_top=0.5, regularize=1, ybc=0)
    base.update(kw)
    return oracle.Params(**base)


# waves of 56 rows x columns of the lattice: below 1280 one column per wave,
# below 3584 two, below 40960 three (from 9216 on loaded two ahead), then four
SIZES = [(6, 6), (9, 56), (8, 57), (33, 113), (7, 250), (301, 400), (683, 57 * 4),
         (640, 401), (1027, 57 * 15), (2051, 57 * 20)]


@pytest.mark.parametrize("layout", ["column", "soa"])
@pytest.mark.parametrize("ybc", ["walls", "periodic"])
@pytest.mark.parametrize("shape", SIZES)
def test_coefficients_step_as_populations(shape, ybc, layout):
    lx, ly = shape
    a, _ = make(lx, ly, ybc=ybc, layout=layout)
    b, _ = make(lx, ly, ybc=ybc, layout=layout)
    a.step(2)
    for _ in range(3):
        f = a.get_state()
        b.set_state(f)
        a.step(1)  # from coefficients
        b.step(1)  # from populations
        assert torch.equal(a.get_state(), b.get_state())
    ref = oracle.run(host(f), params(ybc=1 if ybc == "periodic" else 0), 1)
    assert np.abs(host(a.populations()) - ref).max() <= 1e-13 * np.abs(ref).max()


@pytest.mark.parametrize("ybc", ["walls", "periodic"])
@pytest.mark.parametrize("shape", [(8, 57), (301, 400), (1027, 57 * 15)])
def test_tape_and_transposed_steps(shape, ybc):
    """The recorded moments do not depend on the form, and a run of transposed
    steps (coefficients between them) equals single ones (compact arrays)."""
    lx, ly = shape
    a, _ = make(lx, ly, ybc=ybc)
    b, _ = make(lx, ly, ybc=ybc)
    a.step(2)
    b.set_state(a.get_state())
    ta, tb = a.new_tape(3), b.new_tape(3)
    a.step_record(3, ta)
    b.step_record(3, tb)
    assert torch.equal(ta, tb)
    lam = a.lambda_from(np.random.default_rng(3).standard_normal((37, lx, ly)))
    ref, spare = lam.clone(), a.new_lambda()
    for j in (2, 1, 0):
        a.adjoint_step(ta[j], ref, spare)
        ref, spare = spare, ref
    a.adjoint_run(ta, lam)
    assert torch.equal(lam, ref)


# two steps per launch from 310000 sites on: waves of 52 rows, chunks of columns
# that are walked four at a time; and up to 128 columns of windows (of 52 rows,
# between walls one of 64).  400 x 400 and 65 x 65 lie between
@pytest.mark.parametrize("ybc", ["walls", "periodic"])
@pytest.mark.parametrize("shape", [(600, 520), (599, 521), (1201, 310), (6, 52000), (8, 40003),
                                   (31003, 12), (777, 1501), (400, 400), (6, 6), (64, 48),
                                   (64, 64), (128, 52), (64, 65), (65, 65), (7, 900)])
def test_two_steps_per_launch(shape, ybc):
    """Bit-equal to single steps for every count, eager, observed and recorded;
    the scratch buffer holds the state before the last step."""
    lx, ly = shape
    a, _ = make(lx, ly, ybc=ybc)
    b, _ = make(lx, ly, ybc=ybc)
    g = a.capture(6)  # makes two steps
    b.step(2)
    for n in (5, 7, 10, 6):
        a.step(n)
        for _ in range(n):
            b.step(1)
        assert torch.equal(a.get_state(), b.get_state())
        assert torch.equal(a.get_scratch(), b.get_scratch())
    for _ in range(2):
        g.replay()
        a.step(10)
        b.set_state(b.get_state())  # from populations
        for _ in range(16):
            b.step(1)
        assert torch.equal(a.get_state(), b.get_state())
    series = a.run_observed(17, 7)
    for k in range(2):
        for _ in range(7):
            b.step(1)
        assert torch.equal(series[k], b.observables()[1])
    for _ in range(3):
        b.step(1)
    assert torch.equal(a.get_state(), b.get_state())


def test_readers_of_both_forms_agree():
    lx, ly = 70, 130
    a, _ = make(lx, ly)
    b, _ = make(lx, ly)
    a.step(5)
    b.set_state(a.get_state())
    assert torch.equal(a.populations(), b.populations())
    # the fields of a are its coefficients, those of b sums over populations:
    # 37 roundings of terms up to |c|^2 f
    for x, y in zip(a.moments() + a.observables(), b.moments() + b.observables()):
        assert float((x - y).abs().max()) <= 1e-14 * max(1.0, float(y.abs().max()))
    (ka, la), (kb, lb_) = a.loss_ke(), b.loss_ke()
    assert float((ka - kb).abs()) <= 1e-13 * float(kb)
    assert float((la - lb_).abs().max()) <= 1e-14


@pytest.mark.parametrize("layout", ["column", "soa"])
@pytest.mark.parametrize("ybc", ["walls", "periodic"])
def test_change_of_collision_and_kernel(ybc, layout):
    """regularized -> plain BGK -> split -> regularized on one lattice."""
    lx, ly = 40, 61
    a, _ = make(lx, ly, ybc=ybc, layout=layout)
    a.step(3)
    f = host(a.populations())
    y = 1 if ybc == "periodic" else 0
    for kw, p in ((dict(regularize=0), params(regularize=0, ybc=y)),
                  (dict(regularize=1, kernel="split"), params(ybc=y)),
                  (dict(kernel="fused"), params(ybc=y)),
                  (dict(regularize=0, kernel="split"), params(regularize=0, ybc=y))):
        a.set_params(**kw)
        a.step(2)
        f = oracle.run(f, p, 2)
        assert np.abs(host(a.populations()) - f).max() <= 1e-13 * np.abs(f).max()


def test_split_stages_after_fused_steps():
    lx, ly = 40, 61
    a, _ = make(lx, ly)
    b, _ = make(lx, ly)
    a.step(2)
    before = a.get_state()
    a.step(1)
    after = a.get_state()
    assert torch.equal(a.get_scratch(), before)  # the previous state
    a.bc()  # on the scratch buffer; the state stays
    ref = oracle.bc(host(before), 1.5, 0.5)
    assert np.abs(host(a.get_scratch()) - ref).max() <= 1e-13 * np.abs(ref).max()
    assert torch.equal(a.get_state(), after)
    a.halo()
    a.propagate()
    b.set_state(after)
    b.propagate()
    ga, gb = host(a.get_scratch()), host(b.get_scratch())
    known = ~np.isnan(oracle.propagate(host(after), ybc=0))
    assert np.array_equal(ga[known], gb[known])
    a.bc()
    a.collide()
    c, _ = make(lx, ly)
    c.step(3)
    c.step(1)
    c.collide()  # of the scratch buffer: the state before the last step
    ref = oracle.collide(host(after), params())
    assert np.abs(host(c.get_state()) - ref).max() <= 1e-13 * np.abs(ref).max()
    ref = oracle.run(host(after), params(), 1)
    assert np.abs(host(a.get_state()) - ref).max() <= 1e-13 * np.abs(ref).max()


def test_recorded_graph_after_the_state_was_replaced():
    """A graph finds populations (after set_state), coefficients (after steps
    or a replay) and, with plain BGK in between, either."""
    lx, ly = 50, 70
    a, f = make(lx, ly)
    b, _ = make(lx, ly)
    g = a.capture(2)
    b.step(2)
    for k in range(3):
        g.replay()
        b.step(2)
        assert torch.equal(a.get_state(), b.get_state())
        noise = 1 + 1e-3 * torch.rand((37, lx, ly), dtype=torch.float64, device="cuda")
        state = b.get_state() * noise
        a.set_state(state)
        b.set_state(state)
        g.replay()
        a.step(2)
        b.step(4)
        assert torch.equal(a.get_state(), b.get_state())
        assert torch.equal(a.observables()[1], b.observables()[1])
    for lb in (a, b):
        lb.set_params(regularize=0)
        lb.step(2)
        lb.set_params(regularize=1)
    g.replay()
    b.step(2)
    assert torch.equal(a.get_state(), b.get_state())
