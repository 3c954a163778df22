"""Which form a state buffer is in, across calls and recorded graphs.

A recorded graph may run at any time on the workspace it was recorded on, also
after the lattice was restarted, given other parameters or another state; so
every call has to find the state and the scratch buffer in whatever form they
are then.  Each test compares with a lattice that makes the same steps eagerly,
or with the CPU oracle.
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

G = (1e-3, -2e-3)
LX, LY = 50, 70  # ragged tiles, two waves of rows


def host(t):
    torch.cuda.synchronize()
    return t.detach().cpu().numpy()


def fields(lx=LX, ly=LY, seed=21):
    return workload.rt_fields(lx, ly, seed=seed)[:4]


def make(lx=LX, ly=LY, **kw):
    return LB(lx, ly, *fields(lx, ly), g=G, **kw)


def params(**kw):
    base = dict(tau=0.7, gx=G[0], gy=G[1], t_bottom=1.5, t_top=0.5, regularize=1, ybc=0)
    base.update(kw)
    return oracle.Params(**base)


def noisy(lb):
    noise = 1 + 1e-3 * torch.rand(lb.state_shape, dtype=torch.float64, device="cuda")
    return lb.get_state() * noise


def close(x, y):
    """The same values through other sums: some hundred FP64 roundings of terms
    no larger than the largest value."""
    x, y = host(x), y if isinstance(y, np.ndarray) else host(y)
    return np.abs(x - y).max() <= 1e-13 * np.abs(y).max()


# -- the scratch buffer ----------------------------------------------------------

KW = [dict(), dict(layout="soa"), dict(kernel="split_mfma"), dict(regularize=0)]


@pytest.mark.parametrize("kw", KW)
@pytest.mark.parametrize("recorded", [False, True])
def test_scratch_after_fused_steps(recorded, kw):
    """After fused steps the scratch buffer holds the state before the last
    one: get_scratch, bc and collide find it, whatever happened to the state
    or was recorded in between."""
    par = {k: kw[k] for k in ("kernel", "regularize") if k in kw}
    for replace in (False, True):
        a = make(layout=kw.get("layout", "column"))
        if recorded:
            a.capture(2)
        a.step(2)
        before = host(a.get_state())
        a.step(1)
        a.set_params(**par)
        if replace:
            a.set_state(noisy(a))
        state = a.get_state()
        assert np.array_equal(host(a.get_scratch()), before)
        a.bc()
        ref = oracle.bc(before, 1.5, 0.5)
        assert close(a.get_scratch(), ref)
        a.bc()  # once more: nothing changes
        assert close(a.get_scratch(), ref)
        assert torch.equal(a.get_state(), state)
        a.collide()  # of the scratch buffer, walls included
        assert close(a.get_scratch(), ref)
        p = params(regularize=kw.get("regularize", 1))
        assert close(a.get_state(), oracle.collide(ref, p))
        a.step(1)
        assert close(a.get_state(), oracle.run(oracle.collide(ref, p), p, 1))


def test_bc_of_other_wall_temperatures():
    """bc twice: the second one's walls count."""
    a = make()
    a.step(3)
    before = host(a.get_scratch())
    a.bc()
    a.set_params(t_bottom=1.25, t_top=0.75)
    a.bc()
    assert close(a.get_scratch(), oracle.bc(before, 1.25, 0.75))
    p = make(ybc="periodic")
    p.step(3)
    before = p.get_scratch()
    p.bc()  # no walls
    assert torch.equal(p.get_scratch(), before)


# -- plain BGK and the split stages ----------------------------------------------

@pytest.mark.parametrize("kernel", ["split", "split_lds", "split_wide", "split_mfma"])
@pytest.mark.parametrize("layout", ["column", "soa"])
@pytest.mark.parametrize("ybc", ["walls", "periodic"])
@pytest.mark.parametrize("recorded", [False, True])
def test_split_stages_of_a_stepped_state(recorded, ybc, layout, kernel):
    """halo, propagate, bc, collide of a state that fused steps left, with and
    without a recording before; lb_step's split path likewise."""
    a = make(ybc=ybc, layout=layout)
    if recorded:
        a.capture(2)
    a.step(3)
    f = host(a.get_state())
    a.set_params(kernel=kernel)
    a.halo()
    a.propagate()
    known = ~np.isnan(oracle.propagate(f, ybc=int(ybc == "periodic")))
    assert np.array_equal(host(a.get_scratch())[known],
                          oracle.propagate(f, ybc=int(ybc == "periodic"))[known])
    assert np.array_equal(host(a.get_state()), f)
    a.bc()
    a.collide()
    p = params(ybc=int(ybc == "periodic"))
    f = oracle.run(f, p, 1)
    assert close(a.get_state(), f)
    a.set_params(kernel="fused")
    a.step(2)
    a.set_params(kernel=kernel)
    a.step(2)
    assert close(a.get_state(), oracle.run(f, p, 4))


@pytest.mark.parametrize("shape", [(LX, LY), (280, 280), (6, 6), (40, 130)])
@pytest.mark.parametrize("layout", ["column", "soa"])
@pytest.mark.parametrize("ybc", ["walls", "periodic"])
def test_bgk_from_either_form(ybc, layout, shape):
    """Single and double plain BGK steps from coefficients and from the
    populations these stand for: the same bits; a recorded graph of them
    likewise, replayed between regularized steps."""
    a, b = (make(*shape, ybc=ybc, layout=layout) for _ in range(2))
    g = None
    for n in (1, 6, 10):
        a.set_params(regularize=1)
        b.set_params(regularize=1)
        a.step(2)
        b.step(2)
        b.set_state(b.get_state())
        a.set_params(regularize=0)
        b.set_params(regularize=0)
        a.step(n)
        for _ in range(n):
            b.step(1)
        assert torch.equal(a.get_state(), b.get_state())
        if g is None:
            g = a.capture(6)
            b.step(2)
        for reg in (0, 1):
            a.set_params(regularize=reg)
            b.set_params(regularize=reg)
            a.step(2)
            b.step(2)
            g.replay()
            b.set_params(regularize=0)
            b.set_state(b.get_state())
            b.step(6)
            assert torch.equal(a.get_state(), b.get_state())


def test_tape_of_bgk_from_either_form():
    a, b = make(), make()
    a.step(2)
    b.set_state(a.get_state())
    ta, tb = a.new_tape(3), b.new_tape(3)
    for lb, t in ((a, ta), (b, tb)):
        lb.set_params(regularize=0)
        lb.step_record(3, t)
    assert torch.equal(ta, tb)
    assert torch.equal(a.get_state(), b.get_state())


# -- restarts --------------------------------------------------------------------

SHAPES = [(LX, LY), (600, 520), (200, 130), (400, 300)]  # each choice of step kernel


@pytest.mark.parametrize("layout", ["column", "soa"])
@pytest.mark.parametrize("shape", SHAPES)
def test_recorded_graph_after_a_restart(shape, layout):
    """A graph stays valid when its lattice is restarted: it finds the new
    populations or the new equilibrium, and every reader its result."""
    a, b = (make(*shape, layout=layout) for _ in range(2))
    g = a.capture(6)
    f = fields(*shape, seed=5)
    state = noisy(b)

    def both():
        assert torch.equal(a.get_state(), b.get_state())
        assert torch.equal(a.populations(), b.populations())
        for x, y in zip(a.moments() + a.observables(), b.moments() + b.observables()):
            assert torch.equal(x, y)
        (ka, la), (kb, lb_) = a.loss_ke(), b.loss_ke()
        assert torch.equal(ka, kb) and torch.equal(la, lb_)

    for n in (1, 2, 5, 6):  # eager steps that follow
        for lb in (a, b):
            lb.reinit(*f)
            lb.set_state(state)
        g.replay()
        b.step(6)
        both()
        assert torch.equal(a.get_scratch(), b.get_scratch())
        a.step(n)
        for _ in range(n):
            b.step(1)
        both()
        for lb in (a, b):
            lb.reinit(*f)
        g.replay()
        b.step(6)
        both()
    tape = [lb.new_tape(2) for lb in (a, b)]
    for lb, t in zip((a, b), tape):
        lb.reinit(*f)
        lb.set_state(state)
    g.replay()
    b.step(6)
    a.step_record(2, tape[0])
    b.step_record(2, tape[1])
    assert torch.equal(tape[0], tape[1])
    both()


def test_recorded_graph_after_other_parameters_and_a_restart():
    """Recorded with the projection, replayed on a lattice restarted without."""
    a, b = make(), make()
    g = a.capture(2)
    f = fields(seed=5)
    for lb in (a, b):
        lb.set_params(regularize=0)
        lb.reinit(*f)
    g.replay()
    b.set_params(regularize=1)
    b.step(2)
    b.set_params(regularize=0)
    assert close(a.get_state(), b.get_state())
    for x, y in zip(a.moments() + a.observables(), b.moments() + b.observables()):
        assert close(x, y)
    a.step(3)
    b.step(3)
    assert close(a.get_state(), b.get_state())
    a.set_params(check_finite=1)
    a.step(1)  # raises if it misreads the state


def test_state_replaced_inside_a_graph():
    """The state is replaced, or the lattice restarted, by the graph itself."""
    a, b = make(), make()
    state = noisy(b)
    f = [torch.as_tensor(v, device="cuda") for v in fields(seed=5)]
    a.step(2)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        a.set_state(state)
    h = torch.cuda.CUDAGraph()
    with torch.cuda.graph(h):
        a.reinit(*f)
    torch.cuda.synchronize()
    for _ in range(2):
        a.reinit(*f)
        a.step(2)
        g.replay()
        b.set_state(state)
        assert torch.equal(a.get_state(), state)
        a.step(4)
        b.step(4)
        assert torch.equal(a.get_state(), b.get_state())
        a.set_state(state)
        h.replay()
        b.reinit(*f)
        assert torch.equal(a.get_state(), b.get_state())
        a.step(4)
        b.step(4)
        assert torch.equal(a.get_state(), b.get_state())


# one, two, three (loaded one and two ahead) and four columns per wave, ragged
SWEEPS = [(6, 6), (33, 113), (301, 400), (683, 57 * 4), (1027, 57 * 15), (2051, 57 * 20)]


@pytest.mark.parametrize("layout", ["column", "soa"])
@pytest.mark.parametrize("ybc", ["walls", "periodic"])
@pytest.mark.parametrize("shape", SWEEPS)
def test_sweep_that_finds_populations(shape, ybc, layout):
    """A graph recorded on coefficients, with and without a tape, replayed on a
    state just given as populations: the bits of eager steps."""
    a, b = (make(*shape, ybc=ybc, layout=layout) for _ in range(2))
    g = a.capture(2)
    tape, ref = a.new_tape(2), b.new_tape(2)
    torch.cuda.synchronize()
    h = torch.cuda.CUDAGraph()
    with torch.cuda.graph(h):
        a.step_record(2, tape)
    torch.cuda.synchronize()
    state = noisy(b)
    for _ in range(2):
        for lb in (a, b):
            lb.set_state(state)
        g.replay()
        b.step(2)
        assert torch.equal(a.get_state(), b.get_state())
        for lb in (a, b):
            lb.set_state(state)
        h.replay()
        b.step_record(2, ref)
        assert torch.equal(a.get_state(), b.get_state())
        assert torch.equal(tape, ref)
