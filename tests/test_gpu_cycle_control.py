"""Cycle control inside the stage launches: the step sequence over odd and even numbers
of cycles per call, clipping at t_stop, calls one after another, and graph replays of an
odd number of cycles."""
import pytest

import oracle as O
from gpu_util import bit_equal, gpu_box, need_gpu, oracle_params
from paper_2304_13746_amd import inputs as I

pytestmark = pytest.mark.gpu

DIMS = (20, 18, 17)


def start():
    s = I.turbulence(DIMS, seed=21, kpeak=2.0, mach=0.6, b0=(0.2, 0.1, -0.3))
    return s, s.pop("_l")


@pytest.mark.parametrize("integrator", ["rk2", "rk3", "euler"])
@pytest.mark.parametrize("emf", ["ec", "uct_hll"])
def test_calls_of_uneven_lengths(integrator, emf):
    need_gpu()
    s, l = start()
    box = gpu_box(DIMS, l, integrator=integrator, emf=emf)
    box.set_state(s)
    o, t, dt = O.copy_state(s), 0.0, 0.0
    p = oracle_params(DIMS, l, integrator=integrator, emf=emf)
    for n in (1, 2, 3, 0, 1, 1, 4):
        box.step(n)
        t, dt, _ = O.step(p, o, t, dt, n)
        g, tg, dg, _ = box.get_state_numpy()
        assert (tg, dg) == (t, dt) and bit_equal(g, o), n


@pytest.mark.parametrize("integrator", ["rk2", "rk3", "euler"])
def test_t_stop(integrator):
    need_gpu()
    s, l = start()
    p = oracle_params(DIMS, l, integrator=integrator)
    o = O.copy_state(s)
    t, dt, _ = O.step(p, o, 0.0, 0.0, 2)
    stop = t + 0.4 * dt  # inside the third cycle
    o = O.copy_state(s)
    t, dt, _ = O.step(p, o, 0.0, 0.0, 5, stop)
    box = gpu_box(DIMS, l, integrator=integrator)
    box.set_state(s)
    box.step(5, stop)
    g, tg, dg, _ = box.get_state_numpy()
    assert tg == t == stop and dg == dt and bit_equal(g, o)


def test_replays_of_an_odd_number_of_cycles():
    torch = need_gpu()
    from paper_2304_13746_amd.batch import BoxBatch
    s, l = start()
    box = gpu_box(DIMS, l)
    box.set_state(s)
    o, t, dt = O.copy_state(s), 0.0, 0.0
    graph = BoxBatch([box]).capture(3)
    for _ in range(3):
        graph.replay()
        box.step(2)
        t, dt, _ = O.step(oracle_params(DIMS, l), o, t, dt, 5)
        g, tg, dg, _ = box.get_state_numpy()
        assert (tg, dg) == (t, dt) and bit_equal(g, o)
