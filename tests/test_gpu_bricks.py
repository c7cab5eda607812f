"""Small FP64 boxes, whose stages run as bricks: bit for bit with the oracle at the edges
of both brick shapes, at the largest box of each and one cell past it, and in groups."""
import numpy as np
import pytest

import oracle as O
from gpu_util import bit_equal, gpu_box, need_gpu, oracle_params, run_both
from paper_2304_13746_amd import inputs as I

pytestmark = pytest.mark.gpu


def start(dims, riemann="hlld", seed=3):
    """Random cells (the turbulence generator needs more than one cell)."""
    rng = np.random.default_rng(seed)
    h = 1.0 / max(dims)
    f = lambda a, b: rng.uniform(a, b, dims[::-1])  # noqa: E731
    none = riemann == "hllc"
    s = I.assemble(f(0.7, 1.3), f(-0.5, 0.5), f(-0.5, 0.5), f(-0.5, 0.5), f(0.5, 0.8),
                   *(f(0.0, 0.0) if none else f(-0.4, 0.4) for _ in range(3)), 5.0 / 3.0)
    return s, tuple(n * h for n in dims)


# 256 bricks: (16, 32, 16) of 4x4x2, (32, 32, 32) of 8x4x4
@pytest.mark.parametrize("dims", [(1, 1, 1), (4, 4, 2), (5, 4, 2), (3, 7, 5), (16, 32, 16), (17, 32, 16),
                                  (32, 32, 32), (33, 32, 32), (8, 1, 100), (100, 3, 9)])
@pytest.mark.parametrize("riemann", ["hlld", "hll", "hllc"])
def test_sizes(dims, riemann):
    need_gpu()
    s, l = start(dims, riemann)
    g, o, gd, od, (tg, to) = run_both(s, dims, 3, l=l, riemann=riemann, per_step=True)
    assert bit_equal(g, o) and gd == od and tg == to


@pytest.mark.parametrize("integrator", ["rk3", "euler"])
def test_integrators(integrator):
    need_gpu()
    dims = (18, 20, 14)
    s, l = start(dims)
    g, o, gd, od, (tg, to) = run_both(s, dims, 4, l=l, integrator=integrator)
    assert bit_equal(g, o) and gd == od and tg == to


def test_requested_shape_and_status():
    """A requested shape marches, with the same bits; a non-physical cell is latched."""
    need_gpu()
    from paper_2304_13746_amd import _lib as L
    dims = (20, 12, 10)
    s, l = start(dims)
    out = []
    for kw in ({}, {"zchunk": 2}, {"tile": 2}):
        box = gpu_box(dims, l, **kw)
        box.set_state(s)
        box.step(3)
        out.append(box.get_state_numpy()[:3])
        box.close()
    assert all(bit_equal(a[0], out[0][0]) and a[1:] == out[0][1:] for a in out)
    s["en"][7, 3, 11] = -1.0
    box = gpu_box(dims, l)
    box.set_state(s, 0.0, 1e-5)
    assert box.get_state(check=False)[3] == L.MHD_OK
    box.step(1)
    assert box.get_state(check=False)[3] == L.MHD_ERR_NONPHYSICAL


def test_groups():
    """Groups that fit as bricks of either shape, and one that stops fitting none."""
    torch = need_gpu()
    from paper_2304_13746_amd.batch import BoxBatch
    for dims in ([(8, 8, 4), (9, 5, 3)], [(16, 16, 16), (20, 16, 8), (7, 30, 5)],
                 [(32, 32, 32), (16, 16, 16), (24, 8, 8)]):
        stream = torch.cuda.Stream()
        steps = [3, 1, 4][:len(dims)]
        states = [start(d, seed=60 + i) for i, d in enumerate(dims)]
        boxes = [gpu_box(d, l, stream=stream) for d, (_, l) in zip(dims, states)]
        for box, (s, _) in zip(boxes, states):
            box.set_state(s)
        BoxBatch(boxes).step(steps)
        for box, d, n, (s, l) in zip(boxes, dims, steps, states):
            o = O.copy_state(s)
            t, dt, _ = O.step(oracle_params(d, l), o, 0.0, 0.0, n)
            g, tg, dg, _ = box.get_state_numpy()
            assert bit_equal(g, o) and (tg, dg) == (t, dt)
