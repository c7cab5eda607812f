"""FP64 PPM and LimO3 limiters on data that sits on their decisions: constant runs, exact
extrema, linear and parabolic runs, steps and equal second differences, bit for bit with
the oracle."""
import numpy as np
import pytest

import oracle as O
from gpu_util import FIELDS, bit_equal, gpu_box, need_gpu, oracle_params

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("riemann", ["hlld", "hllc"])
@pytest.mark.parametrize("recon", ["ppm", "limo3"])
@pytest.mark.parametrize("axis", [0, 1, 2])
def test_limiter_decisions(axis, recon, riemann):
    need_gpu()
    rng = np.random.default_rng(8)
    dims = [26, 9, 9]
    dims[0], dims[axis] = dims[axis], dims[0]
    shape = tuple(dims[::-1])
    # small whole numbers along the axis: most limiters meet equalities and exact zeros
    line = lambda: rng.integers(-2, 3, dims[axis]).astype(float)  # noqa: E731
    runs = [line(), np.cumsum(rng.integers(-1, 2, dims[axis])).astype(float) % 3.0, np.zeros(dims[axis])]
    along = lambda q: q.reshape([-1 if d == axis else 1 for d in range(3)][::-1]) * np.ones(shape)  # noqa: E731
    rho = 2.0 + 0.5 * along(runs[0])
    p = 1.0 + 0.25 * along(runs[1])
    v = [0.125 * along(line()) for _ in range(3)]
    b = [np.zeros(shape) if riemann == "hllc" else 0.25 * along(line()) for _ in range(3)]
    if riemann != "hllc":
        b[axis] = np.full(shape, 0.5)
    bc = [0.5 * (q + np.roll(q, -1, 2 - d)) for d, q in enumerate(b)]
    en = p / (5.0 / 3.0 - 1.0) + 0.5 * rho * (v[0] ** 2 + v[1] ** 2 + v[2] ** 2) \
        + 0.5 * (bc[0] ** 2 + bc[1] ** 2 + bc[2] ** 2)
    s = {f: np.ascontiguousarray(q) for f, q in zip(FIELDS, [rho, rho * v[0], rho * v[1], rho * v[2], en, *b])}
    box = gpu_box(dims, riemann=riemann, recon=recon)
    box.set_state(s)
    o, t, dt = O.copy_state(s), 0.0, 0.0
    for _ in range(3):
        box.step(1)
        t, dt, _ = O.step(oracle_params(dims, riemann=riemann, recon=recon), o, t, dt, 1)
        g, tg, dg, _ = box.get_state_numpy()
        assert (tg, dg) == (t, dt) and bit_equal(g, o)
    box.close()
