"""FP64 bit for bit with the oracle where the operands of its quotients and roots leave
the ordinary range: units far from one, and velocities and fields whose tails fall
through the smallest normal number to zero."""
import numpy as np
import pytest

import oracle as O
from gpu_util import FIELDS, bit_equal, gpu_box, need_gpu, oracle_params

pytestmark = pytest.mark.gpu

DIMS = (26, 12, 11)
SCHEMES = [("hlld", "plm", "ec"), ("hll", "plm", "ec"), ("hlld", "limo3", "ec"), ("hlld", "ppm", "ec"),
           ("hllc", "plm", "ec"), ("hllc", "ppm", "ec"), ("hlld", "plm", "uct_hll"), ("hlld", "plm", "uct_hlld")]


def state(rng, riemann, v_amp, rho_unit, v_unit, p_amp=0.1):
    nx, ny, nz = DIMS
    shape = (nz, ny, nx)
    rho = (1.0 + 0.2 * rng.random(shape)) * rho_unit
    p = (0.6 + p_amp * rng.random(shape)) * rho_unit * v_unit ** 2
    v = [v_amp * rng.uniform(-1, 1, shape) * v_unit for _ in range(3)]
    b = [v_amp * rng.uniform(-1, 1, shape) * v_unit * rho_unit ** 0.5 for _ in range(3)]
    if riemann == "hllc":
        b = [np.zeros(shape) for _ in range(3)]
    bc = [0.5 * (q + np.roll(q, -1, 2 - d)) for d, q in enumerate(b)]
    en = p / (5.0 / 3.0 - 1.0) + 0.5 * rho * (v[0] ** 2 + v[1] ** 2 + v[2] ** 2) \
        + 0.5 * (bc[0] ** 2 + bc[1] ** 2 + bc[2] ** 2)
    a = [rho, rho * v[0], rho * v[1], rho * v[2], en, *b]
    return {f: np.ascontiguousarray(q) for f, q in zip(FIELDS, a)}


def check(s, riemann, recon, emf, unit_time):
    box = gpu_box(DIMS, riemann=riemann, recon=recon, emf=emf)
    box.set_state(s)
    o = O.copy_state(s)
    p = oracle_params(DIMS, riemann=riemann, recon=recon, emf=emf)
    t, dt, _ = O.step(p, o, 0.0, 0.0, 3)
    box.step(3)
    g, tg, dg, _ = box.get_state_numpy()
    assert 0.0 < dt * unit_time < 1.0
    assert (tg, dg) == (t, dt)
    assert bit_equal(g, o), {f: float(np.max(np.abs(g[f] - o[f]))) for f in FIELDS}
    box.close()


@pytest.mark.parametrize("riemann,recon,emf", SCHEMES)
@pytest.mark.parametrize("axis", [0, 1, 2])
def test_tails(riemann, recon, emf, axis):
    """Velocities and fields that fall by some ten orders of magnitude a cell, to zero."""
    need_gpu()
    rng = np.random.default_rng(17 + axis)
    n = DIMS[2 - axis]
    d = np.minimum(np.arange(n), n - np.arange(n))
    fall = np.array([float("1e-%d" % k) for k in (660 * d) // n])
    amp = fall.reshape([-1 if q == axis else 1 for q in range(3)]) * 0.5
    # one pressure: differences of it would drive flows of their own size everywhere
    check(state(rng, riemann, amp, 1.0, 1.0, 0.0), riemann, recon, emf, 1.0)


@pytest.mark.parametrize("riemann,recon,emf", SCHEMES)
@pytest.mark.parametrize("rho_unit,v_unit", [(2.0 ** 140, 2.0 ** -60), (2.0 ** -140, 2.0 ** 60), (2.0 ** -90, 2.0 ** -40)])
def test_units(riemann, recon, emf, rho_unit, v_unit):
    need_gpu()
    rng = np.random.default_rng(5)
    check(state(rng, riemann, 0.5, rho_unit, v_unit), riemann, recon, emf, v_unit)


def test_uniform_at_rest():
    """Zero differences, zero field and zero velocity everywhere: nothing moves."""
    need_gpu()
    for riemann in ("hlld", "hll", "hllc"):
        for recon in ("plm", "limo3", "ppm"):
            shape = DIMS[::-1]
            s = {f: np.full(shape, {"rho": 1.3, "en": 0.9}.get(f, 0.0)) for f in FIELDS}
            box = gpu_box(DIMS, riemann=riemann, recon=recon)
            box.set_state(s)
            box.step(2)
            assert bit_equal(box.get_state_numpy()[0], s)
            box.close()
