"""FP64 limiters that are skipped where a wave's cells hold one state (LimO3, and PPM without
a field): bit for bit with the oracle on gas that is uniform but for one variable, in a few
cells, along one axis, or everywhere at one density."""
import numpy as np
import pytest

import oracle as O
from gpu_util import bit_equal, gpu_box, need_gpu, oracle_params

pytestmark = pytest.mark.gpu

DIMS = (60, 33, 29)
SCHEMES = [("hlld", "limo3", "ec"), ("hll", "limo3", "ec"), ("hllc", "limo3", "ec"), ("hllc", "ppm", "ec"),
           ("hlld", "limo3", "uct_hll")]


def uniform(riemann, speed):
    shape = DIMS[::-1]
    s = {f: np.full(shape, v) for f, v in zip(("rho", "mx", "my", "mz", "en"), (1.3, speed, -speed, 0.0, 1.9))}
    s.update({f: np.full(shape, 0.0 if riemann == "hllc" else b) for f, b in zip(("bx", "by", "bz"), (0.3, 0.0, -0.2))})
    return s


def check(s, riemann, recon, emf):
    box = gpu_box(DIMS, riemann=riemann, recon=recon, emf=emf, integrator="rk3")
    box.set_state(s)
    box.step(3)
    g, t, dt, _ = box.get_state_numpy()
    box.close()
    o = O.copy_state(s)
    to, dto, _ = O.step(oracle_params(DIMS, riemann=riemann, recon=recon, emf=emf, integrator="rk3"), o, 0.0, 0.0, 3)
    assert (t, dt) == (to, dto) and bit_equal(g, o)


@pytest.mark.parametrize("riemann,recon,emf", SCHEMES)
@pytest.mark.parametrize("speed", [0.0, 0.2])
@pytest.mark.parametrize("field", ["rho", "my", "en", "bx"])
def test_a_few_cells(field, speed, riemann, recon, emf):
    need_gpu()
    if field == "bx" and riemann == "hllc":
        field = "mz"
    s = uniform(riemann, speed)
    s[field][14:16, 15, 30:33] += 0.05
    check(s, riemann, recon, emf)


@pytest.mark.parametrize("riemann,recon,emf", SCHEMES)
@pytest.mark.parametrize("axis", [0, 1, 2])
def test_along_one_axis(axis, riemann, recon, emf):
    need_gpu()
    rng = np.random.default_rng(axis)
    s = uniform(riemann, 0.1)
    for f in ("en", "mx"):  # one density
        s[f] += 0.05 * rng.random(DIMS[axis]).reshape([-1 if 2 - q == axis else 1 for q in range(3)])
    check(s, riemann, recon, emf)
