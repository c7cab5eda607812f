"""FP64 LimO3 bit for bit with the oracle beside cells that hold no number: the limiter of a
cell whose neighbour is NaN or infinite, and ratios that overflow, as a division gives them."""
import numpy as np
import pytest

import oracle as O
from gpu_util import FIELDS, gpu_box, need_gpu, oracle_params

pytestmark = pytest.mark.gpu

DIMS = (20, 12, 11)


@pytest.mark.parametrize("riemann,emf", [("hlld", "ec"), ("hll", "ec"), ("hlld", "uct_hlld")])
@pytest.mark.parametrize("what", ["nan", "minus_nan", "no_density", "overflow"])
def test_limo3(what, riemann, emf):
    need_gpu()
    rng = np.random.default_rng(12)
    shape = DIMS[::-1]
    s = {"rho": 1.0 + 0.2 * rng.random(shape), "en": 1.0 + 0.1 * rng.random(shape)}
    s.update({f: 0.1 * rng.uniform(-1.0, 1.0, shape) for f in ("mx", "my", "mz")})
    s.update({f: np.zeros(shape) for f in ("bx", "by", "bz")})
    if what == "overflow":  # ratios of either sign beyond the largest number
        s["rho"][5, 6] = 1.0
        s["mx"][5, 6, 4:13] = [0.0, 1e-310, 0.3, 0.3, 0.3 + 1e-16, -0.2, -0.2 - 3e-17, 1e-312, 0.0]
    else:
        s["en" if "nan" in what else "rho"][5, 6, 7] = {"nan": np.nan, "minus_nan": -np.nan,
                                                       "no_density": 0.0}[what]
    box = gpu_box(DIMS, riemann=riemann, recon="limo3", emf=emf)
    box.set_state(s, 0.0, 1e-3)
    box.step(1)
    g, t, dt, _ = box.get_state_numpy(check=False)
    box.close()
    o = O.copy_state(s)
    to, dto, _ = O.step(oracle_params(DIMS, riemann=riemann, recon="limo3", emf=emf), o, 0.0, 1e-3, 1,
                        check=False)
    assert (t, dt) == (to, dto)
    for f in FIELDS:
        assert np.array_equal(g[f], o[f], equal_nan=True), f
