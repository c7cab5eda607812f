"""FP64 bit for bit with the oracle where nothing carries a wave: cells without a field
whose pressure is zero or negative.  The status is latched there, and the state that comes
back beside it is what the scheme gives for a signal speed of zero; and so for a cell
without density and for speeds beyond the largest number."""
import numpy as np
import pytest

import oracle as O
from gpu_util import FIELDS, gpu_box, need_gpu, oracle_params

pytestmark = pytest.mark.gpu

DIMS = (26, 12, 11)
SCHEMES = [("hlld", "plm", "ec"), ("hll", "plm", "ec"), ("hlld", "limo3", "ec"), ("hll", "limo3", "ec"),
           ("hlld", "ppm", "ec"), ("hllc", "plm", "ec"), ("hllc", "limo3", "ec"), ("hllc", "ppm", "ec"),
           ("hll", "plm", "uct_hll"), ("hlld", "plm", "uct_hlld")]
CELLS = {"one": np.s_[5, 6, 7], "pair": np.s_[5, 6, 7:9], "region": np.s_[2:8, 3:9, 4:16]}


# bricks and columns of the default scheme (a requested length marches)
@pytest.mark.parametrize("zchunk", [0, 3])
@pytest.mark.parametrize("riemann,recon,emf", SCHEMES)
@pytest.mark.parametrize("cells", sorted(CELLS))
@pytest.mark.parametrize("pressure", [0.0, -0.01])
def test_no_pressure_no_field(pressure, cells, riemann, recon, emf, zchunk):
    need_gpu()
    from paper_2304_13746_amd import _lib as L
    rng = np.random.default_rng(4)
    shape = DIMS[::-1]
    rho = 1.0 + 0.2 * rng.random(shape)
    p = 0.6 + 0.1 * rng.random(shape)
    p[CELLS[cells]] = pressure
    none = np.zeros(shape)
    s = dict(zip(FIELDS, [rho, none, none, none, p / (5.0 / 3.0 - 1.0), none, none, none]))
    s = {f: a.copy() for f, a in s.items()}
    box = gpu_box(DIMS, riemann=riemann, recon=recon, emf=emf, zchunk=zchunk)
    box.set_state(s, 0.0, 1e-3)
    box.step(1)
    g, t, dt, rc = box.get_state_numpy(check=False)
    box.close()
    o = O.copy_state(s)
    to, dto, _ = O.step(oracle_params(DIMS, riemann=riemann, recon=recon, emf=emf), o, 0.0, 1e-3, 1,
                        check=False)
    assert rc == L.MHD_ERR_NONPHYSICAL and (t, dt) == (to, dto)
    for f in FIELDS:
        assert np.array_equal(g[f], o[f], equal_nan=True), f
    if cells == "one":
        assert all(np.isfinite(g[f]).all() for f in FIELDS)


@pytest.mark.parametrize("riemann", ["hlld", "hll", "hllc"])
@pytest.mark.parametrize("recon", ["plm", "limo3", "ppm"])
def test_first_step(recon, riemann):
    """The first step of such a state, from signal speeds alone."""
    need_gpu()
    rng = np.random.default_rng(9)
    shape = DIMS[::-1]
    rho = 1.0 + 0.2 * rng.random(shape)
    p = 0.6 + 0.1 * rng.random(shape)
    p[CELLS["region"]] = 0.0
    v = 0.1 * rng.uniform(-1.0, 1.0, shape)
    none = np.zeros(shape)
    s = dict(zip(FIELDS, [rho, rho * v, none, none, p / (5.0 / 3.0 - 1.0) + 0.5 * rho * v * v, none, none, none]))
    s = {f: a.copy() for f, a in s.items()}
    box = gpu_box(DIMS, riemann=riemann, recon=recon)
    box.set_state(s)
    dt = box.get_state(check=False)[2]
    box.close()
    # a cycle measures the step of the state that it starts from
    o = O.copy_state(s)
    assert dt == O.step(oracle_params(DIMS, riemann=riemann, recon=recon), o, 0.0, 1e-3, 1, check=False)[1]


@pytest.mark.parametrize("zchunk", [0, 3])
@pytest.mark.parametrize("riemann,recon,emf", [c for c in SCHEMES if c[0] != "hllc"])
def test_no_density(riemann, recon, emf, zchunk):
    """A cell without density that has momentum: infinite velocities, as a division gives."""
    need_gpu()
    rng = np.random.default_rng(7)
    shape = DIMS[::-1]
    s = {"rho": 1.0 + 0.2 * rng.random(shape), "en": 1.0 + 0.1 * rng.random(shape)}
    s.update({f: 0.1 * rng.uniform(-1.0, 1.0, shape) for f in ("mx", "my", "mz")})
    s.update({f: np.zeros(shape) for f in ("bx", "by", "bz")})
    s["rho"][5, 6, 7] = 0.0
    box = gpu_box(DIMS, riemann=riemann, recon=recon, emf=emf, zchunk=zchunk)
    box.set_state(s, 0.0, 1e-3)
    box.step(1)
    g, t, dt, _ = box.get_state_numpy(check=False)
    box.close()
    o = O.copy_state(s)
    to, dto, _ = O.step(oracle_params(DIMS, riemann=riemann, recon=recon, emf=emf), o, 0.0, 1e-3, 1,
                        check=False)
    assert (t, dt) == (to, dto)
    for f in FIELDS:
        assert np.array_equal(g[f], o[f], equal_nan=True), f


@pytest.mark.parametrize("riemann,recon,emf", [c for c in SCHEMES if c[0] != "hllc"])
@pytest.mark.parametrize("pressure", [1e200, np.inf])
def test_infinite_speed(pressure, riemann, recon, emf):
    """A speed whose square overflows: infinite, so the next step is zero."""
    need_gpu()
    rng = np.random.default_rng(3)
    shape = DIMS[::-1]
    p = 0.6 + 0.1 * rng.random(shape)
    p[5, 6, 7] = pressure
    s = {f: np.zeros(shape) for f in FIELDS}
    s["rho"], s["en"] = 1.0 + 0.2 * rng.random(shape), p / (5.0 / 3.0 - 1.0)
    box = gpu_box(DIMS, riemann=riemann, recon=recon, emf=emf)
    box.set_state(s, 0.0, 1e-3)
    box.step(2)
    g, t, dt, _ = box.get_state_numpy(check=False)
    box.close()
    o = O.copy_state(s)
    to, dto, _ = O.step(oracle_params(DIMS, riemann=riemann, recon=recon, emf=emf), o, 0.0, 1e-3, 2,
                        check=False)
    assert (t, dt) == (to, dto)
    for f in FIELDS:
        assert np.array_equal(g[f], o[f], equal_nan=True), f
