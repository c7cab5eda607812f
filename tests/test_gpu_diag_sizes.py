"""Diagnostics at the sizes where the reduction can go wrong: fewer cells than one
block has threads, rows of one cell, and counts that its stride does not divide."""
import math

import numpy as np
import pytest

from gpu_util import gpu_box, need_gpu

pytestmark = pytest.mark.gpu

FIELDS = ("rho", "mx", "my", "mz", "en", "bx", "by", "bz")


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("dims", [(1, 1, 1), (1, 7, 3), (511, 1, 1), (3, 57, 3), (65, 33, 130), (97, 64, 61)])
def test_totals_and_divb(dims, precision):
    need_gpu()
    rng = np.random.default_rng(3)
    nx, ny, nz = dims
    dt = np.float32 if precision == "fp32" else np.float64
    s = {f: (1.0 + 0.5 * rng.standard_normal((nz, ny, nx))).astype(dt).astype(np.float64) for f in FIELDS}
    l = (1.25, 0.75, 2.0)
    box = gpu_box(dims, l, precision=precision)
    box.set_state(s, 0.0, 1e-3)
    d = box.diagnostics()
    box.close()
    dx, dy, dz = (b / n for b, n in zip(l, dims))
    # the exact sum rounded once, then the product with the cell volume (two roundings of
    # its own): 4 units of 2^-53; twice that for the root of the mean square
    tol = 4 * 2.0 ** -53
    got = [d["mass"], *d["mom"], d["energy"], *d["bflux"]]
    for f, g in zip(FIELDS, got):
        want = math.fsum(s[f].ravel()) * (dx * dy * dz)
        assert abs(g - want) <= tol * abs(want), (f, g, want)
    up = lambda a, axis: np.roll(a, -1, axis=axis)  # noqa: E731
    div = ((up(s["bx"], 2) - s["bx"]) * (1.0 / dx) + (up(s["by"], 1) - s["by"]) * (1.0 / dy)) \
        + (up(s["bz"], 0) - s["bz"]) * (1.0 / dz)
    assert d["divb_max"] == float(np.max(np.abs(div)))
    rms = math.sqrt(math.fsum((div * div).ravel()) / div.size)
    assert abs(d["divb_rms"] - rms) <= 2 * tol * rms
