"""State copies: every byte of every field, for arrays at any alignment of their values,
sizes that a vector does not divide, and memory that a kernel may not touch directly."""
import ctypes as C

import numpy as np
import pytest

from gpu_util import FIELDS, gpu_box, need_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("dims", [(1, 1, 1), (3, 1, 1), (5, 7, 3), (64, 33, 31), (101, 75, 52)])
@pytest.mark.parametrize("offset", [0, 1, 2, 3])
def test_round_trip(dims, offset, precision):
    torch = need_gpu()
    from paper_2304_13746_amd import _lib as L
    from paper_2304_13746_amd.box import _view
    nx, ny, nz = dims
    n = nx * ny * nz
    rng = np.random.default_rng(n + offset)
    box = gpu_box(dims, precision=precision)

    def arrays(fill):
        # one value before and after each array shows a copy that runs over
        big = torch.full((8, n + 8), fill, dtype=box.dtype, device="cuda")
        return big, {f: big[q, offset + 1:offset + 1 + n] for q, f in enumerate(FIELDS)}

    _, src = arrays(0.0)
    for f in FIELDS:
        src[f].copy_(torch.from_numpy(1.0 + rng.random(n)))
    big, dst = arrays(-7.0)
    torch.cuda.synchronize()
    L.check(box.lib.mhd_set_state(box.ctx, C.byref(_view(src)), 0.25, 1e-3), "set")
    t, dt = C.c_double(), C.c_double()
    assert box.lib.mhd_get_state(box.ctx, C.byref(_view(dst)), C.byref(t), C.byref(dt)) == L.MHD_OK
    assert (t.value, dt.value) == (0.25, 1e-3)
    for f in FIELDS:
        assert torch.equal(src[f], dst[f]), f
    mask = torch.ones(n + 8, dtype=torch.bool)
    mask[offset + 1:offset + 1 + n] = False
    assert bool((big.cpu()[:, mask] == -7.0).all())
    box.close()


def test_pinned_host_arrays():
    """Arrays that the runtime's copies take and that are not device memory."""
    torch = need_gpu()
    from paper_2304_13746_amd import _lib as L
    from paper_2304_13746_amd.box import _view
    dims, n = (9, 6, 5), 270
    box = gpu_box(dims)
    src = {f: torch.empty(n, dtype=torch.float64, pin_memory=True).copy_(1.0 + torch.rand(n)) for f in FIELDS}
    dst = {f: torch.zeros(n, dtype=torch.float64, pin_memory=True) for f in FIELDS}
    L.check(box.lib.mhd_set_state(box.ctx, C.byref(_view(src)), 0.0, 1e-3), "set")
    L.check(box.lib.mhd_get_state(box.ctx, C.byref(_view(dst)), None, None), "get")
    for f in FIELDS:
        assert torch.equal(src[f], dst[f])
    box.close()


def test_arrays_that_overlap():
    """Fields that go to one array, in part or as a whole: the last one stands, as
    with one copy after another."""
    torch = need_gpu()
    from paper_2304_13746_amd import _lib as L
    from paper_2304_13746_amd.box import _view
    dims, n = (64, 33, 31), 64 * 33 * 31
    box = gpu_box(dims)
    src = {f: torch.rand(n, dtype=torch.float64, device="cuda") + 1.0 for f in FIELDS}
    big = torch.zeros(n + 100, dtype=torch.float64, device="cuda")
    dst = {f: torch.zeros(n, dtype=torch.float64, device="cuda") for f in FIELDS}
    dst["mx"] = dst["my"] = big[:n]
    dst["en"] = big[100:]
    torch.cuda.synchronize()
    L.check(box.lib.mhd_set_state(box.ctx, C.byref(_view(src)), 0.0, 1e-3), "set")
    L.check(box.lib.mhd_get_state(box.ctx, C.byref(_view(dst)), None, None), "get")
    assert torch.equal(big[:100], src["my"][:100])
    for f in FIELDS:
        if f not in ("mx", "my"):
            assert torch.equal(src[f], dst[f]), f
    box.close()
