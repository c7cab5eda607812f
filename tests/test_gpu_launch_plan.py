"""Planes per block chosen at launch: whatever length the rule takes for a box or a
group, FP64 results are bit-identical to the oracle and FP32 results to a run with
another length."""
import pytest

import oracle as O
from gpu_util import bit_equal, gpu_box, need_gpu, oracle_params, run_both
from paper_2304_13746_amd import inputs as I

pytestmark = pytest.mark.gpu


# one plane per block up to a few chunks, extents below and above a tile, one plane in all
@pytest.mark.parametrize("dims", [(16, 16, 16), (25, 9, 1), (24, 8, 2), (3, 5, 40), (130, 70, 37)])
@pytest.mark.parametrize("riemann,emf", [("hlld", "ec"), ("hllc", "ec"), ("hlld", "uct_hll")])
def test_automatic_length(dims, riemann, emf):
    need_gpu()
    # HLLC is for boxes without a field
    s = I.turbulence(dims, seed=13, kpeak=2.0, mach=0.7,
                     b0=(0.0, 0.0, 0.0) if riemann == "hllc" else (0.2, -0.1, 0.3))
    l = s.pop("_l")
    g, o, gd, od, (tg, to) = run_both(s, dims, 3, l=l, riemann=riemann, per_step=True, emf=emf)
    assert bit_equal(g, o) and gd == od and tg == to
    out = []
    for zchunk in (0, 3):
        box = gpu_box(dims, l, precision="fp32", riemann=riemann, emf=emf, zchunk=zchunk)
        box.set_state(s)
        box.step(3)
        out.append(box.get_state_numpy()[:3])
        box.close()
    assert bit_equal(out[0][0], out[1][0]) and out[0][1:] == out[1][1:]


def test_group_with_requested_and_automatic_lengths(tmp_path):
    """Boxes that leave a group one after another, one with a length of its own; after
    tuning every box reports the length that its group was timed with."""
    torch = need_gpu()
    from paper_2304_13746_amd.autotune import Tuner
    from paper_2304_13746_amd.batch import BoxBatch
    dims = [(16, 24, 9), (40, 16, 33), (30, 30, 1), (64, 17, 20)]
    steps, zchunk = [4, 1, 3, 2], [0, 5, 0, 0]
    stream = torch.cuda.Stream()
    states, boxes = [], []
    for i, d in enumerate(dims):
        s = I.turbulence(d, seed=40 + i, kpeak=2.0, mach=0.6, b0=(0.1, 0.2, 0.3))
        states.append((s, s.pop("_l")))
        boxes.append(gpu_box(d, states[-1][1], stream=stream, zchunk=zchunk[i]))
        boxes[-1].set_state(s)
    batch = BoxBatch(boxes)
    batch.step(steps)
    for (s, l), d, n, box in zip(states, dims, steps, boxes):
        o = O.copy_state(s)
        t, dt, _ = O.step(oracle_params(d, l), o, 0.0, 0.0, n)
        g, tg, dg, _ = box.get_state_numpy()
        assert bit_equal(g, o) and (tg, dg) == (t, dt)
    choice = batch.tune(Tuner(str(tmp_path / "tune.json"), reps=1))
    assert {str(d[2]) for d in dims} == set(choice["zchunk_by_nz"])
    for d, box in zip(dims, boxes):
        assert 1 <= box.get_launch()[1] <= d[2]


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_automatic_tile(precision):
    """A box that 18x11 columns cover better takes them, with the bits of 24x8."""
    need_gpu()
    from paper_2304_13746_amd import _lib as L
    dims = (54, 55, 40)
    s = I.turbulence(dims, seed=31, kpeak=2.0, mach=0.7, b0=(0.2, -0.1, 0.3))
    l = s.pop("_l")
    out = []
    for tile in (0, L.TILE_24x8):
        box = gpu_box(dims, l, precision=precision, tile=tile)
        assert box.get_launch()[0] == (L.TILE_18x11 if tile == 0 else tile)
        box.set_state(s)
        box.step(3)
        out.append(box.get_state_numpy()[:3])
        box.close()
    assert bit_equal(out[0][0], out[1][0]) and out[0][1:] == out[1][1:]
