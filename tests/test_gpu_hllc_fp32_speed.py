"""FP32 signal speeds of the field-free solver: those that HLL takes from the fast speed of
the same state, to the bit (cells of edge one, so that a first step holds one speed)."""
import pytest

from gpu_util import FIELDS, need_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("recon", ["plm", "ppm"])
def test_speeds_of_hllc_and_hll(recon):
    torch = need_gpu()
    from paper_2304_13746_amd.box import MHDBox
    boxes = [MHDBox(4, 4, 4, 4.0, 4.0, 4.0, precision="fp32", riemann=r, recon=recon) for r in ("hllc", "hll")]
    gen = torch.Generator().manual_seed(6)
    p = 0.5 + torch.rand(4000, generator=gen)
    for q in p.tolist():  # an ulp in the root of a square shows in one of some 200
        s = {f: torch.full((4, 4, 4), {"rho": 1.0, "en": 1.5 * q}.get(f, 0.0), dtype=torch.float32, device="cuda")
             for f in FIELDS}
        steps = [b.set_state(s).get_state()[2] for b in boxes]
        assert steps[0] == steps[1], q
