"""sht_plan_flops counts a slot by the kernels that compute it: spin kernels, or spin-0
sums in the scalar part of a spin-1 or spin-2 plan."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("spin", [0, 1, 2, 3])
@pytest.mark.parametrize("lmax", [100, 140])
def test_algorithmic_work(spin, lmax):
    import paper_1303_4945_amd as sht
    p = sht.Plan(sht.Geometry.gauss(lmax + 1, 2 * lmax + 1), lmax, spin=spin, polar=False)
    slots = lmax // 2 + 1
    own = 32 if lmax == 140 and spin in (1, 2) else slots   # (71 slots: 32 near the pole)
    k = sum(lmax + 1 - max(m, spin) for m in range(lmax + 1))
    r, c = (10, 16) if spin else (4, 4)
    want = k * own * (r + c) + k * (slots - own) * (4 + 8)
    for d in (sht.ALM2MAP, sht.MAP2ALM):
        assert p.flops(d)[0] == want and p.flops(d)[1] == 0.0
    assert np.isclose(p.flops()[2], 16 * p.ncomp * p.nalm + 32 * p.ncomp * (lmax + 1) ** 2 + 8 * p.ncomp * p.npix)
