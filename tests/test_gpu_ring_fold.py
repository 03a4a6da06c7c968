"""Synthesis rings with fewer pixels than 2 mmax + 1 (their bins fold), against the
oracle.  Tolerance: the parity tests' 1e-11, normwise."""
import pytest

import oracle
import sht_inputs as si
from gpu_util import rel_err, to_dev, to_host

pytestmark = pytest.mark.gpu

TOL64 = 1e-11


def _sht():
    import paper_1303_4945_amd as sht
    return sht


@pytest.mark.parametrize("spin", [0, 2])
def test_short_rings_fold(spin):
    """Rings with fewer pixels than 2 mmax + 1, around the lengths whose bins are
    folded by several threads each (128 bins)."""
    sht = _sht()
    lmax = 150
    nphi = [1, 2, 3, 4, 5, 8, 31, 64, 100, 126, 127, 128, 129, 130, 253, 254, 255, 256, 257, 258]
    g = si.mixed_geometry(nphi, 0.01)
    p = sht.Plan(sht.Geometry.from_inputs(g), lmax, spin=spin, ntrans=2, polar=False)
    a = si.random_alm(lmax, lmax, 2, spin, spectrum="unit", tag=743)
    assert rel_err(to_host(p.alm2map(to_dev(a))), oracle.synthesis(g, lmax, lmax, spin, a)) < TOL64
