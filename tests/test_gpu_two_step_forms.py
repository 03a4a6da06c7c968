"""Spin-0 FP64 matrix-core kernels: the form of the recursion (about the pole or the
equator) is each ring's own, so the phases of a ring do not depend, bit for bit, on
which other rings stand in its wavefront; and small grids, whose first wavefront holds
rings from the pole to the equator, are as accurate as larger ones.

Bound of the relative rms error of a ring: 1.5 (lmax + 1) units of 2^-53 (spectrum 1;
measured 0.3 to 0.8 by the one-step kernels at lmax 31 to 511).
"""
import numpy as np
import pytest

import oracle
import sht_inputs as si
from gpu_util import to_dev, to_host

pytestmark = pytest.mark.gpu


def _phases(g, lmax, a):
    import paper_1303_4945_amd as sht
    p = sht.Plan(sht.Geometry.from_inputs(g), lmax, ntrans=a.shape[0], polar=False)
    p.set_tuning(valu=0)
    return to_host(p.legendre_synth(to_dev(a)))


@pytest.mark.parametrize("lmax,nrings", [(31, 32), (63, 64), (63, 33), (64, 130), (100, 101)])
def test_rings_on_their_own(lmax, nrings):
    g = si.gauss_geometry(nrings, 2 * lmax + 1)
    a = si.random_alm(lmax, lmax, 3, 0, spectrum="unit", tag=790)
    full = _phases(g, lmax, a)
    ref = oracle.synthesis(g, lmax, lmax, 0, a, want_phases=True)[1]
    north = np.arange((nrings + 1) // 2)   # (the mirror rings take the northern colatitude)
    err = np.sqrt(((full - ref)[:, :, north] ** 2).sum(axis=(0, 1, 3, 4)) / (ref[:, :, north] ** 2).sum(axis=(0, 1, 3, 4)))
    assert err.max() < 1.5 * (lmax + 1) * 2.0 ** -53
    h = nrings // 2
    for some in (np.arange(nrings // 8), np.arange(h - 3, h + 3), np.array([h]), np.arange(nrings // 4, nrings // 4 + 2)):
        assert np.array_equal(_phases(g.subset(some), lmax, a), full[:, :, some])
