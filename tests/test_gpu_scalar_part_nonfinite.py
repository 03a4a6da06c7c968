"""Inf and NaN through plans with a scalar part (spins 1 and 2, FP64): as in the spin
kernels, which run alone in a plan of three transforms, they reach whatever a sum with
them enters, also with weight 0 (X at m = 0).
"""
import numpy as np
import pytest

import sht_inputs as si
from gpu_util import to_dev, to_host

pytestmark = pytest.mark.gpu

LMAX = 140


def _plans(spin, valu):
    import paper_1303_4945_amd as sht
    g = sht.Geometry.from_inputs(si.gauss_geometry(LMAX + 1, 2 * LMAX + 1))
    p = sht.Plan(g, LMAX, spin=spin, polar=False)
    p.set_tuning(valu=valu)
    return p, sht.Plan(g, LMAX, spin=spin, ntrans=3, polar=False)


@pytest.mark.parametrize("valu", [1, 0])
@pytest.mark.parametrize("spin", [1, 2])
@pytest.mark.parametrize("comp,l,m,reim,value", [(0, 120, 110, 0, np.nan), (1, 130, 3, 1, np.inf), (0, 60, 0, 0, np.nan),
                                                 (1, 2, 2, 0, -np.inf), (0, LMAX, LMAX, 1, np.nan)])
def test_coefficient(comp, l, m, reim, value, spin, valu):
    """Every ring of both maps is hit."""
    p, q = _plans(spin, valu)
    a = si.random_alm(LMAX, LMAX, 1, spin, tag=840)
    a[0, comp, si.alm_index(LMAX, l, m), reim] = value
    got = to_host(p.alm2map(to_dev(a)))[0].reshape(2, LMAX + 1, -1)
    ref = to_host(q.alm2map(to_dev(np.repeat(a, 3, axis=0))))[1].reshape(2, LMAX + 1, -1)
    hit, least = ~np.isfinite(got).all(axis=-1), ~np.isfinite(ref).all(axis=-1)
    assert hit.all() and (hit | ~least).all()


@pytest.mark.parametrize("valu", [1, 0])
@pytest.mark.parametrize("spin", [1, 2])
@pytest.mark.parametrize("ring", [0, 1, 40, 70, 139])
def test_pixel(ring, spin, valu):
    """A pixel of a ring of either kind: every coefficient that takes part is hit."""
    p, q = _plans(spin, valu)
    ls, ms = si.lm_arrays(LMAX, LMAX)
    rng = np.random.default_rng(ring)
    for comp, value in ((0, np.nan), (1, np.inf)):
        x = rng.standard_normal((1, 2, p.npix))
        x[0, comp, ring * (2 * LMAX + 1) + 7] = value
        got = ~np.isfinite(to_host(p.map2alm(to_dev(x)))[0])
        ref = ~np.isfinite(to_host(q.map2alm(to_dev(np.repeat(x, 3, axis=0))))[1])
        assert got[:, ls >= spin, 0].all() and got[:, (ls >= spin) & (ms > 0), 1].all()
        assert (got | ~ref).all() and not got[:, ms == 0, 1].any()
