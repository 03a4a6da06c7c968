"""Spin-0 FP64 matrix-core kernels (two-step recursion in each class of l + m),
against the oracle at the edges of their shapes.

Degree ranges around the chunks of 16 (synthesis) and 32 (analysis) degrees, slot
counts around the 32-slot wavefronts, 64-slot tiles and 256-slot passes, transform
counts around one, two and four column blocks; Inf and NaN inputs; the results
independent of the column blocks.  Tolerance: the parity tests' 1e-11, normwise.
"""
import numpy as np
import pytest

import oracle
import sht_inputs as si
from gpu_util import rel_err, to_dev, to_host

pytestmark = pytest.mark.gpu

TOL64 = 1e-11


def _sht():
    import paper_1303_4945_amd as sht
    return sht


def _check(g, lmax, mmax, ntrans, **kw):
    sht = _sht()
    p = sht.Plan(sht.Geometry.from_inputs(g), lmax, mmax, ntrans=ntrans, **kw)
    p.set_tuning(valu=0)
    a = si.random_alm(lmax, mmax, ntrans, 0, spectrum="unit", tag=740)
    ref = oracle.synthesis(g, lmax, mmax, 0, a)
    assert rel_err(to_host(p.alm2map(to_dev(a))), ref) < TOL64
    assert rel_err(to_host(p.map2alm(to_dev(ref))), oracle.analysis(g, lmax, mmax, 0, ref)) < TOL64
    return p


@pytest.mark.parametrize("lmax", [0, 1, 14, 15, 16, 17, 30, 31, 32, 33, 63, 64, 65])
def test_degree_ranges(lmax):
    _check(si.gauss_geometry(lmax + 1, 2 * lmax + 1), lmax, lmax, 3)


@pytest.mark.parametrize("nslots", [1, 31, 32, 33, 64, 65, 128, 129, 255, 257, 520])
def test_slot_counts(nslots):
    _check(si.gauss_geometry(2 * nslots, 24, 0.1), 40, 23, 5)


@pytest.mark.parametrize("ntrans", [1, 7, 8, 9, 15, 16, 17, 24, 31, 32, 33, 40])
def test_column_blocks(ntrans):
    sht = _sht()
    lmax = 47
    g = si.gauss_geometry(lmax + 1, 2 * lmax + 1)
    p = _check(g, lmax, lmax, ntrans)
    a = to_dev(si.random_alm(lmax, lmax, ntrans, 0, tag=741))
    mp = p.alm2map(a)
    back = to_host(p.map2alm(mp))
    for s_ncb in (1, 2):
        for a_ncb in (1, 2):
            p.set_tuning(synth_ncb=s_ncb, anal_ncb=a_ncb, anal_tpw=1 if a_ncb == 2 else 2)
            assert np.array_equal(to_host(p.alm2map(a)), to_host(mp))
            assert np.array_equal(to_host(p.map2alm(mp)), back)


@pytest.mark.parametrize("kw", [dict(polar=False), dict(rescale_bits=128)])
def test_scales(kw):
    """Every (m, slot) kept: the longest runs below scale 0, whose chunks take no products."""
    lmax = 250
    _check(si.gauss_geometry(lmax + 1, 2 * lmax + 1), lmax, lmax, 4, **kw)


def test_nonfinite_inputs():
    """An Inf or NaN coefficient reaches every ring of its transform (also where its
    lambda underflows: a product with zero), one in a map every coefficient; the other
    transforms are untouched; ignored entries (Im a_l0) never matter."""
    sht = _sht()
    lmax = 200
    g = si.gauss_geometry(lmax + 1, 2 * lmax + 1)
    p = sht.Plan(sht.Geometry.from_inputs(g), lmax, ntrans=4, polar=False)
    a = si.random_alm(lmax, lmax, 4, 0, tag=742)
    clean = to_host(p.alm2map(to_dev(a)))
    b = a.copy()
    b[1, 0, si.alm_index(lmax, 160, 150), 0] = np.nan
    b[2, 0, si.alm_index(lmax, 170, 160), 1] = np.inf
    b[3, 0, si.alm_index(lmax, 5, 0), 1] = np.nan
    mp = to_host(p.alm2map(to_dev(b)))
    assert np.array_equal(mp[[0, 3]], clean[[0, 3]])
    for x in mp[1:3]:       # (a real Fourier sum keeps some pixels of a ring finite)
        assert not np.isfinite(x.reshape(lmax + 1, -1)).all(axis=1).any()
    m2 = clean.copy()
    m2[1, 0, 10 * (2 * lmax + 1) + 3] = np.nan
    back, ref = to_host(p.map2alm(to_dev(m2))), to_host(p.map2alm(to_dev(clean)))
    assert np.array_equal(back[[0, 2, 3]], ref[[0, 2, 3]])
    _, ms = si.lm_arrays(lmax, lmax)
    assert not np.isfinite(back[1, 0, :, 0]).any() and not np.isfinite(back[1, 0, ms > 0, 1]).any()
