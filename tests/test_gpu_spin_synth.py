"""Spin synthesis on the matrix cores, against the oracle and against the batches'
one-wavefront kernel (same products in the same order: equal bit for bit).

Degree ranges around the chunks of 16 (from l0, or one below it where l0 + m is odd),
slot tiles around the one, two and four wavefronts of a work group, transforms around
one and two column blocks, both precisions, derivative maps, Inf and NaN inputs.
Tolerances: FP64 the parity tests' 1e-11, normwise; FP32 products only bit for bit.
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


def _batch_of_one(p, direction, x):
    sht = _sht()
    b = sht.Batch([p])
    b.configure(sht.QUEUE_COST, 2)
    return to_host(b.execute(direction, [x])[0])


def _check(g, lmax, mmax, spin, ntrans, precision):
    sht = _sht()
    p = sht.Plan(sht.Geometry.from_inputs(g), lmax, mmax, spin=spin, ntrans=ntrans, precision=precision)
    p.set_tuning(valu=0)
    a = si.random_alm(lmax, mmax, ntrans, spin, spectrum="unit", tag=750 + spin)
    b = a.copy()
    b[:, :, si.lm_arrays(lmax, mmax)[0] < spin] = np.nan   # no part of the input
    pix = np.concatenate([np.arange(g.ofs[y], g.ofs[y] + g.nphi[y]) for y in range(g.nrings)])
    mp = to_host(p.alm2map(to_dev(b)))[..., pix]
    if precision == "fp64":
        assert rel_err(mp, oracle.synthesis(g, lmax, mmax, spin, a)[..., pix]) < TOL64
    assert np.array_equal(mp, _batch_of_one(p, sht.ALM2MAP, to_dev(b))[..., pix])


@pytest.mark.parametrize("precision", ["fp64", "fp32_mfma"])
@pytest.mark.parametrize("lmax", [3, 15, 16, 17, 18, 19, 20, 34, 35, 50])
def test_degree_ranges(lmax, precision):
    _check(si.gauss_geometry(lmax + 1, 2 * lmax + 1), lmax, lmax, 3, 2, precision)


@pytest.mark.parametrize("precision", ["fp64", "fp32_mfma"])
@pytest.mark.parametrize("ntrans", [2, 5])
@pytest.mark.parametrize("nslots", [1, 31, 33, 64, 65, 97, 129, 160, 225, 256])
def test_slot_tiles(nslots, ntrans, precision):
    _check(si.gauss_geometry(2 * nslots, 24, 0.1), 30, 11, 4, ntrans, precision)


@pytest.mark.parametrize("precision", ["fp64", "fp32_mfma"])
@pytest.mark.parametrize("ntrans", [2, 3, 4, 5, 7, 8, 9, 16, 17])
def test_column_blocks(ntrans, precision):
    _check(si.gauss_geometry(140, 257), 128, 120, 5, ntrans, precision)


def test_derivative_maps_and_single_ring():
    sht = _sht()
    lmax = 70
    g = si.gauss_geometry(71, 141)
    p = sht.Plan(sht.Geometry.from_inputs(g), lmax, lmax, spin=1, ntrans=3)
    a = si.random_alm(lmax, lmax, 3, 0, spectrum="unit", tag=760)
    assert rel_err(to_host(p.alm2map_deriv1(to_dev(a))), oracle.deriv_synthesis(g, lmax, lmax, a)) < TOL64
    # a lone ring on the equator: every second value of its recursions is zero
    _check(g.subset(np.array([35])), lmax, lmax, 3, 2, "fp64")


@pytest.mark.parametrize("precision", ["fp64", "fp32_mfma"])
def test_nonfinite_inputs(precision):
    """An Inf or NaN coefficient reaches every ring of its transform, also where its
    lambda underflows; the other transforms are untouched."""
    sht = _sht()
    lmax = 200
    g = si.gauss_geometry(lmax + 1, 2 * lmax + 1)
    p = sht.Plan(sht.Geometry.from_inputs(g), lmax, spin=3, ntrans=3, polar=False, precision=precision)
    a = si.random_alm(lmax, lmax, 3, 3, tag=761)
    clean = to_host(p.alm2map(to_dev(a)))
    b = a.copy()
    b[1, 0, si.alm_index(lmax, 160, 150), 0] = np.nan
    b[2, 1, si.alm_index(lmax, 170, 160), 1] = np.inf
    mp = to_host(p.alm2map(to_dev(b)))
    assert np.array_equal(mp[0], clean[0])
    for x in mp[1:]:
        assert not np.isfinite(x.reshape(2, lmax + 1, -1)).all(axis=-1).any()
