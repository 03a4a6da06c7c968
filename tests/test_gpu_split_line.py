"""Spin-1 and spin-2 plans with a scalar part: which rings it takes.

The scalar part divides by sin^s t, so it must not take rings next to a pole, however
many a given grid has there, and must start only where the division does not show
beside the error of the spin kernels.  Those kernels alone are in a plan of at most 64
slots, which has no scalar part.
"""
import numpy as np
import pytest

import oracle
import sht_inputs as si
from gpu_util import rel_err, to_dev, to_host

pytestmark = pytest.mark.gpu

TOL64 = 1e-11   # the parity tests' bound, normwise; here ring by ring


def _sht():
    import paper_1303_4945_amd as sht
    return sht


def _grid(theta):
    theta = np.sort(np.asarray(theta, dtype=np.float64))
    n = theta.size
    return si.Geometry(theta, np.full(n, 64, dtype=np.int64), np.zeros(n), np.full(n, 0.1),
                       64 * np.arange(n, dtype=np.int64))


@pytest.mark.parametrize("valu", [1, 0])
@pytest.mark.parametrize("spin", [1, 2])
@pytest.mark.parametrize("npolar", [33, 40, 47, 48, 65])
def test_rings_next_to_a_pole(npolar, spin, valu):
    """Rings within 1e-3 of a pole, the pole itself among them (theta 0, or pi in one
    case), beside 40 others: ring by ring against the oracle, and the analysis of maps
    that only the polar rings fill."""
    sht = _sht()
    lmax = 40
    rng = np.random.default_rng(npolar)
    polar = np.concatenate([[0.0, 1e-12], 10.0 ** rng.uniform(-8, -3, npolar - 2)])
    if npolar == 48:
        polar = np.pi - polar
    g = _grid(np.concatenate([polar, rng.uniform(0.4, 2.7, 40)]))
    p = sht.Plan(sht.Geometry.from_inputs(g), lmax, spin=spin)
    p.set_tuning(valu=valu)
    a = si.random_alm(lmax, lmax, 1, spin, spectrum="unit", tag=770 + spin)
    ref = oracle.synthesis(g, lmax, lmax, spin, a).reshape(2, g.nrings, 64)
    got = to_host(p.alm2map(to_dev(a))).reshape(2, g.nrings, 64)
    for y in range(g.nrings):
        if np.abs(ref[:, y]).max() > 0.0:
            assert rel_err(got[:, y], ref[:, y]) < TOL64, (y, g.theta[y])
        else:
            assert np.abs(got[:, y]).max() == 0.0, (y, g.theta[y])
    near = np.sin(g.theta) < 2e-3
    m = np.where(near[None, :, None], ref, 0.0).reshape(1, 2, -1)
    assert rel_err(to_host(p.map2alm(to_dev(m))), oracle.analysis(g, lmax, lmax, spin, m)) < TOL64


@pytest.mark.parametrize("valu", [1, 0])
@pytest.mark.parametrize("spin,lmax,lo,hi", [(2, 60, 0.2, 0.33), (2, 60, 0.65, 0.75), (2, 130, 0.2, 0.33),
                                             (2, 130, 0.5, 0.6), (1, 60, 0.2, 0.33), (1, 60, 0.45, 0.55)])
def test_error_beside_the_line(spin, lmax, lo, hi, valu):
    """The same rings in a plan with a scalar part and in one of 64 slots without: the
    relative rms error of the phases against the oracle grows by a tenth at most (at
    most 1.5 of it here: 60 rings, whose own scatter is about 1/10 of either)."""
    sht = _sht()
    rng = np.random.default_rng(5)
    mine = np.arcsin(rng.uniform(lo, hi, 60))
    small = _grid(mine)
    large = _grid(np.concatenate([mine, np.linspace(0.01, 0.05, 32), rng.uniform(0.9, 1.5, 60)]))
    a = si.random_alm(lmax, lmax, 1, spin, spectrum="powerlaw", tag=780)
    F = oracle.synthesis(small, lmax, lmax, spin, a, want_phases=True)[1][0]

    def err(g):
        p = sht.Plan(sht.Geometry.from_inputs(g), lmax, spin=spin)
        p.set_tuning(valu=valu)
        x = to_host(p.legendre_synth(to_dev(a)))[0][:, np.isin(g.theta, small.theta)]
        return np.sqrt((((x - F) ** 2).sum(axis=(0, 2, 3)) / (F ** 2).sum(axis=(0, 2, 3))).mean())

    assert err(large) < 1.5 * err(small)


@pytest.mark.parametrize("lmax", [300, 340, 383])
def test_error_over_all_rings(lmax):
    """One transform on given colatitudes: the rms error over the rings is that of the
    spin kernels on 64 slots at a time (within 8%: twice the most that the division by
    sin^2 t adds above the line; one form of recursion for 128 slots took 12 to 27%)."""
    sht = _sht()
    n = (lmax + 1) // 2
    g = si.gauss_geometry(lmax + 1, 8)
    north = np.arange(n)
    a = si.random_alm(lmax, lmax, 1, 2, spectrum="powerlaw", tag=785)
    F = oracle.synthesis(g, lmax, lmax, 2, a, rings=north, want_phases=True)[1][0][:, north]

    def err2(some, ref):
        p = sht.Plan(sht.Geometry.from_inputs(g.subset(some)), lmax, spin=2)
        return ((to_host(p.legendre_synth(to_dev(a)))[0][:, :ref.shape[1]] - ref) ** 2).sum()

    whole = err2(np.arange(g.nrings), F)
    parts = sum(err2(np.arange(y, min(y + 64, n)), F[:, y:y + 64]) for y in range(0, n, 64))
    assert whole < 1.08 ** 2 * parts
