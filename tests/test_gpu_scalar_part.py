"""Spin-1 and spin-2 FP64 plans whose slots away from the poles run as spin-0
transforms of banded coefficients, against the oracle.

One transform (vector units, and the matrix-core kernels by tuning): sizes around the
rule that makes the split (more than 64 slots: 128 and 129 Gauss-Legendre rings stand
on either side of it), partly filled slot tiles, mmax < lmax, poles in the grid, rings
without a mirror, the polar criterion off, short rescale steps; every direction.
Several transforms (matrix cores, from 3.3e8 coefficients x slots on): rings and m of
each kind.  Tolerance: the parity tests' 1e-11, normwise (the sums' own rounding grows
about as lmax 2^-53: 1e-13 at lmax 1111).
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


def _fac(lmax, mmax):
    _, ms = si.lm_arrays(lmax, mmax)
    return np.where(ms > 0, 2.0, 1.0)[:, None]


def _unpaired(n):
    """Rings of both hemispheres, none the mirror of another."""
    g = si.gauss_geometry(n, 2 * n + 1)
    keep = np.arange(n)[np.arange(n) % 3 != 1] if n % 2 else np.arange(n)
    return g.subset(keep)


GRIDS = {
    "gl128": (lambda: si.gauss_geometry(128, 255), 127, 127),  # 64 slots: the spin kernels alone
    "gl129": (lambda: si.gauss_geometry(129, 257), 128, 128),  # 65 slots: 32 + 33
    "gl131": (lambda: si.gauss_geometry(131, 200), 127, 90),   # equator ring, aliased bins
    "ecp": (lambda: si.ecp_geometry(193, 194, si.ECP_CC), 95, 95),
    "hp": (lambda: si.healpix_geometry(40), 100, 100),
    "unpaired": (lambda: _unpaired(141), 99, 99),
    "low": (lambda: si.gauss_geometry(700, 24), 14, 11),       # degrees within one chunk
}


@pytest.mark.parametrize("valu", [1, 0])
@pytest.mark.parametrize("spin", [1, 2])
@pytest.mark.parametrize("grid", list(GRIDS))
def test_scalar_part_against_oracle(grid, spin, valu):
    sht = _sht()
    make, lmax, mmax = GRIDS[grid]
    g = make()
    p = sht.Plan(sht.Geometry.from_inputs(g), lmax, mmax, spin=spin)
    p.set_tuning(valu=valu)
    a = si.random_alm(lmax, mmax, 1, spin, spectrum="unit", tag=700 + spin)
    # entries that take no part: degrees below the spin
    ls, _ = si.lm_arrays(lmax, mmax)
    b = a.copy()
    b[:, :, ls < spin] = np.inf
    ref = oracle.synthesis(g, lmax, mmax, spin, a)
    pix = np.concatenate([np.arange(g.ofs[y], g.ofs[y] + g.nphi[y]) for y in range(g.nrings)])
    mp = to_host(p.alm2map(to_dev(b)))
    assert rel_err(mp[..., pix], ref[..., pix]) < TOL64
    assert rel_err(to_host(p.map2alm(to_dev(ref))), oracle.analysis(g, lmax, mmax, spin, ref)) < TOL64
    adj = oracle.adjoint_synthesis(g, lmax, mmax, spin, ref)
    assert rel_err(to_host(p.adjoint(to_dev(ref))), adj) < TOL64
    assert rel_err(to_host(p.alm2map_grad(to_dev(ref))), _fac(lmax, mmax) * adj) < TOL64
    # the staged steps run the same kernels
    F = p.legendre_synth(to_dev(a))
    assert rel_err(to_host(p.ring_synth(F))[..., pix], ref[..., pix]) < TOL64
    G = p.ring_anal(to_dev(ref))
    assert rel_err(to_host(p.legendre_anal(G)), to_host(p.map2alm(to_dev(ref)))) == 0.0


@pytest.mark.parametrize("spin,ntrans", [(1, 2), (2, 9)])
def test_scalar_part_of_several_transforms(spin, ntrans):
    sht = _sht()
    lmax, mmax = 1111, 1090
    g = si.gauss_geometry(lmax + 1, 2 * mmax + 1)
    p = sht.Plan(sht.Geometry.from_inputs(g), lmax, mmax, spin=spin, ntrans=ntrans)
    a = si.random_alm(lmax, mmax, ntrans, spin, spectrum="unit", tag=705 + spin)
    b = a.copy()
    b[:, :, si.lm_arrays(lmax, mmax)[0] < spin] = np.nan
    mp = to_host(p.alm2map(to_dev(b)))
    rings = [0, 1, 40, 63, 64, 65, 95, 96, 300, 555, 556, 600, 1015, 1016, 1047, 1048, 1110, 1111]
    sub = [0, ntrans - 1]
    ref = oracle.synthesis(g, lmax, mmax, spin, np.ascontiguousarray(a[sub]), rings=rings)
    for y in rings:
        px = slice(g.ofs[y], g.ofs[y] + g.nphi[y])
        assert rel_err(mp[sub][..., px], ref[..., px]) < TOL64, y
    ms = [0, 1, 2, 15, 500, 900, mmax]
    idx = np.isin(si.lm_arrays(lmax, mmax)[1], ms)
    ref = oracle.analysis(g, lmax, mmax, spin, np.ascontiguousarray(mp[sub]), ms=ms)
    got = to_host(p.map2alm(to_dev(mp)))[sub]
    assert rel_err(got[:, :, idx], ref[:, :, idx]) < TOL64


@pytest.mark.parametrize("valu", [1, 0])
def test_scalar_part_derivative_maps(valu):
    sht = _sht()
    lmax, mmax = 130, 97
    g = si.gauss_geometry(140, 201)
    p = sht.Plan(sht.Geometry.from_inputs(g), lmax, mmax, spin=1)
    p.set_tuning(valu=valu)
    a = si.random_alm(lmax, mmax, 1, 0, spectrum="unit", tag=710)
    ref = oracle.deriv_synthesis(g, lmax, mmax, a)
    assert rel_err(to_host(p.alm2map_deriv1(to_dev(a))), ref) < TOL64
    adj = oracle.deriv_adjoint(g, lmax, mmax, ref)
    assert rel_err(to_host(p.deriv1_adjoint(to_dev(ref))), adj) < TOL64
    assert rel_err(to_host(p.alm2map_deriv1_grad(to_dev(ref))), _fac(lmax, mmax) * adj) < TOL64


@pytest.mark.parametrize("kw", [dict(polar=False), dict(rescale_bits=128), dict(polar_T=20.0),
                                dict(real_harmonics=True)])
@pytest.mark.parametrize("valu", [1, 0])
def test_scalar_part_options(kw, valu):
    """Polar criterion off, short rescale steps, a criterion that drops most polar m
    (error of the dropped terms: exp(-20)), real storage."""
    sht = _sht()
    lmax = 140
    g = si.gauss_geometry(lmax + 1, 2 * lmax + 1)
    p = sht.Plan(sht.Geometry.from_inputs(g), lmax, spin=2, **kw)
    p.set_tuning(valu=valu)
    a = si.random_alm(lmax, lmax, 1, 2, spectrum="unit", tag=720)
    syn = oracle.synthesis_real if "real_harmonics" in kw else oracle.synthesis
    ana = oracle.analysis_real if "real_harmonics" in kw else oracle.analysis
    tol = 1e-7 if "polar_T" in kw else TOL64
    ref = syn(g, lmax, lmax, 2, a)
    assert rel_err(to_host(p.alm2map(to_dev(a))), ref) < tol
    assert rel_err(to_host(p.map2alm(to_dev(ref))), ana(g, lmax, lmax, 2, ref)) < tol


def test_scalar_part_follows_retuning_and_batches():
    """Vector and matrix kernels agree; batches (a plan of either kind and one without
    a scalar part) equal the plans bit for bit under every schedule; the
    allocation-free call equals the plain one."""
    import torch
    sht = _sht()
    plans, alms, maps = [], [], []
    for k, (lmax, nt) in enumerate([(130, 1), (150, 1), (100, 3)]):
        g = sht.Geometry.from_inputs(si.gauss_geometry(lmax + 1, 2 * lmax + 1))
        p = sht.Plan(g, lmax, spin=2, ntrans=nt)
        plans.append(p)
        alms.append(to_dev(si.random_alm(lmax, lmax, nt, 2, tag=730 + k)))
        maps.append(p.alm2map(alms[-1]))
        ref, back = to_host(maps[-1]), to_host(p.map2alm(maps[-1]))
        assert np.array_equal(to_host(p.execute_noalloc(sht.ALM2MAP, alms[-1])), ref)
        if nt == 1:
            p.set_tuning(valu=0)
            assert rel_err(to_host(p.alm2map(alms[-1])), ref) < 1e-13
            assert rel_err(to_host(p.map2alm(maps[-1])), back) < 1e-13
    plans[0].set_tuning(valu=1)
    assert np.array_equal(to_host(plans[0].alm2map(alms[0])), to_host(maps[0]))
    maps = [p.alm2map(x) for p, x in zip(plans, alms)]
    b = sht.Batch(plans)
    st = torch.cuda.Stream()
    for conc in (1, 0, 2):
        b.configure(sht.QUEUE_COST, conc)
        for s in (None, st):
            m = b.alm2map(alms, stream=s)
            a2 = b.map2alm(m, stream=s)
            torch.cuda.synchronize()
            for p, x, y, z in zip(plans, maps, m, a2):
                assert torch.equal(x, y)
                assert torch.equal(p.map2alm(x), z)
