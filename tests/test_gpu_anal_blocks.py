"""Spin-0 FP64 analysis on the matrix cores in its shapes of one, two and four column
blocks per work group (each with its own split of slots and outputs over the
wavefronts): plans large enough for the rule that chooses them, transform counts that
fill the blocks and that leave them partly empty, slots around the 256 of a pass, band
limits around the 32 degrees of a chunk, mmax < lmax, Inf and NaN.

Against the shape of one block, which the tuning can ask for: equal bit for bit (the
partial sums are added in one order).  That shape against the oracle on sampled m: the
parity tests' 1e-11, normwise.
"""
import os
import subprocess
import sys

import numpy as np
import pytest

import oracle
import sht_inputs as si
from gpu_util import rel_err, to_dev, to_host

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
TOL64 = 1e-11

# transforms -> (mmax from which the rule takes more than one block, blocks)
SHAPES = {9: (640, 2), 15: (640, 2), 16: (640, 2), 25: (320, 4), 31: (320, 4), 32: (320, 4), 41: (214, 2), 57: (160, 4)}


def _sht():
    import paper_1303_4945_amd as sht
    return sht


def _maps(g, ntrans, tag):
    rng = np.random.default_rng([13034945, tag])
    return rng.standard_normal((ntrans, 1, g.npix))


def _both(p, x, run="map2alm"):
    t = p.tuning()
    many = to_host(getattr(p, run)(x))
    assert t["anal_ncb"] == 2
    p.set_tuning(anal_ncb=1, anal_tpw=2)
    one = to_host(getattr(p, run)(x))
    p.set_tuning(**t)
    return many, one


@pytest.mark.parametrize("ntrans", list(SHAPES))
@pytest.mark.parametrize("nslots,extra", [(1, 0), (33, 31), (65, 1), (129, 32), (257, 5), (300, 33)])
def test_blocks_of_columns(ntrans, nslots, extra):
    sht = _sht()
    mmax = SHAPES[ntrans][0]
    lmax = mmax + extra
    if nslots > 1:
        g = si.gauss_geometry(2 * nslots - 1, 16, 0.1)   # one ring without a mirror
    else:
        g = si.gauss_geometry(2, 16, 0.1)
    p = sht.Plan(sht.Geometry.from_inputs(g), lmax, mmax, ntrans=ntrans)
    x = _maps(g, ntrans, 810 + ntrans)
    many, one = _both(p, to_dev(x))
    assert np.array_equal(many, one)
    sub = sorted({0, 7, 8, ntrans - 1})
    ms = [0, 1, mmax // 2, mmax - 1, mmax]
    ref = oracle.analysis(g, lmax, mmax, 0, np.ascontiguousarray(x[sub]), ms=ms)
    idx = np.isin(si.lm_arrays(lmax, mmax)[1], ms)
    assert rel_err(many[sub][:, :, idx], ref[:, :, idx]) < TOL64
    grad, grad1 = _both(p, to_dev(x), "alm2map_grad")
    assert np.array_equal(grad, grad1)


@pytest.mark.parametrize("ntrans", [16, 31])
def test_nonfinite_maps(ntrans):
    """An Inf or NaN pixel reaches every coefficient of its transform and no other."""
    sht = _sht()
    mmax = SHAPES[ntrans][0]
    g = si.gauss_geometry(70, 16, 0.1)
    p = sht.Plan(sht.Geometry.from_inputs(g), mmax, ntrans=ntrans, polar=False)
    x = _maps(g, ntrans, 830)
    clean = to_host(p.map2alm(to_dev(x)))
    x[8, 0, 5] = np.nan
    x[ntrans - 1, 0, 16 * 34 + 3] = np.inf
    many, one = _both(p, to_dev(x))
    assert np.array_equal(many, one, equal_nan=True)
    hit = [8, ntrans - 1]
    rest = [t for t in range(ntrans) if t not in hit]
    assert np.array_equal(many[rest], clean[rest])
    ms = si.lm_arrays(mmax, mmax)[1]
    for t in hit:
        assert not np.isfinite(many[t, 0, :, 0]).any() and not np.isfinite(many[t, 0, ms > 0, 1]).any()
        assert (many[t, 0, ms == 0, 1] == 0.0).all()


def test_rule_takes_these_shapes():
    """The shapes that the other tests mean to run are the ones that run."""
    script = ("import torch, paper_1303_4945_amd as sht\n"
              "for n, m in %r:\n"
              "    p = sht.Plan(sht.Geometry.gauss(8, 16), m, ntrans=n)\n"
              "    p.map2alm(torch.zeros(p.map_shape, dtype=torch.float64, device='cuda'))\n"
              "torch.cuda.synchronize()\n" % [(n, m) for n, (m, _) in SHAPES.items()])
    r = subprocess.run([sys.executable, "-u", "-c", script], cwd=ROOT, env=dict(os.environ, SHT_LOG="3"),
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-2000:]
    got = [int(ln.split(": ")[1].split()[0]) for ln in r.stderr.splitlines() if "two-step Legendre analysis" in ln]
    assert got == [b for _, b in SHAPES.values()]
