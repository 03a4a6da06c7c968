"""A tuning file written before a plan shape had a scalar part holds timings of other
kernels: its lines are not taken for such plans."""
import pytest

pytestmark = pytest.mark.gpu


def test_lines_of_other_kernels(tmp_path, monkeypatch):
    import paper_1303_4945_amd as sht
    f = tmp_path / "tune.txt"
    monkeypatch.setenv("SHT_TUNE_CACHE", str(f))
    lmax = 140
    g = sht.Geometry.gauss(lmax + 1, 2 * lmax + 1)
    line = ("sht-tuning gfx950 lmax=%d mmax=%d spin=%d ntrans=1 nrings=%d prec=0"
            "|synth_ncb=1,synth_mblock=2,anal_ncb=1,anal_tpw=2,valu=0\n")
    f.write_text(line % (lmax, lmax, 2, lmax + 1) + line % (lmax, lmax, 0, lmax + 1))
    split, scalar = sht.Plan(g, lmax, spin=2), sht.Plan(g, lmax)
    default = split.tuning()
    for p in (split, scalar):
        p.autotune(0.0)
    assert split.tuning() == default and default["valu"] == 1
    assert scalar.tuning()["valu"] == 0   # this shape's kernels are the ones timed
    split.autotune(5.0)
    best = split.tuning()
    other = sht.Plan(g, lmax, spin=2)
    other.autotune(0.0)
    assert other.tuning() == best
