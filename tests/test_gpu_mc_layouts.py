"""Layouts of the Monte Carlo kernel: several samples to a wave, lanes of uneven
cell counts, the widest lanes, few waves, and non-finite samples; against the
FP64 oracle at the tolerances of the other Monte Carlo tests."""
import numpy as np
import pytest

from tests.gpu_util import RTOL, assert_rel, say
from tests.test_gpu_embed import make_case
from tests.test_gpu_mc import oracle_mc, run_mc

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
R = pytest.importorskip("paper_2001_10635_amd")


@pytest.fixture(scope="module")
def rc():
    r = R.Reach(0)
    yield r
    r.close()


@pytest.fixture(autouse=True)
def _reset(rc):
    yield
    rc.set_option("mc.waves", 0)


@pytest.mark.parametrize("dtype", [np.float64, np.float32], ids=["f64", "f32"])
@pytest.mark.parametrize("variant", ["ctm", "rd", "rd_cell", "lin3", "lin3_cell"])
@pytest.mark.parametrize("n,m,nsteps", [(2, 9001, 4), (16, 9001, 4), (33, 5003, 5), (64, 5003, 3),
                                        (130, 3001, 3), (300, 3001, 2), (777, 2051, 2)])
def test_mc_samples_sharing_a_wave_match_oracle(rc, variant, n, m, nsteps, dtype):
    """More samples than the SIMDs hold waves: wide lanes, several samples per
    wave, the last wave's places not all taken."""
    case = make_case(variant, n, dtype, seed=4000 + n)
    say(f"mc layout {variant} n={n} m={m} {np.dtype(dtype).name}")
    g_min, g_max, st = run_mc(rc, *case, nsteps, m, 7 + n, s0=3)
    assert st == R.REACH_OK
    o_min, o_max = oracle_mc(*case, nsteps, m, 7 + n, dtype, s0=3)
    assert_rel(g_min, o_min, RTOL[np.dtype(dtype)], "min")
    assert_rel(g_max, o_max, RTOL[np.dtype(dtype)], "max")


@pytest.mark.parametrize("variant", ["ctm", "rd_cell"])
@pytest.mark.parametrize("n", [2049, 2561, 3585, 3841, 3842, 3843, 4095])
def test_mc_f32_widest_lanes_match_oracle(rc, variant, n):
    """FP32 lengths next to the edges of the widest lanes (3841 and 3842 fit no
    segment layout)."""
    case = make_case(variant, n, np.float32, seed=n)
    say(f"mc widest {variant} n={n}")
    g_min, g_max, st = run_mc(rc, *case, 9, 12, n)
    assert st == R.REACH_OK
    o_min, o_max = oracle_mc(*case, 9, 12, n, np.float32)
    assert_rel(g_min, o_min, 1e-5, "min")
    assert_rel(g_max, o_max, 1e-5, "max")


@pytest.mark.parametrize("n,m,waves", [(64, 50, 1), (100, 50, 3), (1100, 21, 5), (16, 3000, 4),
                                       (2048, 9, 2)])
def test_mc_few_waves_give_the_same_bits(rc, n, m, waves):
    """Samples per wave and workgroups do not change a value."""
    case = make_case("rd", n, np.float64, seed=n)
    ref = run_mc(rc, *case, 11, m, 3)
    rc.set_option("mc.waves", waves)
    say(f"mc waves={waves} n={n} m={m}")
    got = run_mc(rc, *case, 11, m, 3)
    assert got[2] == ref[2] == R.REACH_OK
    assert np.array_equal(got[0], ref[0]) and np.array_equal(got[1], ref[1])


@pytest.mark.parametrize("dtype", [np.float64, np.float32], ids=["f64", "f32"])
@pytest.mark.parametrize("n,m", [(64, 40), (64, 5003), (300, 40)])
@pytest.mark.parametrize("bad", [np.nan, np.inf, -np.inf])
def test_mc_nonfinite_samples_reach_min_and_max(rc, n, m, bad, dtype):
    """A non-finite box end: the same dimensions as in the oracle are NaN in both
    min and max (a NaN sample is never dropped) and the status says so."""
    kind, prm, lo, hi, pl, ph, dt = make_case("rd", n, dtype, seed=n)
    hi[n // 3] = bad
    say(f"mc non-finite {bad} n={n} m={m} {np.dtype(dtype).name}")
    g_min, g_max, st = run_mc(rc, kind, prm, lo, hi, pl, ph, dt, 2, m, 5)
    assert st == R.REACH_E_NONFINITE
    o_min, o_max = oracle_mc(kind, prm, lo, hi, pl, ph, dt, 2, m, 5, dtype)
    for g, o in ((g_min, o_min), (g_max, o_max)):
        f = np.isfinite(o)
        assert np.array_equal(f, np.isfinite(g)) and not f.all()
        assert_rel(g[f], o[f], RTOL[np.dtype(dtype)], "finite dimensions")


@pytest.mark.parametrize("variant", ["ctm", "rd", "lin3"])
@pytest.mark.parametrize("n", [40, 64, 100])
def test_mc_samples_sharing_a_wave_give_the_bits_of_samples_alone(variant, n, capfd, monkeypatch):
    """Many samples share waves, a few take one each (the calls' log says so): the
    min / max of a large range is bit for bit that of the small ones it holds."""
    import re
    monkeypatch.setenv("REACH_LOG", "1")
    r = R.Reach(0)
    try:
        kind, prm, lo, hi, pl, ph, dt = make_case(variant, n, np.float64, seed=n)
        dev = lambda a: None if a is None else torch.from_numpy(np.ascontiguousarray(a)).cuda()
        args = (kind, prm, dev(lo), dev(hi), dt, 6)
        kw = dict(p_lo=dev(pl), p_hi=dev(ph))
        say(f"mc shared waves {variant} n={n}")
        capfd.readouterr()
        mn, mx = r.montecarlo(*args, 20000, 3, **kw)
        parts = [r.montecarlo(*args, 250, 3, s0=s, **kw) for s in range(0, 20000, 250)]
        assert r.sync() == R.REACH_OK
        spw = [int(x) for x in re.findall(r'"samples_per_wave": (\d+)', capfd.readouterr().err)]
        assert spw[0] > 1 and set(spw[1:]) == {1}
        assert torch.equal(mn, torch.stack([p[0] for p in parts]).min(0).values)
        assert torch.equal(mx, torch.stack([p[1] for p in parts]).max(0).values)
    finally:
        r.close()
