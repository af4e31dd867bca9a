"""Window layouts of the embedding on chains that do not fill the chip: windows
cut for many waves, the last window ending with the chain, both sides of the
last pass compared in one block, the sign-specialised LIN3 kernels, and calls
without a workspace; against the FP64 oracle at the tolerances of the other
embedding tests, or bitwise."""
import numpy as np
import pytest

from tests.gpu_util import RTOL, assert_rel, say, to_dev, to_host
from tests.test_gpu_embed import VARIANTS, make_case, run_gpu, run_oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
R = pytest.importorskip("paper_2001_10635_amd")


@pytest.fixture(scope="module")
def rc():
    r = R.Reach(0)
    yield r
    r.close()


@pytest.fixture(autouse=True)
def _reset_options(rc):
    yield
    for k in ("embed.E", "embed.K", "embed.S"):
        rc.set_option(k, 0)


@pytest.mark.parametrize("dtype", [np.float64, np.float32], ids=["f64", "f32"])
@pytest.mark.parametrize("variant", VARIANTS)
@pytest.mark.parametrize("n", [129, 383, 1537, 12001, 70001])
def test_default_windows_match_oracle(rc, variant, n, dtype):
    """Default plans of short chains: few cells per lane, several windows, odd
    lengths (the last window then starts at an odd cell)."""
    case = make_case(variant, n, dtype, seed=2000 + n)
    for nsteps in (9, 50):
        say(f"windows {variant} n={n} {np.dtype(dtype).name} N={nsteps}")
        g_lo, g_hi, st = run_gpu(rc, *case, nsteps)
        assert st == R.REACH_OK
        o_lo, o_hi = run_oracle(*case, nsteps)
        assert_rel(g_lo, o_lo, RTOL[np.dtype(dtype)], "lower")
        assert_rel(g_hi, o_hi, RTOL[np.dtype(dtype)], "upper")


@pytest.mark.parametrize("variant", VARIANTS)
@pytest.mark.parametrize("n", [385, 386, 1281, 3000])
@pytest.mark.parametrize("E,K", [(6, 11), (20, 17)])
def test_window_shapes_are_bitwise_equal(rc, variant, n, E, K):
    """The 6- and 20-cell tiles give the bits of the 2-cell ones, whether the
    chain fills the last window, ends just past one or just before."""
    S = 2 if variant.startswith("lin3") else 1
    if S == 2 and E == 20:
        pytest.skip("the coupled LIN3 chain has tiles of up to 16 cells")
    case = make_case(variant, n, np.float64, seed=n)
    outs = []
    for e, k in ((E, K), (2, 5)):
        for key, v in (("embed.S", S), ("embed.E", e), ("embed.K", k)):
            rc.set_option(key, v)
        say(f"window shape {variant} n={n} E={e} K={k}")
        outs.append(run_gpu(rc, *case, 23))
    assert outs[0][2] == outs[1][2] == R.REACH_OK
    assert np.array_equal(outs[0][0], outs[1][0]) and np.array_equal(outs[0][1], outs[1][1])


@pytest.mark.parametrize("dtype", [np.float64, np.float32], ids=["f64", "f32"])
@pytest.mark.parametrize("inputs", ["none", "scalar", "cell"])
@pytest.mark.parametrize("coef", [(0.5, -1.0, 0.75, 1.5), (-0.5, -1.0, 0.75, -1.5),
                                  (0.5, -1.0, -0.75, 1.5), (-0.5, -1.0, -0.75, -1.5),
                                  (0.0, -1.0, -0.75, 0.0), (-0.5, 0.0, 0.0, 1.5)],
                         ids=lambda c: "_".join(map(str, c)))
def test_lin3_sign_patterns_match_oracle(rc, coef, inputs, dtype):
    """Each sign of the couplings and of the input factor, at one cell per lane
    (odd lanes exchange sides) and several, one window and many."""
    _, _, lo, hi, pl, ph, dt = make_case("lin3_cell" if inputs == "cell" else "lin3", 777, dtype, 5)
    if inputs == "none":
        pl = ph = None
    rt = RTOL[np.dtype(dtype)]
    for n in (40, 777):
        c = (R.REACH_LIN3, coef, lo[:n], hi[:n], pl if inputs != "cell" else pl[:n],
             ph if inputs != "cell" else ph[:n], dt)
        o_lo, o_hi = run_oracle(*c, 19)
        for E, K in ((0, 0), (1, 3), (4, 6), (8, 9)):
            rc.set_option("embed.E", E)
            rc.set_option("embed.K", K)
            say(f"lin3 signs {coef} {inputs} {np.dtype(dtype).name} n={n} E={E} K={K}")
            g_lo, g_hi, st = run_gpu(rc, *c, 19)
            assert st == R.REACH_OK
            assert_rel(g_lo, o_lo, rt, "lower")
            assert_rel(g_hi, o_hi, rt, "upper")


@pytest.mark.parametrize("coef", [(-0.5, -1.0, 0.75, -1.5), (-0.5, -1.0, -0.75, 1.5),
                                  (0.5, -1.0, 0.75, 1.5), (0.0, -1.0, 0.0, 0.0)],
                         ids=lambda c: "_".join(map(str, c)))
@pytest.mark.parametrize("bad", [np.inf, -np.inf, np.nan])
def test_lin3_nonfinite_states_spread_as_in_the_oracle(rc, coef, bad):
    """A non-finite cell reaches both sides through the zero coefficients of
    the sign split (0 times inf is NaN): the same cells as in the oracle are
    finite, and those have its values."""
    _, _, lo, hi, pl, ph, dt = make_case("lin3", 1500, np.float64, 9)
    hi[700] = bad
    o_lo, o_hi = run_oracle(R.REACH_LIN3, coef, lo, hi, pl, ph, dt, 12)
    for E, K in ((0, 0), (1, 2), (4, 5), (8, 12)):
        rc.set_option("embed.E", E)
        rc.set_option("embed.K", K)
        say(f"lin3 non-finite {coef} {bad} E={E} K={K}")
        g_lo, g_hi, st = run_gpu(rc, R.REACH_LIN3, coef, lo, hi, pl, ph, dt, 12)
        assert st == R.REACH_E_NONFINITE
        for g, o in ((g_lo, o_lo), (g_hi, o_hi)):
            f = np.isfinite(o)
            assert np.array_equal(f, np.isfinite(g)) and not f.all()
            assert_rel(g[f], o[f], 1e-12, "finite cells")


@pytest.mark.parametrize("variant", ["ctm", "rd"])
@pytest.mark.parametrize("cell", [0, 1, 250, 2499, 4999])
def test_order_reported_from_any_window(rc, variant, cell):
    """lower > upper in one cell of a many-window chain reaches the status."""
    kind, prm, lo, hi, pl, ph, dt = make_case(variant, 5000, np.float64, seed=3)
    say(f"order {variant} cell={cell}")
    assert run_gpu(rc, kind, prm, lo, hi, pl, ph, dt, 20)[2] == R.REACH_OK
    lo[cell], hi[cell] = hi[cell] + 3.0, lo[cell]
    assert run_gpu(rc, kind, prm, lo, hi, pl, ph, dt, 1)[2] == R.REACH_E_ORDER


@pytest.mark.parametrize("variant,n,nsteps", [("ctm", 700, 60), ("rd", 1500, 33), ("lin3", 900, 40),
                                              ("rd", 3000, 20), ("ctm", 5000, 20)])
def test_calls_without_a_workspace_still_run(rc, variant, n, nsteps):
    """A chain that one window holds, or a run of one pass of the widest
    windows, needs no workspace; with one, more windows and passes run, with
    the same bits.  In place too."""
    kind, prm, lo, hi, pl, ph, dt = make_case(variant, n, np.float64, seed=n)
    ref = run_gpu(rc, kind, prm, lo, hi, pl, ph, dt, nsteps)
    dev = lambda a: None if a is None else to_dev(a)
    x_lo, x_hi, p_lo, p_hi = dev(lo), dev(hi), dev(pl), dev(ph)
    sysd = R.make_system(kind, n, prm, 0 if pl is None else pl.size)
    r_lo, r_hi = torch.empty_like(x_lo), torch.empty_like(x_hi)
    say(f"no workspace {variant} n={n} N={nsteps}")
    R.reach_embed_rk4(rc.ctx, sysd, R.REACH_F64, x_lo, x_hi, p_lo, p_hi, 0.0, dt, nsteps, r_lo, r_hi)
    assert rc.sync() == R.REACH_OK
    assert np.array_equal(to_host(r_lo), ref[0]) and np.array_equal(to_host(r_hi), ref[1])
    if n <= 1536:
        R.reach_embed_rk4(rc.ctx, sysd, R.REACH_F64, x_lo, x_hi, p_lo, p_hi, 0.0, dt, nsteps,
                          x_lo, x_hi)
        assert rc.sync() == R.REACH_OK
        assert np.array_equal(to_host(x_lo), ref[0]) and np.array_equal(to_host(x_hi), ref[1])


@pytest.mark.parametrize("variant", ["ctm", "rd_cell", "lin3"])
@pytest.mark.parametrize("n", [60, 700, 5001])
@pytest.mark.parametrize("nsteps", [0, 1, 9, 70])
def test_gb_results_over_its_inputs(rc, variant, n, nsteps):
    """Growth bound into the box's own arrays, and into an array that a per-cell
    input shares: the same bits as into arrays of its own (passes that write
    the box themselves, and those that leave it to the combining kernel)."""
    kind, prm, lo, hi, pl, ph, dt = make_case(variant, n, np.float64, seed=n + nsteps)
    dev = lambda a: None if a is None else to_dev(a)
    x_lo, x_hi, p_lo, p_hi = dev(lo), dev(hi), dev(pl), dev(ph)
    say(f"gb aliases {variant} n={n} N={nsteps}")
    a_lo, a_hi = rc.growth_bound(kind, prm, x_lo, x_hi, dt, nsteps, p_lo=p_lo, p_hi=p_hi)
    assert rc.sync() == R.REACH_OK
    y_lo, y_hi = x_lo.clone(), x_hi.clone()
    rc.growth_bound(kind, prm, y_lo, y_hi, dt, nsteps, p_lo=p_lo, p_hi=p_hi, r_lo=y_lo, r_hi=y_hi)
    assert rc.sync() == R.REACH_OK
    assert torch.equal(y_lo, a_lo) and torch.equal(y_hi, a_hi)
    if variant == "rd_cell":
        q_lo, q_hi = p_lo.clone(), p_hi.clone()
        rc.growth_bound(kind, prm, x_lo, x_hi, dt, nsteps, p_lo=q_lo, p_hi=q_hi, r_lo=q_lo,
                        r_hi=q_hi)
        assert rc.sync() == R.REACH_OK
        assert torch.equal(q_lo, a_lo) and torch.equal(q_hi, a_hi)
