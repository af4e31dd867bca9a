"""Embeddings in flight at the same time, captured, or with result arrays that
overlap their inputs: the same bits as the call by itself."""
import numpy as np
import pytest

from tests.gpu_util import say, to_dev
from tests.test_gpu_embed import make_case

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
R = pytest.importorskip("paper_2001_10635_amd")

NP = {R.REACH_F64: np.float64, R.REACH_F32: np.float32}


@pytest.fixture(scope="module")
def rc():
    r = R.Reach(0)
    yield r
    r.close()


def dev_case(variant, n, dtc, seed):
    """(kind, prm, dt, device arrays x_lo, x_hi, p_lo, p_hi) of one chain."""
    kind, prm, lo, hi, pl, ph, dt = make_case(variant, n, NP[dtc], seed=seed)
    return (kind, prm, dt) + tuple(None if a is None else to_dev(a) for a in (lo, hi, pl, ph))


def embed(rc, case, dtc, nsteps, r_lo, r_hi, ws=None, stream=None):
    kind, prm, dt, x_lo, x_hi, p_lo, p_hi = case
    sysd = R.make_system(kind, x_lo.numel(), prm, 0 if p_lo is None else p_lo.numel())
    R.reach_embed_rk4(rc.ctx, sysd, dtc, x_lo, x_hi, p_lo, p_hi, 0.0, dt, nsteps, r_lo, r_hi, ws,
                      0 if ws is None else ws.numel(), stream)


@pytest.mark.parametrize("variant,n,dtc,nsteps", [
    ("rd", 1000, R.REACH_F64, 100), ("ctm", 4000, R.REACH_F32, 90), ("lin3_cell", 900, R.REACH_F64, 40),
    ("rd_cell", 2048, R.REACH_F64, 60), ("rd", 5000, R.REACH_F64, 20), ("ctm", 9000, R.REACH_F32, 12),
    ("lin3_cell", 5000, R.REACH_F64, 12)])
@pytest.mark.parametrize("streams", [2, 18])
def test_streams_share_one_object(rc, variant, n, dtc, nsteps, streams):
    """Chains that one window holds, and runs of one pass, on several streams of
    one object (more streams than the context keeps scratch slots for), and with
    one workspace given to all: they use none, so no call changes another's box."""
    cases = [dev_case(variant, n, dtc, 40 + k) for k in range(streams)]
    refs = []
    for c in cases:
        refs.append(rc.embed(c[0], c[1], c[3], c[4], c[2], nsteps, p_lo=c[5], p_hi=c[6]))
        assert rc.sync() == R.REACH_OK
    st = [torch.cuda.Stream() for _ in range(streams)]
    ws = torch.empty(2 * n * cases[0][3].element_size(), dtype=torch.uint8, device="cuda")
    outs = [(torch.empty_like(c[3]), torch.empty_like(c[4])) for c in cases]
    torch.cuda.synchronize()
    say(f"streams {variant} n={n} N={nsteps} streams={streams}")
    for shared in (False, True):
        for lo, hi in outs:
            lo.zero_()
            hi.zero_()
        torch.cuda.synchronize()
        for _ in range(3):
            for c, s, (lo, hi) in zip(cases, st, outs):
                if shared:
                    embed(rc, c, dtc, nsteps, lo, hi, ws, s)
                else:
                    rc.embed(c[0], c[1], c[3], c[4], c[2], nsteps, p_lo=c[5], p_hi=c[6], r_lo=lo,
                             r_hi=hi, stream=s)
        torch.cuda.synchronize()
        assert rc.sync() == R.REACH_OK
        for (lo, hi), (a, b) in zip(outs, refs):
            assert torch.equal(lo, a) and torch.equal(hi, b)


def test_workspace_bytes_of_chains_one_window_holds(rc):
    """No workspace: nothing of the caller's is written but the results."""
    for n in (1, 64, 129, 1000, 2048):
        assert R.reach_workspace_bytes(rc.ctx, R.make_system(R.REACH_RD, n, (1.0,), 0),
                                       R.REACH_F64, 0) == 0
    assert R.reach_workspace_bytes(rc.ctx, R.make_system(R.REACH_RD, 3000, (1.0,), 0),
                                   R.REACH_F64, 0) == 2 * 3000 * 8


@pytest.mark.parametrize("variant", ["ctm", "rd", "lin3"])
@pytest.mark.parametrize("n", [200, 1000])
def test_captured_call_keeps_to_its_own_arrays(rc, variant, n):
    """A captured embedding replays beside eager ones of the same object and
    stream, and after the object's workspace has grown."""
    c = dev_case(variant, n, R.REACH_F64, 3)
    other = dev_case(variant, n, R.REACH_F64, 4)
    big = dev_case(variant, 70001, R.REACH_F64, 5)
    ref = rc.embed(c[0], c[1], c[3], c[4], c[2], 70, p_lo=c[5], p_hi=c[6])
    oref = rc.embed(other[0], other[1], other[3], other[4], other[2], 70, p_lo=other[5],
                    p_hi=other[6])
    assert rc.sync() == R.REACH_OK
    lo, hi = torch.empty_like(c[3]), torch.empty_like(c[4])
    o_lo, o_hi = torch.empty_like(c[3]), torch.empty_like(c[4])
    s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
    g = torch.cuda.CUDAGraph()
    say(f"capture {variant} n={n}")
    with torch.cuda.graph(g, stream=s1):
        rc.embed(c[0], c[1], c[3], c[4], c[2], 70, p_lo=c[5], p_hi=c[6], r_lo=lo, r_hi=hi)
    for k in range(4):
        lo.zero_()
        o_lo.zero_()
        torch.cuda.synchronize()
        with torch.cuda.stream(s2):
            g.replay()
        rc.embed(other[0], other[1], other[3], other[4], other[2], 70, p_lo=other[5],
                 p_hi=other[6], r_lo=o_lo, r_hi=o_hi, stream=s1)
        torch.cuda.synchronize()
        assert rc.sync() == R.REACH_OK
        assert torch.equal(lo, ref[0]) and torch.equal(hi, ref[1])
        assert torch.equal(o_lo, oref[0]) and torch.equal(o_hi, oref[1])
        if k == 1:
            rc.embed(big[0], big[1], big[3], big[4], big[2], 70, p_lo=big[5], p_hi=big[6])


@pytest.mark.parametrize("variant", ["rd_cell", "lin3_cell", "rd"])
@pytest.mark.parametrize("n", [60, 500, 1000])
@pytest.mark.parametrize("nsteps", [1, 20, 100])
def test_results_over_inputs(rc, variant, n, nsteps):
    """A chain that one window holds, its box into the arrays of its inputs, and
    into arrays a few cells past the box's own: the same bits as into others."""
    c = dev_case(variant, n, R.REACH_F64, 70 + n)
    ref = rc.embed(c[0], c[1], c[3], c[4], c[2], nsteps, p_lo=c[5], p_hi=c[6])
    assert rc.sync() == R.REACH_OK
    say(f"results over inputs {variant} n={n} N={nsteps}")
    # (a scalar input: the first cell of the result)
    q_lo, q_hi = torch.zeros_like(c[3]), torch.zeros_like(c[4])
    k = c[5].numel()
    q_lo[:k], q_hi[:k] = c[5], c[6]
    d = c[:5] + (q_lo[:k], q_hi[:k])
    embed(rc, d, R.REACH_F64, nsteps, q_lo, q_hi)
    assert rc.sync() == R.REACH_OK
    assert torch.equal(q_lo, ref[0]) and torch.equal(q_hi, ref[1])
    # the lower box shifted by 3 cells (each side's wave reads before it writes)
    y = torch.zeros(n + 3, dtype=torch.float64, device="cuda")
    y[:n] = c[3]
    hi = torch.empty_like(c[4])
    embed(rc, c[:3] + (y[:n],) + c[4:], R.REACH_F64, nsteps, y[3:], hi)
    assert rc.sync() == R.REACH_OK
    assert torch.equal(y[3:], ref[0]) and torch.equal(hi, ref[1])


@pytest.mark.parametrize("variant", ["ctm", "rd", "rd_cell", "lin3"])
@pytest.mark.parametrize("n", [1, 64, 100, 128, 700, 1536, 5000])
@pytest.mark.parametrize("nsteps", [1, 7, 45])
@pytest.mark.parametrize("K", [0, 3])
def test_crossed_results(rc, variant, n, nsteps, K):
    """r_lo over x_hi and r_hi over x_lo, one of the two, and both sides from one
    array that a result replaces: each side's wave reads the box first."""
    c = dev_case(variant, n, R.REACH_F64, 90 + n)
    ref = rc.embed(c[0], c[1], c[3], c[4], c[2], nsteps, p_lo=c[5], p_hi=c[6])
    one = rc.embed(c[0], c[1], c[3], c[3], c[2], nsteps, p_lo=c[5], p_hi=c[6])
    assert rc.sync() == R.REACH_OK
    rc.set_option("embed.K", K)
    ws = torch.empty(2 * n * 8, dtype=torch.uint8, device="cuda")
    say(f"crossed {variant} n={n} N={nsteps} K={K}")
    try:
        for cross in ("both", "lo", "hi", "same"):
            lo, hi = c[3].clone(), c[4].clone()
            if cross == "same":
                r_lo, r_hi, want, hi = lo, torch.empty_like(lo), one, lo
            else:
                r_lo = torch.empty_like(lo) if cross == "hi" else hi
                r_hi = torch.empty_like(hi) if cross == "lo" else lo
                want = ref
            embed(rc, c[:3] + (lo, hi) + c[5:], R.REACH_F64, nsteps, r_lo, r_hi, ws)
            assert rc.sync() == R.REACH_OK
            assert torch.equal(r_lo, want[0]) and torch.equal(r_hi, want[1]), cross
    finally:
        rc.set_option("embed.K", 0)


@pytest.mark.parametrize("pack", [0, 1, 2])
@pytest.mark.parametrize("split", [0, 1])
@pytest.mark.parametrize("nq", [3, 80, 4300])
def test_batch_crossed_results(rc, pack, split, nq):
    """Batches in which some queries' results replace the other side's box or
    input, run packed or not: the boxes of the same queries with results of
    their own.  4300 queries pack by default, the longest one side per wave."""
    qs, refs, keep = [], [], []
    for k in range(nq):
        variant = ("ctm", "rd", "lin3")[k % 3]
        n, nsteps = 5 + (37 * k) % 200, 1000 if k % 40 == 1 else 8 + k % 30
        c = dev_case(variant, n, R.REACH_F64, 300 + k % 17)
        kind, prm, dt, lo, hi, pl, ph = c
        n_in = 0 if pl is None else 1
        own = [torch.empty_like(lo), torch.empty_like(hi)]
        refs.append((kind, n, prm, lo, hi, own, dt, nsteps, pl, ph, n_in))
        x_lo, x_hi = lo.clone(), hi.clone()
        r_lo, r_hi = torch.empty_like(lo), torch.empty_like(hi)
        how = k % 5
        if how == 0:
            r_lo, r_hi = x_hi, x_lo
        elif how == 1:
            r_lo = x_hi
        elif how == 2 and n_in:            # the results over the other side's input
            r_lo[:1], r_hi[:1] = ph, pl
            pl, ph = r_hi[:1], r_lo[:1]
        elif how == 3:
            r_lo, r_hi = x_lo, x_hi
        qs.append((kind, n, prm, x_lo, x_hi, r_lo, r_hi, dt, nsteps, pl, ph, n_in))
    make = lambda q, r_lo, r_hi: R.make_query(q[0], q[1], q[2], R.REACH_F64, q[3], q[4], r_lo, r_hi,
                                              q[-5], q[-4], q[-3], q[-2], n_in=q[-1])
    a = R.query_array([make(q, *q[5]) for q in refs])
    b = R.query_array([make(q, q[5], q[6]) for q in qs])
    nb = R.reach_batch_workspace_bytes(nq)
    ws = torch.empty(nb, dtype=torch.uint8, device="cuda")
    say(f"batch crossed nq={nq} pack={pack} split={split}")
    R.reach_embed_rk4_each(rc.ctx, a)
    assert rc.sync() == R.REACH_OK
    try:
        rc.set_option("batch.pack", pack)
        rc.set_option("batch.split", split)
        R.reach_embed_rk4_batch(rc.ctx, b, ws, nb)
        assert rc.sync() == R.REACH_OK
    finally:
        rc.set_option("batch.pack", 0)
        rc.set_option("batch.split", 0)
    for k, (q, ref) in enumerate(zip(qs, refs)):
        assert torch.equal(q[5], ref[5][0]) and torch.equal(q[6], ref[5][1]), k


@pytest.mark.parametrize("variant", ["lin3", "lin3_cell"])
@pytest.mark.parametrize("n", [1025, 5000])
@pytest.mark.parametrize("nsteps", [1, 10, 11, 12])
def test_lin3_runs_of_one_pass_need_no_workspace(rc, variant, n, nsteps):
    c = dev_case(variant, n, R.REACH_F64, 7)
    ref = rc.embed(c[0], c[1], c[3], c[4], c[2], nsteps, p_lo=c[5], p_hi=c[6])
    lo, hi = torch.empty_like(c[3]), torch.empty_like(c[4])
    say(f"no workspace {variant} n={n} N={nsteps}")
    embed(rc, c, R.REACH_F64, nsteps, lo, hi)
    assert rc.sync() == R.REACH_OK
    assert torch.equal(lo, ref[0]) and torch.equal(hi, ref[1])


@pytest.mark.parametrize("kind,prm,n,dtc,cut", [
    (R.REACH_RD, (1.0,), 130, R.REACH_F64, False), (R.REACH_RD, (1.0,), 384, R.REACH_F64, False),
    (R.REACH_RD, (1.0,), 1000, R.REACH_F64, True), (R.REACH_LIN3, (-0.5, -1.0, 0.75, -1.5), 130,
                                                    R.REACH_F64, False),
    (R.REACH_CTM, (0.5, 1 / 6, 40.0, 20.0), 4096, R.REACH_F32, True)])
def test_short_chains_stay_in_one_window_unless_it_pays(rc, kind, prm, n, dtc, cut):
    """100 steps: cut only where eight streams at once do not lose by it."""
    plan = R.reach_plan_embed(rc.ctx, R.make_system(kind, n, prm, 0), dtc, 100)
    assert (plan["tiles"] > 1) == cut and (plan["passes"] > 1) == cut


@pytest.mark.parametrize("n", [100003, 500001])
def test_autotuner_keeps_a_default_it_has_not_beaten(tmp_path, monkeypatch, n):
    """The default shape of these sizes is 6 or 20 cells a lane, widths the scan
    leaves out: it is timed all the same, and where it wins nothing is recorded
    for the bucket's other sizes."""
    monkeypatch.setenv("REACH_AUTOTUNE_CACHE", str(tmp_path / "tune.txt"))
    r = R.Reach(0)
    try:
        c = dev_case("rd", n, R.REACH_F64, 5)
        sysd = R.make_system(c[0], n, c[1], 1)
        other = R.make_system(c[0], n * 15 // 16, c[1], 1)   # of the same bucket
        before = [R.reach_plan_embed(r.ctx, x, R.REACH_F64, 1000) for x in (sysd, other)]
        ws = torch.empty(2 * n * 8, dtype=torch.uint8, device="cuda")
        lo, hi = torch.empty_like(c[3]), torch.empty_like(c[4])
        say(f"autotune n={n}")
        best = R.reach_autotune_embed(r.ctx, sysd, R.REACH_F64, c[3], c[4], c[5], c[6], c[2], 8,
                                      lo, hi, ws, ws.numel())
        after = [R.reach_plan_embed(r.ctx, x, R.REACH_F64, 1000) for x in (sysd, other)]
        line = (tmp_path / "tune.txt").read_text().split()
        if best["E"] == before[0]["E"]:
            assert after == before and line[7] == "0"
        else:
            assert line[7] == str(best["E"]) == str(after[1]["E"])
    finally:
        r.close()


def test_tuned_shape_leaves_chains_of_one_window_alone(tmp_path, monkeypatch):
    arch = torch.cuda.get_device_properties(0).gcnArchName.split(":")[0]
    cache = tmp_path / "tune.txt"
    sysd = [R.make_system(R.REACH_RD, n, (1.0,), 0) for n in (1500, 5000)]
    plans = []
    for text in ("", f"reach2 embed {arch} 2 0 10 0 16 6 1 1.0\nreach2 embed {arch} 2 0 12 0 16 6 1 1.0\n",
                 f"reach2 embed {arch} 2 0 12 0 16 6 1 1.0\nreach2 embed {arch} 2 0 12 0 0 0 0 1.0\n"):
        cache.write_text(text)
        monkeypatch.setenv("REACH_AUTOTUNE_CACHE", str(cache))
        r = R.Reach(0)
        plans.append([R.reach_plan_embed(r.ctx, s, R.REACH_F64, 100) for s in sysd])
        r.close()
    assert plans[1][0] == plans[0][0] and plans[1][0]["tiles"] > 1
    assert (plans[1][1]["E"], plans[1][1]["K"]) == (16, 6)
    assert plans[2] == plans[0]


@pytest.mark.parametrize("n,K", [(100, 16), (100, 31), (128, 20), (600, 127), (768, 96), (1200, 160)])
def test_growth_bound_takes_every_K_its_window_holds(rc, n, K):
    """Option gb.K without gb.E, steps per pass that 4, 16 and 24 cells a lane
    hold: the bits of the default plan; the first one past them is refused."""
    c = dev_case("rd", n, R.REACH_F64, 11)
    ref = rc.growth_bound(c[0], c[1], c[3], c[4], c[2], 200, p_lo=c[5], p_hi=c[6])
    assert rc.sync() == R.REACH_OK
    rc.set_option("gb.K", K)
    try:
        say(f"gb.K={K} n={n}")
        got = rc.growth_bound(c[0], c[1], c[3], c[4], c[2], 200, p_lo=c[5], p_hi=c[6])
        assert rc.sync() == R.REACH_OK
        assert torch.equal(got[0], ref[0]) and torch.equal(got[1], ref[1])
        rc.set_option("gb.K", 8 * {100: 4, 128: 4, 600: 16, 768: 16, 1200: 24}[n])
        with pytest.raises(R.ReachError):
            rc.growth_bound(c[0], c[1], c[3], c[4], c[2], 200, p_lo=c[5], p_hi=c[6])
    finally:
        rc.set_option("gb.K", 0)


@pytest.mark.parametrize("kinds", [("ctm", "rd"), ("lin3",), ("ctm", "lin3", "rd")])
@pytest.mark.parametrize("nq", [90, 1100, 4300, 6500])
@pytest.mark.parametrize("long", [20, 1000])
def test_batch_layouts_equal_single_runs(rc, kinds, nq, long):
    """Default batches, unpacked and packed, of equally short queries (every item
    whole) and of some much longer ones (narrowed packs, the longest items one
    side per wave): every box is the one the query gets by itself, and flags
    of whole items, sides and packs reach the status."""
    base = {k: [dev_case(k, n, R.REACH_F64, 500 + n) for n in (4, 33, 64, 65, 200, 257, 512)]
            for k in kinds}
    a, b, outs = [], [], []
    for k in range(nq):
        cs = base[kinds[k % len(kinds)]]
        kind, prm, dt, lo, hi, pl, ph = cs[(k // 3) % len(cs)]
        nsteps = long if k % 50 == 7 else 12 + k % 9
        o = [torch.empty_like(lo) for _ in range(4)]
        outs.append(o)
        for dst, r in ((a, o[:2]), (b, o[2:])):
            dst.append(R.make_query(kind, lo.numel(), prm, R.REACH_F64, lo, hi, r[0], r[1], dt, nsteps,
                                    pl, ph, n_in=0 if pl is None else 1))
    nb = R.reach_batch_workspace_bytes(nq)
    ws = torch.empty(nb, dtype=torch.uint8, device="cuda")
    say(f"batch layouts {kinds} nq={nq} long={long}")
    R.reach_embed_rk4_each(rc.ctx, R.query_array(a))
    assert rc.sync() == R.REACH_OK
    arr = R.query_array(b)
    for _ in range(2):
        R.reach_embed_rk4_batch(rc.ctx, arr, ws, nb)
    assert rc.sync() == R.REACH_OK
    for k, o in enumerate(outs):
        assert torch.equal(o[0], o[2]) and torch.equal(o[1], o[3]), k
    for k in (0, 7, nq - 1):
        for bad, want in ((float("inf"), R.REACH_E_NONFINITE), (None, R.REACH_E_ORDER)):
            q = b[k]
            n = q.sys.n
            lo = torch.ones(n, dtype=torch.float64, device="cuda")
            hi = lo + 0.1
            if bad is None:
                lo[n // 2] = 9.0
            else:
                hi[n // 2] = bad
            x = R.query_array(b)
            x[k].x_lo, x[k].x_hi = lo.data_ptr(), hi.data_ptr()
            x[k].nsteps = 1 if bad is None else q.nsteps
            R.reach_embed_rk4_batch(rc.ctx, x, ws, nb)
            assert rc.sync() == want, (k, bad)


def shaped(rc, call, c, nsteps, E, K, over=False):
    """One call at E cells a lane and K steps a pass, with its results over the box if
    `over`: (status, lower, upper)."""
    kind, prm, dt, x_lo, x_hi, p_lo, p_hi = c
    if over:
        x_lo, x_hi = x_lo.clone(), x_hi.clone()
    r = (x_lo, x_hi) if over else (torch.empty_like(x_lo), torch.empty_like(x_hi))
    names = ("gb.E", "gb.K") if call == "gb" else ("embed.E", "embed.K", "embed.S")
    for name, v in zip(names, (E, K, 1)):
        rc.set_option(name, v)
    try:
        f = rc.growth_bound if call == "gb" else rc.embed
        f(kind, prm, x_lo, x_hi, dt, nsteps, p_lo=p_lo, p_hi=p_hi, r_lo=r[0], r_hi=r[1])
        return (rc.sync(),) + r
    finally:
        for name in names:
            rc.set_option(name, 0)


@pytest.mark.parametrize("call", ["gb", "embed"])
@pytest.mark.parametrize("variant", ["rd", "ctm", "rd_cell"])
@pytest.mark.parametrize("windows", [256, 257, 400, 512, 513, 1300])
def test_windows_of_more_than_one_and_two_a_compute_unit(rc, call, variant, windows):
    """FP64 windows just below, in and past the range where the sides of a window
    are blocks of their own and a last kernel brings them together: the bits of
    another shape, also with the results over the box, and the same flags."""
    E, K = 8, 20
    n = 64 * E + (windows - 1) * (64 * E - 8 * K) - 3
    c = dev_case(variant, n, R.REACH_F64, windows)
    for nsteps in (K, 3 * K):
        say(f"{call} {variant} windows={windows} N={nsteps}")
        ref = shaped(rc, call, c, nsteps, 4, 9)
        assert ref[0] == R.REACH_OK
        for over in (False, True):
            got = shaped(rc, call, c, nsteps, E, K, over)
            assert got[0] == R.REACH_OK
            assert torch.equal(got[1], ref[1]) and torch.equal(got[2], ref[2])
    for bad, want in ((float("inf"), R.REACH_E_NONFINITE), (None, R.REACH_E_ORDER)):
        lo, hi = c[3].clone(), c[4].clone()
        part = slice(n // 2, n // 2 + 700)
        if bad is None:
            lo[part], hi[part] = c[4][part], c[3][part]
        else:
            hi[n // 2] = bad
        # (so short a time that the inputs' interval does not open the crossed part again)
        case = c[:2] + (0.01 * c[2], lo, hi) + c[5:]
        assert shaped(rc, call, case, K, E, K)[0] == want
        assert shaped(rc, call, c, K, E, K)[0] == R.REACH_OK
