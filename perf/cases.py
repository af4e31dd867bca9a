"""Performance cases of the interval-reachability library.

Each case is one call (or one burst of calls) that a user of the library makes
through its public entry points, on the box recipes of this repository's
workloads, drawn on the GPU from a seed:

  embed    reach_embed_rk4: the mixed-monotonicity box of a chain
  tube     reach_embed_rk4_tube: the box after every few steps
  growth   reach_growth_bound: the contraction / growth-bound box
  mc       reach_montecarlo: the sampled box
  heat     reach_embed_rk4 of the 3-D heat grid
  batch    reach_embed_rk4_batch: many small queries at once

``listed`` holds the standing cases and ``draw`` gives others of the same
ranges; ``exact`` recomputes a case in plain torch at 64 bits.
"""
from __future__ import annotations

import math

import torch

import paper_2001_10635_amd as R

DEV = "cuda:0"

# systems and boxes of the repository's workloads
CTM_PRM = (0.5, 1.0 / 6.0, 40.0, 20.0)     # v, w, c, q
RD_PRM = (1.0,)                            # h
LIN3_PRM = (-0.5, -1.0, 0.75, -1.5)        # aL, aD, aR, b
HEAT_ALPHA = 1.0e-5
DT = {"ctm": 0.01, "rd": 0.1, "lin3": 0.05, "heat": 0.02}
KIND = {"ctm": R.REACH_CTM, "rd": R.REACH_RD, "lin3": R.REACH_LIN3, "heat": R.REACH_HEAT3D}
PRM = {"ctm": CTM_PRM, "rd": RD_PRM, "lin3": LIN3_PRM}
U_LO, U_HI = -0.1, 0.1
# operations of one state-step (one cell and side, one RK4 step): four
# right-hand sides, three stage inputs of 2, the weighted sum 5, the update 2
OPS = {"ctm": 4 * 6 + 13, "rd": 4 * 8 + 13, "lin3": 4 * 7 + 13, "heat": 40}
# most work of a drawn case: the largest listed ones' (2^26 cells of both
# sides, 100 steps of the reaction-diffusion chain)
MOST_FLOPS = 45 * 2.0 * (1 << 26) * 100


# ------------------------------------------------------------------- cases

def listed():
    return [
        # the smallest embedding: one road of 64 links, where launches and the
        # serial chain of stages count
        dict(name="embed_ctm_64_f64", call="embed", system="ctm", n=64, n_in=0, f64=True,
             steps=100),
        # its Monte Carlo check with 1000 samples
        dict(name="mc_ctm_64_f64", call="mc", system="ctm", n=64, n_in=0, f64=True, steps=100,
             m=1000),
        # an ordinary discretised chain of odd length: more than one wavefront's
        # window, far less than fills the chip
        dict(name="embed_rd_100003_f64", call="embed", system="rd", n=100003, n_in=1, f64=True,
             steps=400),
        # a reach tube of a 12000-state system in single precision
        dict(name="tube_ctm_12000_f32", call="tube", system="ctm", n=12000, n_in=0, f64=False,
             steps=200, every=20),
        # coupled lower and upper sides, an input for every cell
        dict(name="embed_lin3_2p20_f64", call="embed", system="lin3", n=1 << 20, n_in=1 << 20,
             f64=True, steps=100),
        # the benchmark's chain at its size, a tenth of its steps
        dict(name="embed_rd_2p26_f64", call="embed", system="rd", n=1 << 26, n_in=1, f64=True,
             steps=100),
        # the growth-bound method on a middling chain
        dict(name="growth_rd_1000000_f64", call="growth", system="rd", n=1000000, n_in=1,
             f64=True, steps=200),
        # the Monte Carlo workload at its size, fewer samples and steps
        dict(name="mc_ctm_4096_f32", call="mc", system="ctm", n=4096, n_in=0, f64=False,
             steps=100, m=1 << 14),
        # a chain that is no multiple of a wavefront, its input drawn per sample
        dict(name="mc_rd_1100_f64", call="mc", system="rd", n=1100, n_in=1, f64=True, steps=100,
             m=20000),
        # the heat diffusion case study at its size, 8 of its 1000 steps
        dict(name="heat_1000_f64", call="heat", nx=1000, ny=1000, nz=1000, f64=True, steps=8),
        # a ragged grid of ordinary size
        dict(name="heat_200_f32", call="heat", nx=200, ny=180, nz=150, f64=False, steps=40),
        # the query mix (4 to 512 cells, 10 to 1000 steps), planning and upload included
        dict(name="batch_10000_f64", call="batch", nq=10000),
    ]


def _log_int(rng, lo, hi):
    return min(hi, int(math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))))


def draw(rng):
    call = rng.choice(["embed", "embed", "embed", "tube", "growth", "mc", "mc", "heat", "heat",
                       "batch"])
    if call == "batch":
        return dict(call="batch", nq=_log_int(rng, 64, 20000))
    f64 = rng.random() < 0.6
    if call == "heat":
        nx, ny, nz = (_log_int(rng, 24, 640) for _ in range(3))
        steps = _log_int(rng, 4, 60)
        most = MOST_FLOPS / (OPS["heat"] * 2.0 * nx * ny * nz)
        return dict(call="heat", nx=nx, ny=ny, nz=nz, f64=f64, steps=max(2, min(steps, int(most))))
    system = rng.choice(["ctm", "rd", "lin3"])
    steps = _log_int(rng, 20, 400)
    if call == "mc":
        n = _log_int(rng, 16, 2048 if f64 else 4096)
        m = _log_int(rng, 500, 30000)
        most = MOST_FLOPS / 2 / (OPS[system] * float(n) * m)
        c = dict(call="mc", system=system, n=n, f64=f64, m=m, steps=max(10, min(steps, int(most))))
    else:
        n = _log_int(rng, 16, (1 << 25) if call == "embed" else (1 << 22))
        most = MOST_FLOPS / (OPS[system] * 2.0 * n)
        c = dict(call=call, system=system, n=n, f64=f64, steps=max(20, min(steps, int(most))))
        if call == "tube":
            c["every"] = rng.choice([5, 10, 20])
            c["steps"] = c["every"] * max(1, min(c["steps"] // c["every"], 10))
    c["n_in"] = 0 if system == "ctm" else rng.choice([0, 1, c["n"]])
    return c


# ------------------------------------------------------------------ inputs

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _uniform(g, n):
    return torch.rand(n, generator=g, device=DEV, dtype=torch.float64)


def _chain_box(system, n, f64, seed):
    """The workloads' box recipe of a chain: (lo, hi)."""
    g = _gen(seed)
    u0, u1 = _uniform(g, n), _uniform(g, n)
    if system == "ctm":
        lo = 12.0 + 12.0 * u0
        hi = lo + 2.0 * u1
    else:
        s = torch.sin(torch.arange(1, n + 1, device=DEV, dtype=torch.float64)
                      * (math.pi / (n + 1)))
        s = s * (0.9 + 0.2 * u0)
        lo, hi = s - 0.01 * u1, s + 0.01 * u1
    dt = torch.float64 if f64 else torch.float32
    return lo.to(dt), hi.to(dt)


def _chain_inputs(n_in, f64, seed):
    if n_in == 0:
        return None, None
    dt = torch.float64 if f64 else torch.float32
    if n_in == 1:
        return (torch.full((1,), U_LO, device=DEV, dtype=dt),
                torch.full((1,), U_HI, device=DEV, dtype=dt))
    g = _gen(seed + 7919)
    mid = 0.1 * (_uniform(g, n_in) - 0.5)
    w = 0.05 * _uniform(g, n_in)
    return (mid - w).to(dt), (mid + w).to(dt)


def _heat_box(c, seed):
    """Heated corner block [1 - 0.1 U, 1 + 0.1 U'], elsewhere [0, 0.01 U']."""
    g = _gen(seed)
    nx, ny, nz = c["nx"], c["ny"], c["nz"]
    dt = torch.float64 if c["f64"] else torch.float32
    hi = torch.rand((nz, ny, nx), generator=g, device=DEV, dtype=dt)
    lo = torch.zeros_like(hi)
    hot = (slice(0, (nz + 1) // 2), slice(0, (ny + 1) // 2), slice(0, (nx + 1) // 2))
    v = hi[hot].clone()
    hi.mul_(0.01)
    hi[hot] = 1.0 + 0.1 * v
    lo[hot] = 1.0 - 0.1 * torch.rand(v.shape, generator=g, device=DEV, dtype=dt)
    return lo.reshape(-1), hi.reshape(-1)


def _heat_prm(c):
    # the case study's unit cube: spacing 1 / 1000 at every grid size, so that
    # alpha / dx^2 dt is the stated run's
    return (float(c["nx"]), float(c["ny"]), float(c["nz"]), HEAT_ALPHA, 1.0e-3)


def _queries(nq):
    """Kind, n and steps of the query mix, log-uniform like the served stream
    (the mix belongs to the case; the boxes come from the seed)."""
    g = torch.Generator()
    g.manual_seed(nq)
    u = torch.rand((nq, 3), generator=g, dtype=torch.float64).tolist()
    out = []
    for a, b, d in u:
        n = min(512, int(math.exp(b * math.log(513 / 4)) * 4))
        steps = min(1000, int(math.exp(d * math.log(1001 / 10)) * 10))
        out.append(("ctm" if a < 0.5 else "rd", n, steps))
    return out


def _query_boxes(qs, seed):
    """All queries' boxes one after another: (starts, lo, hi)."""
    starts, total = [], 0
    for _, n, _ in qs:
        starts.append(total)
        total += n
    g = _gen(seed + 1)
    u0, u1 = _uniform(g, total), _uniform(g, total)
    ns = torch.tensor([n for _, n, _ in qs])
    kind = torch.tensor([k == "ctm" for k, _, _ in qs])
    first = torch.repeat_interleave(torch.tensor(starts), ns).to(DEV)
    size = torch.repeat_interleave(ns, ns).to(DEV)
    ctm = torch.repeat_interleave(kind, ns).to(DEV)
    cell = torch.arange(total, device=DEV) - first
    s = torch.sin(math.pi * (cell + 1).double() / (size + 1).double()) * (0.9 + 0.2 * u0)
    lo = torch.where(ctm, 12.0 + 12.0 * u0, s - 0.01 * u1)
    hi = torch.where(ctm, 12.0 + 12.0 * u0 + 2.0 * u1, s + 0.01 * u1)
    return starts, lo, hi


def prepare(case, seed):
    rc = R.Reach(0)
    st = dict(call=case["call"], rc=rc)
    if case["call"] == "batch":
        qs = _queries(case["nq"])
        starts, lo, hi = _query_boxes(qs, seed)
        pl, ph = _chain_inputs(1, True, seed)
        r_lo, r_hi = torch.empty_like(lo), torch.empty_like(hi)
        arr = []
        for (kind, n, steps), o in zip(qs, starts):
            ad = [t.data_ptr() + 8 * o for t in (lo, hi, r_lo, r_hi)]
            arr.append(R.make_query(KIND[kind], n, PRM[kind], R.REACH_F64, *ad, DT[kind], steps,
                                    p_lo=pl if kind == "rd" else None,
                                    p_hi=ph if kind == "rd" else None,
                                    n_in=1 if kind == "rd" else 0))
        nb = R.reach_batch_workspace_bytes(len(qs))
        st.update(arr=R.query_array(arr), ws=torch.empty(nb, dtype=torch.uint8, device=DEV), nb=nb,
                  keep=(lo, hi, pl, ph), r_lo=r_lo, r_hi=r_hi)
        return st
    if case["call"] == "heat":
        lo, hi = _heat_box(case, seed)
        pl = ph = None
        st.update(kind=R.REACH_HEAT3D, prm=_heat_prm(case), dt=DT["heat"])
    else:
        lo, hi = _chain_box(case["system"], case["n"], case["f64"], seed)
        pl, ph = _chain_inputs(case["n_in"], case["f64"], seed)
        st.update(kind=KIND[case["system"]], prm=PRM[case["system"]], dt=DT[case["system"]])
    st.update(lo=lo, hi=hi, pl=pl, ph=ph, steps=case["steps"])
    if case["call"] == "mc":
        st.update(m=case["m"], seed=int(seed) & 0x7FFFFFFF)
    if case["call"] == "tube":
        slots = case["steps"] // case["every"]
        st["every"] = case["every"]
        st["sys"] = R.make_system(st["kind"], lo.numel(), st["prm"], case["n_in"])
        st["dtc"] = R.dtype_code(lo.dtype)
        st["nb"] = R.reach_workspace_bytes(rc.ctx, st["sys"], st["dtc"], 0)
        st["ws"] = torch.empty(max(1, st["nb"]), dtype=torch.uint8, device=DEV)
        st["r_lo"] = torch.empty((slots, lo.numel()), dtype=lo.dtype, device=DEV)
        st["r_hi"] = torch.empty_like(st["r_lo"])
    else:
        st["r_lo"], st["r_hi"] = torch.empty_like(lo), torch.empty_like(hi)
    return st


def run(s):
    rc, call = s["rc"], s["call"]
    if call == "batch":
        R.reach_embed_rk4_batch(rc.ctx, s["arr"], s["ws"], s["nb"])
    elif call == "mc":
        rc.montecarlo(s["kind"], s["prm"], s["lo"], s["hi"], s["dt"], s["steps"], s["m"],
                      s["seed"], p_lo=s["pl"], p_hi=s["ph"], r_min=s["r_lo"], r_max=s["r_hi"])
    elif call == "growth":
        rc.growth_bound(s["kind"], s["prm"], s["lo"], s["hi"], s["dt"], s["steps"], p_lo=s["pl"],
                        p_hi=s["ph"], r_lo=s["r_lo"], r_hi=s["r_hi"])
    elif call == "tube":
        R.reach_embed_rk4_tube(rc.ctx, s["sys"], s["dtc"], s["lo"], s["hi"], s["pl"], s["ph"], 0.0,
                               s["dt"], s["steps"], s["every"], s["r_lo"], s["r_hi"], s["ws"],
                               s["nb"])
    else:
        rc.embed(s["kind"], s["prm"], s["lo"], s["hi"], s["dt"], s["steps"], p_lo=s["pl"],
                 p_hi=s["ph"], r_lo=s["r_lo"], r_hi=s["r_hi"])
    return {"lo": s["r_lo"], "hi": s["r_hi"]}


# -------------------------------------------------------------------- work

def work(case):
    if case["call"] == "batch":
        # the mix's mean sizes: n and steps are independent and log-uniform
        n = (513 - 4) / math.log(513 / 4)
        steps = (1001 - 10) / math.log(1001 / 10)
        ops = 0.5 * (OPS["ctm"] + OPS["rd"])
        return {"bytes": 32.0 * n * case["nq"], "flops": 2.0 * ops * n * steps * case["nq"]}
    size = 8 if case["f64"] else 4
    if case["call"] == "heat":
        n = float(case["nx"]) * case["ny"] * case["nz"]
        return {"bytes": 4.0 * n * size, "flops": 2.0 * OPS["heat"] * n * case["steps"]}
    n, ops = float(case["n"]), OPS[case["system"]]
    if case["call"] == "mc":
        return {"bytes": (4.0 * n + 2.0 * case["n_in"]) * size,
                "flops": ops * n * case["steps"] * case["m"]}
    out = case["steps"] // case["every"] if case["call"] == "tube" else 1
    return {"bytes": (2.0 * n + 2.0 * n * out + 2.0 * case["n_in"]) * size,
            "flops": 2.0 * ops * n * case["steps"]}


# ------------------------------------------------------------------- exact

def _shift(y, left_value, right_value):
    """(y_{i-1}, y_{i+1}) along the last axis with the given values outside."""
    left = torch.full_like(y[..., :1], left_value)
    right = torch.full_like(y[..., :1], right_value)
    return torch.cat((left, y[..., :-1]), -1), torch.cat((y[..., 1:], right), -1)


def _f_ctm(y):
    v, w, c, q = CTM_PRM
    flux = torch.clamp(torch.minimum(v * y, _shift(y, 0.0, -math.inf)[1].neg_().add_(c).mul_(w)),
                       max=q)
    return _shift(flux, 0.0, 0.0)[0].sub_(flux)


def _f_rd(y, u):
    left, right = _shift(y, 0.0, 0.0)
    return left.add_(right).sub_(y, alpha=2.0).div_(RD_PRM[0] ** 2).sub_(y * y * y).add_(u)


def _d_lin3(x, xh, p, ph):
    aL, aD, aR, b = LIN3_PRM
    src = [xh if k < 0 else x for k in (aL, aR)]
    left, right = _shift(src[0], 0.0, 0.0)[0], _shift(src[1], 0.0, 0.0)[1]
    return aD * x + aL * left + aR * right + b * (ph if b < 0 else p)


def _rk4(f, z, dt, steps, seen=None):
    """Classical RK4 on a tuple of tensors; `seen` is called after each step."""
    for k in range(steps):
        k1 = f(z)
        acc = k1
        k2 = f(tuple(a + dt / 2 * b for a, b in zip(z, k1)))
        acc = tuple(a.add_(b, alpha=2.0) for a, b in zip(acc, k2))
        k3 = f(tuple(a + dt / 2 * b for a, b in zip(z, k2)))
        acc = tuple(a.add_(b, alpha=2.0) for a, b in zip(acc, k3))
        k4 = f(tuple(a + dt * b for a, b in zip(z, k3)))
        z = tuple(a + (c.add_(b)).mul_(dt / 6) for a, b, c in zip(z, k4, acc))
        if seen:
            seen(k + 1, z)
    return z


def _exact_chain(case, seed):
    system, n = case["system"], case["n"]
    lo, hi = (t.double() for t in _chain_box(system, n, case["f64"], seed))
    pl, ph = _chain_inputs(case["n_in"], case["f64"], seed)
    pl, ph = (0.0, 0.0) if pl is None else (pl.double(), ph.double())
    dt = DT[system]
    if case["call"] == "growth":
        c, r = (lo + hi) / 2, (hi - lo) / 2
        pc, pr = (pl + ph) / 2, (ph - pl) / 2
        sub, diag, sup, b = {
            "ctm": (CTM_PRM[0], 0.0, CTM_PRM[1], 0.0),
            "rd": (1 / RD_PRM[0] ** 2, -2 / RD_PRM[0] ** 2, 1 / RD_PRM[0] ** 2, 1.0),
            "lin3": (abs(LIN3_PRM[0]), LIN3_PRM[1], abs(LIN3_PRM[2]), abs(LIN3_PRM[3])),
        }[system]

        def f(z):
            x, y = z
            left, right = _shift(y, 0.0, 0.0)
            dx = (_f_ctm(x) if system == "ctm" else _f_rd(x, pc) if system == "rd"
                  else _d_lin3(x, x, pc, pc))
            return dx, diag * y + sub * left + sup * right + b * pr

        c, r = _rk4(f, (c, r), dt, case["steps"])
        return {"lo": c - r, "hi": c + r}

    def f(z):
        x, xh = z
        if system == "ctm":
            return _f_ctm(x), _f_ctm(xh)
        if system == "rd":
            return _f_rd(x, pl), _f_rd(xh, ph)
        return _d_lin3(x, xh, pl, ph), _d_lin3(xh, x, ph, pl)

    tube = []

    def seen(k, z):
        if case["call"] == "tube" and k % case["every"] == 0:
            tube.append(z)

    z = _rk4(f, (lo, hi), dt, case["steps"], seen)
    if case["call"] == "tube":
        return {"lo": torch.stack([t[0] for t in tube]), "hi": torch.stack([t[1] for t in tube])}
    return {"lo": z[0], "hi": z[1]}


def _exact_heat(case, seed):
    lo, hi = _heat_box(case, seed)
    a = HEAT_ALPHA / 1.0e-3 ** 2
    shape = (case["nz"], case["ny"], case["nx"])

    def f(z):
        (u,) = z
        out = torch.zeros_like(u)
        for axis in range(3):
            m = u.shape[axis]
            d = u.narrow(axis, 1, m - 1) - u.narrow(axis, 0, m - 1)
            out.narrow(axis, 0, m - 1).add_(d)
            out.narrow(axis, 1, m - 1).sub_(d)
            del d
        out[:, :, -1] -= u[:, :, -1]       # the open face: temperature 0 outside
        return (out.mul_(a),)

    res = []
    for box in (lo, hi):
        res.append(_rk4(f, (box.double().reshape(shape),), DT["heat"], case["steps"])[0].reshape(-1))
    return {"lo": res[0], "hi": res[1]}


def _mulhi64(a, b):
    """High 64 bits of the unsigned product of an int64 tensor and a constant."""
    mask = 0xFFFFFFFF
    a0, a1 = a & mask, (a >> 32) & mask
    b0, b1 = b & mask, (b >> 32) & mask

    def hi32(x):
        return (x >> 32) & mask

    low = a0 * b0
    m1 = a1 * b0
    m2 = a0 * b1
    mid = hi32(low) + (m1 & mask) + (m2 & mask)
    return a1 * b1 + hi32(m1) + hi32(m2) + hi32(mid)


def _signed(v):
    v &= (1 << 64) - 1
    return v - (1 << 64) if v >> 63 else v


def _draws(seed, samples, coords, f64):
    """U(s, j) of the Monte Carlo sampling (Philox4x64-10 at key (seed, 0),
    counter (j / 4, s, 2, 0), word j mod 4), as a [samples, coords] tensor."""
    m0, m1 = 0xD2E7470EE14C6C93, 0xCA5A826395121157
    w0, w1 = 0x9E3779B97F4A7C15, 0xBB67AE8584CAA73B
    b_lo, b_hi = coords[0] // 4, coords[1] // 4
    c0 = torch.arange(b_lo, b_hi + 1, device=DEV).repeat(len(samples), 1)
    c1 = torch.tensor(samples, device=DEV)[:, None].expand_as(c0)
    c2, c3 = torch.full_like(c0, 2), torch.zeros_like(c0)
    k0, k1 = seed, 0
    for _ in range(10):
        h0, l0 = _mulhi64(c0, m0), c0 * _signed(m0)
        h1, l1 = _mulhi64(c2, m1), c2 * _signed(m1)
        c0, c1, c2, c3 = h1 ^ c1 ^ _signed(k0), l1, h0 ^ c3 ^ _signed(k1), l0
        k0, k1 = k0 + w0, k1 + w1
    r = torch.stack((c0, c1, c2, c3), -1).reshape(len(samples), -1)
    r = r[:, coords[0] - 4 * b_lo:coords[1] + 1 - 4 * b_lo]
    if f64:
        return ((r >> 11) & ((1 << 53) - 1)).double() * 2.0 ** -53
    return ((r >> 40) & ((1 << 24) - 1)).double() * 2.0 ** -24


def _exact_mc(case, seed):
    system, n, m = case["system"], case["n"], case["m"]
    lo, hi = (t.double() for t in _chain_box(system, n, case["f64"], seed))
    pl, ph = _chain_inputs(case["n_in"], case["f64"], seed)
    mn, mx = torch.full_like(lo, math.inf), torch.full_like(lo, -math.inf)
    chunk = max(1, (1 << 25) // n)
    for s in range(0, m, chunk):
        ids = list(range(s, min(m, s + chunk)))
        key = int(seed) & 0x7FFFFFFF
        x = lo + _draws(key, ids, (0, n - 1), case["f64"]) * (hi - lo)
        u = 0.0
        if case["n_in"]:
            u = pl.double() + _draws(key, ids, (n, n + case["n_in"] - 1), case["f64"]) \
                * (ph.double() - pl.double())

        def f(z):
            (y,) = z
            return (_f_ctm(y) if system == "ctm" else _f_rd(y, u) if system == "rd"
                    else _d_lin3(y, y, u, u),)

        (x,) = _rk4(f, (x,), DT[system], case["steps"])
        mn, mx = torch.minimum(mn, x.amin(0)), torch.maximum(mx, x.amax(0))
    return {"lo": mn, "hi": mx}


def _exact_batch(case, seed):
    qs = _queries(case["nq"])
    starts, lo, hi = _query_boxes(qs, seed)
    r_lo, r_hi = torch.empty_like(lo), torch.empty_like(hi)
    v, w, c, q = CTM_PRM
    # queries of one kind, sorted by steps, as rows of a padded matrix; rows
    # leave as their steps are done
    for kind in ("ctm", "rd"):
        rows = sorted((k for k in range(len(qs)) if qs[k][0] == kind), key=lambda k: -qs[k][2])
        if not rows:
            continue
        ns = torch.tensor([qs[k][1] for k in rows], device=DEV)
        off = torch.tensor([starts[k] for k in rows], device=DEV)
        width = int(ns.max())
        cell = torch.arange(width, device=DEV)
        ok = cell[None, :] < ns[:, None]
        at = torch.where(ok, off[:, None] + cell, 0)
        left = [qs[k][2] for k in rows]
        for src, dst, u in ((lo, r_lo, U_LO), (hi, r_hi, U_HI)):
            y, live, done = torch.where(ok, src[at], 0.0), len(rows), 0
            last = (cell[None, :] == ns[:, None] - 1)

            def f(z):
                x = z[0]
                o, e = ok[:live], last[:live]
                if kind == "ctm":
                    sup = w * (c - _shift(x, 0.0, 0.0)[1])
                    flux = torch.clamp(torch.where(e, v * x, torch.minimum(v * x, sup)), max=q)
                    k = _shift(flux, 0.0, 0.0)[0] - flux
                else:
                    k = _f_rd(x, u)
                return (torch.where(o, k, 0.0),)

            while live:
                step = left[live - 1] - done
                (y,) = _rk4(f, (y,), DT[kind], step)
                done += step
                gone = live
                while live and left[live - 1] == done:
                    live -= 1
                o = ok[live:gone]
                dst[at[live:gone][o]] = y[live:gone][o]
                y = y[:live]
    return {"lo": r_lo, "hi": r_hi}


def exact(case, seed):
    if case["call"] == "batch":
        return _exact_batch(case, seed)
    if case["call"] == "heat":
        return _exact_heat(case, seed)
    if case["call"] == "mc":
        return _exact_mc(case, seed)
    return _exact_chain(case, seed)
