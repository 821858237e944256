"""Workloads that the library's speed is measured on.

Each case is one call, or one tick of calls, that a program using the library
makes: a plain control update, the device-resident closed loop, a batch, a tick
of served requests, and the two MPPI baselines of the paper's comparison.  The
scenes are synthetic and seeded.  Reference paths come from the package's
workload generator; obstacles stand clear of the path, as they do for a planned
path; the start state is in mid-manoeuvre.  Every case runs on a context with
the library's default launch shapes.

`exact` computes the same update in FP64 with plain torch, from the paper's
equations.
"""
import functools
import math

import numpy as np
import torch

from paper_2508_05773_amd import brmppi as B
from paper_2508_05773_amd import workloads as W

ARENA = 3 << 30      # bytes of device memory a program hands to the library (as the benchmark does)
DS = 0.1             # metres between waypoints

# Fields of a case
#   kind    solve (the new nominal sequence), costs (also every sample's cost),
#           rollouts (also every applied sequence), loop (closed loop), batch, served
#   S, T    samples, horizon; n_obs obstacles; e4: every how-many-th obstacle is a
#           super-ellipse (0: none); moving: every how-many-th one moves (0: none)
#   discs   footprint discs, half on the tractor, half on the trailer (1: the rear axle)
#   mode    guided, plain (MPPI without guidance) or penalty (plain with the
#           collision penalty)
#   scene   road (random segments), bay (reverse parking, parked vehicles on both
#           sides), route (long spline route)
#   Ts      step [s]: horizons of up to 4 s, as most of the package's
#   paper   the vehicle of the paper's experiment in place of the package's
#   updates of a closed loop; count, mix: instances of a batch or of a served tick
#           and which spread of sizes they have
# The weights' temperature is proportional to the horizon, as the costs are: a few
# to a few hundred samples carry the average.


def _one(name, kind, S, T, n_obs, **kw):
    c = dict(kind=kind, S=S, T=T, n_obs=n_obs, e4=0, moving=0, discs=1, mode="guided", scene="road", paper=False, Ts=0.05)
    c.update(kw)
    return dict(c, name=name) if name else c


def listed():
    return [
        # one controller on a small problem (the size of the smoke test): latency
        # and launches are all there is
        _one("small_solve", "solve", 512, 20, 2, Ts=0.1),
        # odd sizes, moving and super-elliptic obstacles, every applied sequence
        # and cost fetched: what a program that draws the rollouts asks for
        _one("ragged_rollouts", "rollouts", 3001, 37, 5, e4=2, moving=3),
        # reverse parking, one blocking update per tick of a host program that
        # measures the state itself
        _one("park_update", "solve", 8192, 50, 8, scene="bay"),
        # the same as a device-resident closed loop, as the benchmark runs it:
        # 40 receding-horizon updates in one call
        _one("park_loop", "loop", 8192, 50, 8, scene="bay", updates=40),
        # the paper's experiment: its vehicle, 5000 rollouts of 120 steps, parked
        # vehicles as super-ellipses and a pedestrian that walks; with its two
        # baselines (a 3 s horizon: over 4.8 s of reversing the trailer's
        # instability magnifies the last bits of FP32)
        _one("paper_guided", "solve", 5000, 120, 8, scene="bay", e4=1, moving=8, paper=True, Ts=0.025),
        _one("paper_plain", "solve", 5000, 120, 8, scene="bay", e4=1, moving=8, paper=True, Ts=0.025, mode="plain"),
        _one("paper_penalty", "solve", 5000, 120, 8, scene="bay", e4=1, moving=8, paper=True, Ts=0.025, mode="penalty"),
        # the whole body covered by discs: four discs times eight obstacles
        _one("footprint_update", "solve", 4096, 60, 8, discs=4, e4=2),
        # more samples than one wave per SIMD, an odd count, costs fetched
        _one("wide_update", "costs", 20011, 64, 12, moving=4),
        # 64 uneven instances solved together each tick (1024 to 16384 samples,
        # 20 to 80 steps, up to 16 obstacles)
        dict(name="batch_64", kind="batch", count=64, mix=3),
        # one tick of a served fleet: 48 uneven requests in flight at once (2048
        # to 32768 samples, up to 32 obstacles, some moving), warm starts resident
        dict(name="served_tick", kind="served", count=48, mix=4),
        # the largest single update: 65536 samples, 100 steps, 32 obstacles
        _one("large_update", "costs", 65536, 100, 32, scene="route", Ts=0.04),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    what = rng.choice(("solve", "solve", "solve", "costs", "costs", "rollouts", "loop", "batch", "served", "baseline", "baseline"))
    if what in ("batch", "served"):
        return dict(kind=what, count=_log(rng, 3, 64 if what == "batch" else 48), mix=rng.randint(5, 9999))
    discs = rng.choice((1, 1, 1, 2, 4)) if what != "baseline" else 1
    n_obs = rng.randint(0, 32 // discs)
    T = _log(rng, 10, 150)
    # no more than the largest listed case: 65536 samples x 100 steps x 32 rows
    top = min(65536.0, 65536 * 100 * 34 / (T * (n_obs * discs * (2 if discs > 1 else 1) + 2)))
    S = _log(rng, 64, top)
    if what == "rollouts":
        S = min(S, 6000)
    kw = dict(e4=rng.choice((0, 0, 1, 2, 3)), moving=rng.choice((0, 0, 2, 5)), discs=discs, scene=rng.choice(("road", "bay")), paper=rng.random() < 0.3)
    kw["Ts"] = rng.choice([t for t in (0.025, 0.04, 0.05, 0.1) if t * T <= 4.0])
    if what == "loop":
        S, T = min(S, 12000), min(T, 60)
        kw["updates"] = rng.randint(5, 40)
    if what == "baseline":
        kw["mode"] = rng.choice(("plain", "penalty"))
        what = rng.choice(("solve", "costs"))
    return _one(None, what, S, T, n_obs, **kw)


# --------------------------------------------------------------------------
# scenes
# --------------------------------------------------------------------------
@functools.lru_cache(maxsize=None)
def _fixed_path(scene):
    return (W.path_c5() if scene == "route" else W.path_c2())[0]


def _obstacles(rng, path, n, r_disc, bay, body):
    """n ellipses beside the path, none of whose inflated bodies reaches a point
    of it, nor of the straight lines that run on from its ends for `body` metres;
    in a bay they are vehicle-sized and stand along its edges.  With the heading
    of the path beside each."""
    obs, along = np.zeros((n, 8), np.float32), np.zeros(n)
    xy = path[:, :2].astype(np.float64)
    on = np.arange(1.0, body + 1.0)[:, None]
    xy_body = np.concatenate([xy] + [e + sg * on * [math.cos(t), math.sin(t)] for e, t in ((xy[0], path[0, 2]), (xy[-1], path[-1, 2])) for sg in (-1.0, 1.0)])
    lo = len(path) // 2 if bay else 0
    for i in range(n):
        mx, my = (2.5, 1.0) if bay else (float(rng.uniform(0.3, 1.5)), float(rng.uniform(0.3, 1.5)))
        reach = (my if bay else max(mx, my)) + r_disc
        for attempt in range(60):
            k = int(rng.integers(lo, len(path)))
            th = float(path[k, 2])
            off = float(rng.choice((-1.0, 1.0))) * (reach + float(rng.uniform(1.6, 4.0)) + 0.25 * attempt)
            cx, cy = xy[k, 0] - off * math.sin(th), xy[k, 1] + off * math.cos(th)
            hd = th + float(rng.uniform(-0.15, 0.15)) if bay else float(rng.uniform(-math.pi, math.pi))
            if np.hypot(xy_body[:, 0] - cx, xy_body[:, 1] - cy).min() > reach + 1.5:
                break
        obs[i] = (cx, cy, mx, my, hd, 2.0, 0.0, 0.0)
        along[i] = th
    return obs, along


def _problem(case, seed, controller=0, T=None, instance=0):
    """the inputs of one update: a workloads.Problem (inputs only)"""
    rng = np.random.default_rng([int(seed) & 0xFFFFFFFF, instance, 77])
    scene = case["scene"]
    path = W.random_segment_path(rng)[0] if scene == "road" else _fixed_path(scene)
    paper = case["paper"]
    r_disc = 1.25 if paper else 1.0
    discs = case["discs"]
    kw = dict(r_disc=r_disc, **(W.PAPER_VEHICLE if paper else {}))
    if discs > 1:
        half = discs // 2
        kw.update(disc_tractor=tuple(2.0 * k + 0.5 for k in range(discs - half)), disc_trailer=tuple(2.5 * k + 1.5 for k in range(half)))
    obs, along = _obstacles(rng, path, case["n_obs"], r_disc, scene == "bay", 8.0 if discs > 1 else 0.0)
    if case["e4"]:
        obs[:: case["e4"], 5] = 4.0
    if case["moving"]:
        for i in range(case["moving"] - 1, len(obs), case["moving"]):
            way = along[i] + float(rng.choice((0.0, math.pi)) + rng.uniform(-0.1, 0.1))
            obs[i, 2:4], obs[i, 5] = 0.5, 2.0      # a pedestrian who walks along the path
            obs[i, 6:8] = 1.2 * math.cos(way), 1.2 * math.sin(way)
    T = case["T"]
    k = int(rng.integers(0, 20))
    x0 = np.zeros(8, np.float32)
    x0[:2] = path[k, :2]
    ahead = path[k + 1, :2].astype(np.float64) - path[k, :2]
    way = 1.0 if ahead[0] * math.cos(path[k, 2]) + ahead[1] * math.sin(path[k, 2]) > 0 else -1.0
    x0[2], x0[3] = way * rng.uniform(0.2, 1.2), rng.uniform(-0.2, 0.2)
    x0[4] = path[k, 2] + rng.uniform(-0.05, 0.05)
    x0[5] = x0[4] + rng.uniform(-0.08, 0.08)
    x0[6], x0[7] = rng.uniform(-0.1, 0.1), DS * k
    u_nom = (rng.standard_normal((T, 3)) * [0.2, 0.05, 0.3] + [0.0, 0.0, 1.0]).astype(np.float32)
    flags = {"guided": 0, "plain": B.GUIDANCE_OFF, "penalty": B.GUIDANCE_OFF | B.COLLISION_PENALTY}[case["mode"]]
    return W.Problem(S=case["S"], T=T, x0=x0, u_nom=u_nom, obstacles=obs, path=path, ds=DS, params=W.make_params(case["Ts"], **kw), lam=0.4 * T,
                     seed=int(rng.integers(0, 2**62)), instance=instance, controller=controller, t0=0.0, flags=flags)


def _members(case):
    """the cases of a batch's or a served tick's instances: their sizes belong to
    the case, not to the seed"""
    rng = np.random.default_rng(case["mix"])
    got = []
    for i in range(case["count"]):
        if case["kind"] == "batch":
            S, T, n = int(rng.choice([1024, 2048, 4096, 8192, 16384])), int(rng.integers(20, 81)), int(rng.integers(0, 17))
            moving = 0
        else:
            S, T, n = int(rng.choice([2048, 8192, 32768])), int(rng.choice([30, 50, 100])), int(rng.integers(0, 33))
            moving = 10
        if rng.random() < 0.2:
            S -= int(rng.integers(1, 500))
        got.append(_one(None, "solve", S, T, n, moving=moving, Ts=0.05 if T <= 80 else 0.04))
    return got


def _problems(case, seed):
    if case["kind"] in ("batch", "served"):
        return [_problem(m, seed, controller=i, instance=i + 1) for i, m in enumerate(_members(case))]
    return [_problem(case, seed)]


# --------------------------------------------------------------------------
# one pass
# --------------------------------------------------------------------------
def prepare(case, seed):
    ctx = B.Context(arena_bytes=ARENA, n_streams=2)
    probs = _problems(case, seed)
    for p in probs:
        ctx.set_path(p.controller, p.path, p.ds)
    kind = case["kind"]
    bufs = [B.ProblemBuffers(p, with_nominal=kind != "served") for p in probs]
    if kind == "served":
        for p in probs:
            B.brmppi_set_nominal(ctx.h, p.controller, p.u_nom)
    return dict(kind=kind, ctx=ctx, bufs=bufs, batch=B.BatchBuffers(bufs) if kind == "batch" else None, updates=case.get("updates"))


def run(state):
    h, kind, bufs = state["ctx"].h, state["kind"], state["bufs"]
    if kind == "solve":
        u, _, _ = B.brmppi_solve(h, bufs[0])
        return dict(u=u)
    if kind == "costs":
        r = B.brmppi_solve_ex(h, bufs[0], want_J=True)
        return dict(u=r["U_new"], J=r["J"])
    if kind == "rollouts":
        r = B.brmppi_solve_ex(h, bufs[0], want_J=True, want_useq=True)
        return dict(u=r["U_new"], J=r["J"], useq=r["useq"])
    if kind == "loop":
        x, u = B.brmppi_closed_loop(h, bufs[0], state["updates"])
        # the states are integrated in FP64 from inputs of FP32: FP32 is what they hold
        return dict(x=x.astype(np.float32), u=u)
    if kind == "batch":
        return dict(u=np.concatenate(B.brmppi_solve_batch(h, state["batch"])[0]))
    tickets = [B.brmppi_submit(h, b)[0] for b in bufs]
    return dict(u=np.concatenate([B.brmppi_wait(h, t, b.c.T)[0] for t, b in zip(tickets, bufs)]))


# --------------------------------------------------------------------------
# the work of one pass
# --------------------------------------------------------------------------
def _update_work(c):
    """Bytes: inputs read once and outputs written once (everything between them
    can stay on the chip).  Flops (fma = 2, a transcendental = 1; Philox's
    integer operations not counted): per sample-step 90 for inputs, angles, cost,
    model and 2x2 solve, 6 per normal, 60 for the hitch rows, and per obstacle row
    70 (e = 2), 90 (e = 4) or 150 (a footprint disc); 10 per obstacle row of the
    penalty."""
    S, T = c["S"], c["T"]
    rows = c["n_obs"] * c["discs"]
    guided = c["mode"] == "guided"
    n4 = len(range(0, c["n_obs"], c["e4"])) * c["discs"] if c["e4"] else 0
    step = 90 + 6 * (5 + rows if guided else 3)
    if guided:
        step += 60 + (150 * rows if c["discs"] > 1 else 70 * (rows - n4) + 90 * n4)
    if c["mode"] == "penalty":
        step += 10 * rows
    out = 12 * T + 16 + (4 * S if c["kind"] in ("costs", "rollouts") else 0) + (12 * S * T if c["kind"] == "rollouts" else 0)
    return 32 * c["n_obs"] + 12 * T + 250 + 16 * 200 + out, float(S) * (T * step + 40)


def work(case):
    members = _members(case) if case["kind"] in ("batch", "served") else [case]
    b, f = map(sum, zip(*(_update_work(m) for m in members)))
    n = case.get("updates", 1) if case["kind"] == "loop" else 1
    return dict(bytes=b * n, flops=f * n)


# --------------------------------------------------------------------------
# the same in FP64, from the paper's equations
# --------------------------------------------------------------------------
_M32 = 0xFFFFFFFF


def _normals(seed, instance, S, tau, K, dev):
    """[K][S] standard normals: Philox4x32-10 (key: the seed; counter: sample,
    step, block, instance), 23-bit uniforms, Box-Muller"""
    nb = (K + 3) // 4
    c0 = torch.arange(S, device=dev, dtype=torch.int64).expand(nb, S)
    c1 = torch.full((nb, S), tau, device=dev, dtype=torch.int64)
    c2 = torch.arange(nb, device=dev, dtype=torch.int64)[:, None].expand(nb, S)
    c3 = torch.full((nb, S), instance, device=dev, dtype=torch.int64)
    k0, k1 = seed & _M32, seed >> 32
    for _ in range(10):
        p0, p1 = c0 * 0xD2511F53, c2 * 0xCD9E8D57      # the low 64 bits: both halves are kept
        c0, c1, c2, c3 = ((p1 >> 32) & _M32) ^ c1 ^ k0, p1 & _M32, ((p0 >> 32) & _M32) ^ c3 ^ k1, p0 & _M32
        k0, k1 = (k0 + 0x9E3779B9) & _M32, (k1 + 0xBB67AE85) & _M32
    u = [((r >> 9).double() + 0.5) / 2.0**23 for r in (c0, c1, c2, c3)]
    r0, r1 = (-2.0 * u[0].log()).sqrt(), (-2.0 * u[2].log()).sqrt()
    a0, a1 = 2.0 * math.pi * u[1], 2.0 * math.pi * u[3]
    return torch.stack([r0 * a0.cos(), r0 * a0.sin(), r1 * a1.cos(), r1 * a1.sin()], 1).reshape(4 * nb, S)[:K]


def _wrap(x):
    return x - 2.0 * math.pi * torch.round(x / (2.0 * math.pi))


def _tracking(P, path, ds, px, py, th1, th2, psi):
    f = psi / ds
    i = f.floor().clamp(0, len(path) - 2)
    t = (f - i).clamp(0.0, 1.0)
    A, E = path[i.long()], path[i.long() + 1]
    rx, ry = A[:, 0] + t * (E[:, 0] - A[:, 0]), A[:, 1] + t * (E[:, 1] - A[:, 1])
    r1, r2 = A[:, 2] + t * _wrap(E[:, 2] - A[:, 2]), A[:, 3] + t * _wrap(E[:, 3] - A[:, 3])
    ex, ey = px - rx, py - ry
    ec, el = r1.sin() * ex - r1.cos() * ey, -r1.cos() * ex - r1.sin() * ey
    return P["Qc"] * ec**2 + P["Ql"] * el**2 + P["Qth1"] * _wrap(th1 - r1) ** 2 + P["Qth2"] * _wrap(th2 - r2) ** 2


def _update(p, x0, u_nom, seed, dev):
    """One update: (U [T][3], costs [S], applied sequences [T][3][S])."""
    P, T, S = p.params, p.T, p.S
    Ts, l1, l2, ch = P["Ts"], P["l1"], P["l2"], P["lh"] / P["l1"]
    ds = float(np.float32(p.ds))
    path = torch.tensor(np.asarray(p.path, np.float64), device=dev)
    discs = [(v, 0.0) for v in P["disc_tractor"]] + [(-P["lh"], v) for v in P["disc_trailer"]]
    ob = torch.tensor(np.asarray(p.obstacles, np.float64).reshape(-1, 8), device=dev)
    rows = ob.repeat(len(discs), 1)
    dA = torch.tensor([a for a, _ in discs], dtype=torch.float64, device=dev).repeat_interleave(len(ob))[:, None]
    dB = torch.tensor([b for _, b in discs], dtype=torch.float64, device=dev).repeat_interleave(len(ob))[:, None]
    cx, cy, mx, my, hd, ee, vx, vy = (rows[:, k : k + 1] for k in range(8))
    co, so, is4 = hd.cos(), hd.sin(), ee == 4.0
    scale = [(mx + P["r_disc"]) ** -ee, (my + P["r_disc"]) ** -ee]
    R = len(rows)
    guided, penalty = not p.flags & B.GUIDANCE_OFF, bool(p.flags & B.COLLISION_PENALTY)
    K = 5 + R if guided else 3
    one = torch.ones(S, dtype=torch.float64, device=dev)
    px, py, v, a, th1, th2, dl, psi = (float(x0[k]) * one for k in range(8))
    alpha = torch.full((2 + R, S), P["alpha0"], dtype=torch.float64, device=dev)
    Ma, J, useq = P["W_a"] + P["rho"], 0.0 * one, []

    def frame(x, y):      # into the obstacles' frames
        return [co * x + so * y, -so * x + co * y]

    def collision(t):
        if not penalty:
            return 0.0
        x = px + dA * th1.cos() - dB * th2.cos() - (cx + vx * t)
        y = py + dA * th1.sin() - dB * th2.sin() - (cy + vy * t)
        q = frame(x, y)
        h = sum(s * torch.where(is4, z**4, z**2) for s, z in zip(scale, q)) - 1.0
        return P["w_col"] * (h.clamp(max=0.0) ** 2).sum(0)

    for tau in range(T):
        t = p.t0 + tau * Ts
        e = _normals(seed, p.instance, S, tau, K, dev)
        uj, uw, un = (u_nom[tau, k] + P[n] * e[k] for k, n in enumerate(("sigma_j", "sigma_w", "sigma_nu")))
        s1, c1, sp, cp, tn = th1.sin(), th1.cos(), (th1 - th2).sin(), (th1 - th2).cos(), dl.tan()
        sec2, kd = 1.0 + tn * tn, tn / l1
        Wt = (sp - ch * cp * tn) / l2                 # trailer heading rate per speed, eq. (6)
        w1, w2 = v * kd, v * Wt
        if guided:
            dkd, Wp, Wd = sec2 / l1, (cp + ch * sp * tn) / l2, -ch * cp * sec2 / l2
            # hitch rows (18), first-order expansion
            D, hh, Lf, g0, g1 = w2 - w1, [], [], [], []
            for s in (1.0, -1.0):
                hdot = -P["kappa"] * a - s * D
                hh.append(P["dtheta_max"] - P["kappa"] * v + s * (th1 - th2) + Ts * hdot)
                Lf.append(Ts * ((-P["kappa"] - s * Ts * (Wt - kd)) * a - s * (1.0 - Ts * v * Wp) * D))
                g0.append(-P["kappa"] * Ts * Ts * one)
                g1.append(-s * Ts * Ts * v * (Wd - dkd))
            hh, Lf, g0, g1 = (torch.stack(q) for q in (hh, Lf, g0, g1))
            if R:
                # obstacle rows (16)-(17): the centre's velocity, acceleration and
                # jerk along the drift, and the inputs' way into the first two
                e1, e2 = (c1, s1), (-s1, c1)
                f2 = (c1 * cp + s1 * sp, s1 * cp - c1 * sp)
                n2 = (-f2[1], f2[0])
                ph, w1d = w1 - w2, a * kd
                w2d = a * Wt + v * Wp * ph
                w2dd = 2 * a * Wp * ph - v * Wt * ph**2 + v * Wp * (w1d - w2d)
                Wpd = ch * sp * sec2 / l2
                w2d_dl = a * Wd + v * Wpd * ph + v * Wp * (v * dkd - v * Wd)
                pos, vel, acc, jrk, vdl, aa, adl = ([], [], [], [], [], [], [])
                for k in range(2):
                    pos.append((px, py)[k] + dA * e1[k] - dB * f2[k] - ((cx, cy)[k] + (vx, vy)[k] * t))
                    vel.append(v * e1[k] + dA * w1 * e2[k] - dB * w2 * n2[k] - (vx, vy)[k])
                    acc.append(a * e1[k] + v * w1 * e2[k] + dA * (w1d * e2[k] - w1**2 * e1[k]) - dB * (w2d * n2[k] - w2**2 * f2[k]))
                    jrk.append(-v * w1**2 * e1[k] + (2 * a * w1 + v * w1d) * e2[k] + dA * (-3 * w1 * w1d * e1[k] - w1**3 * e2[k])
                               + dB * (3 * w2 * w2d * f2[k] + (w2**3 - w2dd) * n2[k]))
                    vdl.append(dA * v * dkd * e2[k] - dB * v * Wd * n2[k])
                    aa.append(e1[k] + dA * kd * e2[k] - dB * Wt * n2[k])
                    adl.append(v**2 * dkd * e2[k] + dA * (a * dkd * e2[k] - 2 * w1 * v * dkd * e1[k]) - dB * (w2d_dl * n2[k] - 2 * w2 * v * Wd * f2[k]))
                h, hd1, hd2, hd3, da, d1, d2 = -1.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0
                for k, (y, yd, ydd, yddd, yl, ya, yal) in enumerate(zip(*(frame(*q) for q in (pos, vel, acc, jrk, vdl, aa, adl)))):
                    q = scale[k]
                    f0, f1 = q * torch.where(is4, y**4, y**2), q * torch.where(is4, 4 * y**3, 2 * y)
                    f2_, f3 = q * torch.where(is4, 12 * y**2, 2 * torch.ones_like(y)), q * torch.where(is4, 24 * y, 0 * y)
                    h = h + f0
                    hd1 = hd1 + f1 * yd
                    hd2 = hd2 + f2_ * yd**2 + f1 * ydd
                    hd3 = hd3 + f3 * yd**3 + 3 * f2_ * yd * ydd + f1 * yddd
                    da, d1, d2 = da + f1 * ya, d1 + f1 * yl, d2 + 2 * f2_ * yd * yl + f1 * yal
                hh = torch.cat([hh, h + Ts * hd1 + 0.5 * Ts**2 * hd2])
                Lf = torch.cat([Lf, Ts * (hd1 + Ts * hd2 + 0.5 * Ts**2 * hd3)])
                g0 = torch.cat([g0, 0.5 * Ts**3 * da])
                g1 = torch.cat([g1, Ts * (Ts * d1 + 0.5 * Ts**2 * d2)])
            mag = hh.abs().clamp(min=P["h_eps"])
            hh = torch.where(hh < 0, -mag, mag)
            # eqs. (11)-(12), the auxiliary inputs eliminated
            b = -Lf - alpha * hh
            pa = P["W_a"] * P["sigma_a"] * e[3:] + P["rho"] * (0.5 * (P["alpha_lo"] + P["alpha_hi"]) - alpha)
            c, r = Ma / hh**2, b - hh * pa / Ma
            n00 = P["W_j"] + P["rho"] + (c * g0 * g0).sum(0)
            n11 = P["W_w"] + P["rho"] + (c * g1 * g1).sum(0)
            n01 = (c * g0 * g1).sum(0)
            y0 = P["W_j"] * uj + 0.5 * P["rho"] * (P["j_lo"] + P["j_hi"]) + (c * g0 * r).sum(0)
            y1 = P["W_w"] * uw + 0.5 * P["rho"] * (P["w_lo"] + P["w_hi"]) + (c * g1 * r).sum(0)
            det = n00 * n11 - n01 * n01
            uj, uw = (n11 * y0 - n01 * y1) / det, (n00 * y1 - n01 * y0) / det
            alpha = alpha + (b - g0 * uj - g1 * uw) / hh
        J = J + _tracking(P, path, ds, px, py, th1, th2, psi) + P["R_j"] * uj**2 + P["R_w"] * uw**2 + P["mu"] * (P["nu_bar"] - un) ** 2 + collision(t)
        useq.append(torch.stack([uj, uw, un]))
        px, py, v, a, th1, th2, dl, psi = (px + Ts * v * c1, py + Ts * v * s1, v + Ts * a, a + Ts * uj, th1 + Ts * w1, th2 + Ts * w2, dl + Ts * uw, psi + Ts * un)
    J = J + _tracking(P, path, ds, px, py, th1, th2, psi) + collision(p.t0 + T * Ts)
    J = torch.where(J.isfinite(), J, torch.full_like(J, math.inf))
    w = torch.exp(-(J - J.min()) / float(np.float32(p.lam)))
    w = w / w.sum()
    useq = torch.stack(useq)
    return (torch.where(w > 0, w * useq, torch.zeros_like(useq))).sum(2), J, useq


def _plant(P, x, u):
    """the closed loop's plant: eq. (6) with the inputs held to their bounds"""
    Ts, l1, l2 = P["Ts"], P["l1"], P["l2"]
    px, py, v, a, th1, th2, dl, psi = x
    j, w = min(max(u[0], P["j_lo"]), P["j_hi"]), min(max(u[1], P["w_lo"]), P["w_hi"])
    t = math.tan(dl)
    return [px + Ts * v * math.cos(th1), py + Ts * v * math.sin(th1), v + Ts * a, a + Ts * j, th1 + Ts * v / l1 * t,
            th2 + Ts * v / l2 * (math.sin(th1 - th2) - P["lh"] / l1 * math.cos(th1 - th2) * t), dl + Ts * w, psi + Ts * u[2]]


def exact(case, seed):
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    probs = _problems(case, seed)
    kind = case["kind"]
    if kind == "loop":
        p = probs[0]
        x, un, xs, us = [float(z) for z in p.x0], torch.tensor(p.u_nom.astype(np.float64), device=dev), [], []
        xs.append(x)
        for k in range(case["updates"]):
            U = _update(p, x, un, p.seed + k, dev)[0]
            us.append(U[0].tolist())
            x = _plant(p.params, x, us[-1])
            xs.append(x)
            un = torch.cat([U[1:], U[-1:]])
        return dict(x=np.array(xs), u=np.array(us))
    got = [_update(p, p.x0, torch.tensor(p.u_nom.astype(np.float64), device=dev), p.seed, dev) for p in probs]
    if kind in ("batch", "served"):
        return dict(u=torch.cat([g[0] for g in got]).cpu().numpy())
    U, J, useq = (z.cpu().numpy() for z in got[0])
    if kind == "solve":
        return dict(u=U)
    return dict(u=U, J=J, useq=useq) if kind == "rollouts" else dict(u=U, J=J)
