"""The work that a user of this package has it do, as cases that can be timed
and whose results can be compared: Rayleigh-Taylor runs, runs watched step by
step, the paper's three kernels called one by one, restarts from populations,
checkpointed gradients and reverse sweeps over kept snapshots.

Every case goes through the public binding (``lbm.Lattice``,
``autograd.rt_temperature``, ``lbm.conservation_noalloc``).  Sizes are those of
the package's own configurations and tests: from the smoke run's 40 x 32 sites
to the 2048 x 4096 lattice, odd and ragged ones among them.

Kinds of cases (``kind``):
  rt       a whole run: init_rt(P), step(n), macros()
  watch    set_state, then n times: step(1), conservation(); macros()
  kernels  set_pops, then n times: propagate(), bc(), collide(); get_pops()
  restart  set_pops, step(n), get_pops(), conservation_noalloc()
  rollout  autograd: rt_temperature forward and backward under a checkpoint
           schedule
  reverse  a reverse sweep by hand over kept snapshots: init_rt, n times
           get_state and step(1); loss_temperature; n times adjoint_step;
           adjoint_init_rt, get_lambda
"""
from __future__ import annotations

import math

import torch
from torch.utils.checkpoint import checkpoint as _recompute

from paper_1703_04594_amd import lbm
from paper_1703_04594_amd.autograd import RolloutConfig, rt_temperature

DEV = "cuda:0"
G_Y, T_BOT, T_TOP = -1e-5, 4.0 / 3.0, 2.0 / 3.0


def _case(name, kind, lx, ly, n, **kw):
    c = {"kind": kind, "lx": lx, "ly": ly, "n": n, "precision": "fp64", "ybc": "walls", "xmode": "wrap",
         "layout": "columns", "step": "fused", "adjoint": "fp64", "schedule": "sqrt", "slots": 0, "tau": 0.7}
    c.update(kw)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # a first trial on a tiny lattice: launches and latency are all there is
        _case("rt 40x32 fp64 x8", "rt", 40, 32, 8),
        # the plain Rayleigh-Taylor configuration, 50 steps
        _case("rt 256x128 fp64 x50", "rt", 256, 128, 50),
        # the forward run of a gradient study: FP32 deviations, long enough to be stepped in one call
        _case("rt 512x512 fp32 x100", "rt", 512, 512, 100, precision="fp32"),
        # the headline lattice in FP64 and in FP32
        _case("rt 2048x4096 fp64 x20", "rt", 2048, 4096, 20),
        _case("rt 2048x4096 fp32 x20", "rt", 2048, 4096, 20, precision="fp32"),
        # a ragged box without walls, x halos copied instead of wrapped, structure-of-arrays storage
        _case("rt 301x1030 fp64 halo x13", "rt", 301, 1030, 13, ybc="periodic", xmode="halo", layout="planes"),
        # a production run whose lattice totals are watched after every step
        _case("watch 1000x1501 fp32 x6", "watch", 1000, 1501, 6, precision="fp32"),
        # the paper's order of kernels, driven one by one (half its 2160 x 8192 lattice each way)
        _case("kernels 1080x4096 fp64 x3", "kernels", 1080, 4096, 3, step="split"),
        # a run taken up again from populations that another program holds
        _case("restart 1024x2048 fp64 x5", "restart", 1024, 2048, 5),
        # the gradient configuration's lattice: FP32 states, FP64 adjoint, sqrt(T) checkpointing
        _case("rollout 512x512 sqrt x36", "rollout", 512, 512, 36, precision="fp32"),
        # the gradient at scale: FP32 states and adjoint, binomial checkpointing in few slots
        _case("rollout 1024x2048 binom x20", "rollout", 1024, 2048, 20, precision="fp32", adjoint="fp32",
              schedule="binomial", slots=6),
        # a reverse sweep written out by hand in FP64 on a ragged lattice
        _case("reverse 211x333 fp64 x10", "reverse", 211, 333, 10),
    ]


# most site updates of a drawn case: well under those of the largest listed one, reverse steps counted threefold
_MOST_UPDATES = 1.2e8


def draw(rng):
    """One more case: any kind, both extents from 24 to 2048 x 4096 sites
    (evenly over their logarithm, so mostly odd), 1 to 100 steps."""
    kind = rng.choice(["rt", "rt", "rt", "watch", "kernels", "restart", "rollout", "reverse"])
    grad = kind in ("rollout", "reverse")
    lx = int(round(math.exp(rng.uniform(math.log(24), math.log(1024 if grad else 2048)))))
    ly = int(round(math.exp(rng.uniform(math.log(24), math.log(1024 if grad else 4096)))))
    most = {"rt": 100, "restart": 100, "watch": 20, "kernels": 20, "rollout": 40, "reverse": 16}[kind]
    n = int(round(math.exp(rng.uniform(0.0, math.log(most)))))
    n = max(1, min(n, int(_MOST_UPDATES / (lx * ly * (4 if grad else 1)))))
    return _case(
        None, kind, lx, ly, n,
        precision=rng.choice(["fp64", "fp32"] if grad else ["fp64", "fp64", "fp32", "fp32", "fp32_f32sums"]),
        ybc="walls" if grad else rng.choice(["walls", "walls", "periodic"]),
        xmode="wrap" if grad else rng.choice(["wrap", "wrap", "wrap", "halo"]),
        layout="columns" if grad else rng.choice(["columns", "columns", "columns", "planes"]),
        step="split" if kind == "kernels" else rng.choice(["fused", "fused", "fused", "split"]),
        adjoint=rng.choice(["fp64", "fp32"]),
        schedule=rng.choice(["sqrt", "binomial"]), slots=rng.randint(2, 6),
        tau=round(rng.uniform(0.6, 1.1), 3))


# ---------------------------------------------------------------------------
# Inputs, from the seed alone (shared by prepare and exact)
# ---------------------------------------------------------------------------
def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(1000003 * int(seed) + 17)


def _interface(case, g):
    """The interface displacement: one uniform draw per column, up to one
    lattice unit either way (so that the flow it starts stands well above the
    rounding of FP32 states)."""
    eta = torch.rand((case["lx"], 1), generator=g, device=DEV, dtype=torch.float64) * 2.0 - 1.0
    return eta.expand(case["lx"], case["ly"]).contiguous()


def _populations(case, g):
    """A flowing, slightly out-of-equilibrium gas: the equilibrium of smooth
    random fields, every population off by about a per cent."""
    lx, ly = case["lx"], case["ly"]
    x = torch.arange(lx, device=DEV, dtype=torch.float64)[:, None] * (2.0 * math.pi / lx)
    y = torch.arange(ly, device=DEV, dtype=torch.float64)[None, :] * (2.0 * math.pi / ly)
    ph = torch.rand(8, generator=g, device=DEV, dtype=torch.float64) * (2.0 * math.pi)
    rho = 1.0 + 0.05 * torch.sin(x + ph[0]) * torch.cos(y + ph[1])
    ux = 0.03 * torch.sin(2 * x + ph[2]) * torch.cos(y + ph[3])
    uy = 0.03 * torch.sin(x + ph[4]) * torch.cos(2 * y + ph[5])
    T = 1.0 + 0.05 * torch.cos(x + ph[6]) * torch.cos(y + ph[7])
    f = torch.empty((37, lx, ly), device=DEV, dtype=torch.float64)
    eq = _Eq(rho, ux, uy, T)
    for l in range(37):
        f[l] = eq(l) * (1.0 + 0.01 * torch.randn((lx, ly), generator=g, device=DEV, dtype=torch.float64))
    if case["precision"] != "fp64":
        for l in range(37):
            f[l] -= W[l]
        f = f.to(torch.float32)
    return f


def prepare(case, seed):
    g = _gen(seed)
    lx, ly, kind = case["lx"], case["ly"], case["kind"]
    st = {"case": case}
    if kind == "rollout":
        st["P"] = _interface(case, g).requires_grad_()
        st["tau"] = torch.tensor(case["tau"], dtype=torch.float64, device=DEV, requires_grad=True)
        st["gT"] = torch.rand((lx, ly), generator=g, device=DEV, dtype=torch.float64) * 0.2 - 0.1
        return st
    st["lat"] = lbm.Lattice(lx, ly, case["tau"], G_Y, T_BOT, T_TOP, precision=case["precision"], ybc=case["ybc"],
                            xmode=case["xmode"], step=case["step"], layout=case["layout"],
                            adjoint=case["adjoint"] if kind == "reverse" else False, device=DEV)
    if kind in ("rt", "reverse"):
        st["P"] = _interface(case, g)
    else:
        st["f0"] = _populations(case, g)
        if kind == "watch":
            st["lat"].set_pops(st["f0"])
            st["state0"] = st["lat"].get_state()
            del st["f0"]
    if kind == "reverse":
        st["target"] = 0.9 + 0.2 * torch.rand((lx, ly), generator=g, device=DEV, dtype=torch.float64)
    if kind == "restart":
        st["totals"] = torch.empty(4, dtype=torch.float64, device=DEV)
    return st


def run(state):
    case = state["case"]
    n, kind = case["n"], case["kind"]
    if kind == "rollout":
        cfg = RolloutConfig(lx=case["lx"], ly=case["ly"], nsteps=n, g_y=G_Y, t_bottom=T_BOT, t_top=T_TOP,
                            precision=case["precision"], checkpoint=case["schedule"], slots=case["slots"],
                            lambda_precision=case["adjoint"])
        T = rt_temperature(state["P"], state["tau"], cfg)
        dP, dtau = torch.autograd.grad(T, (state["P"], state["tau"]), state["gT"])
        return {"T": T.detach(), "dP": dP, "dtau": dtau}
    lat = state["lat"]
    if kind == "rt":
        lat.init_rt(state["P"])
        lat.step(n)
        return list(lat.macros())
    if kind == "watch":
        lat.set_state(state["state0"])
        totals = []
        for _ in range(n):
            lat.step(1)
            totals.append(lat.conservation())
        return {"fields": list(lat.macros()), "totals": totals}
    if kind == "kernels":
        lat.set_pops(state["f0"])
        for _ in range(n):
            lat.propagate()
            lat.bc()
            lat.collide()
        return lat.get_pops()
    if kind == "restart":
        lat.set_pops(state["f0"])
        lat.step(n)
        f = lat.get_pops()
        return {"f": f, "totals": lbm.conservation_noalloc(f, state["totals"])}
    lat.init_rt(state["P"])
    kept = []
    for _ in range(n):
        kept.append(lat.get_state())
        lat.step(1)
    loss = lat.loss_temperature(state["target"])
    dtau = torch.zeros((), dtype=torch.float64, device=DEV)
    for f_n in reversed(kept):
        lat.adjoint_step(f_n, dtau)
    return {"loss": loss, "dtau": dtau, "dP": lat.adjoint_init_rt(state["P"]), "lambda": lat.get_lambda()}


# FLOP of one site: a step (moments, equilibrium, relaxation), a reverse step,
# and what a run begins and ends with (equilibrium of an initial state, moments)
_FLOP_STEP, _FLOP_REVERSE, _FLOP_ENDS = 850, 1490, 400


def work(case):
    """One pass: every call's inputs read once and its outputs written once
    (n steps of one call read and write the populations once)."""
    sites, n, kind = case["lx"] * case["ly"], case["n"], case["kind"]
    pops = 37 * (8 if case["precision"] == "fp64" else 4)
    lam = 37 * (8 if case["adjoint"] == "fp64" else 4)
    if kind == "rt":
        b, f = 8 + pops + 2 * pops + pops + 32, n * _FLOP_STEP
    elif kind == "watch":
        b, f = 2 * pops + n * (2 * pops + pops) + pops + 32, n * (_FLOP_STEP + 140)
    elif kind == "kernels":
        b, f = 2 * pops + n * (2 * pops + 2 * pops) + 2 * pops, n * _FLOP_STEP
    elif kind == "restart":
        b, f = 2 * pops + 2 * pops + 2 * pops + pops, n * _FLOP_STEP
    else:
        # n forward steps whose states are kept, n reverse steps that read them
        b = 8 + pops + n * 2 * pops + pops + 8 + n * (pops + 2 * lam) + lam + 16
        f = n * (_FLOP_STEP + _FLOP_REVERSE)
        if kind == "reverse":
            b += lam + 37 * 8
    return {"bytes": float(sites * b), "flops": float(sites * (f + _FLOP_ENDS))}


# ---------------------------------------------------------------------------
# The same results in plain torch, 64 bits (arXiv:1703.04594, section 3): pull
# streaming of 37 hops, the walls' mirror rule, BGK relaxation towards the
# 4th-order Hermite equilibrium with gravity as a shift of it.
# ---------------------------------------------------------------------------
CS = 1.19697977039307435897239
_W_SHELL = {0: 0.23315066913235250228650, 1: 0.10730609154221900241246, 2: 0.05766785988879488203006,
            4: 0.01420821615845075026469, 5: 0.00535304900051377523273, 8: 0.00101193759267357547541,
            9: 0.00024530102775771734547, 10: 0.00028341425299419821740}


def _hops():
    e = [(a, b) for a in range(-3, 4) for b in range(-3, 4) if a * a + b * b in _W_SHELL]
    return sorted(e, key=lambda v: (v[0] ** 2 + v[1] ** 2, math.atan2(v[1], v[0]) % (2.0 * math.pi)))


E = _hops()
W = [_W_SHELL[a * a + b * b] for a, b in E]


class _Eq:
    """The equilibrium of given fields, one population at a time."""

    def __init__(self, rho, ux, uy, T):
        self.rho, self.ux, self.uy, self.th = rho, ux, uy, T - 1.0
        self.u2 = ux * ux + uy * uy

    def __call__(self, l):
        a = CS * (E[l][0] * self.ux + E[l][1] * self.uy)
        x2 = CS * CS * (E[l][0] ** 2 + E[l][1] ** 2)
        th, u2 = self.th, self.u2
        h2 = (a * a - u2 + th * (x2 - 2.0)) / 2.0
        h3 = a * (a * a - 3.0 * u2 + 3.0 * th * (x2 - 4.0)) / 6.0
        h4 = (a * a * (a * a - 6.0 * u2 + 6.0 * th * (x2 - 6.0)) + u2 * (3.0 * u2 + 6.0 * th * (4.0 - x2))
              + 3.0 * th * th * (x2 * x2 - 8.0 * x2 + 8.0)) / 24.0
        return W[l] * self.rho * (1.0 + a + h2 + h3 + h4)


def _moments(f):
    rho = f[0].clone()
    jx, jy, en = torch.zeros_like(rho), torch.zeros_like(rho), torch.zeros_like(rho)
    for l in range(1, 37):
        a, b = E[l]
        rho = rho + f[l]
        if a:
            jx = jx + (CS * a) * f[l]
        if b:
            jy = jy + (CS * b) * f[l]
        en = en + (CS * CS * (a * a + b * b)) * f[l]
    return rho, jx, jy, en


def _macros(f):
    rho, jx, jy, en = _moments(f)
    ux, uy = jx / rho, jy / rho
    return rho, ux, uy, (en / rho - ux * ux - uy * uy) / 2.0


def _stream(f, walls):
    ly = f[0].shape[1]
    out = []
    rho = sum(f[1:], f[0]) if walls else None
    for l in range(37):
        ex, ey = E[l]
        p = torch.roll(f[l], shifts=(ex, ey), dims=(0, 1))
        if walls and ey:
            one = torch.ones((), dtype=torch.float64, device=p.device)
            ew = _Eq(one, 0 * one, 0 * one, (T_BOT if ey > 0 else T_TOP) * one)(l)
            r = torch.roll(rho, shifts=ex, dims=0)
            if ey > 0:
                p = torch.cat([ew * r[:, [ey - y - 1 for y in range(ey)]], p[:, ey:]], dim=1)
            else:
                p = torch.cat([p[:, :ly + ey], ew * r[:, [2 * ly - 1 - (y - ey) for y in range(ly + ey, ly)]]], dim=1)
        out.append(p)
    return out


def _step(f, tau, walls):
    f = _stream(f, walls)
    rho, ux, uy, T = _macros(f)
    eq = _Eq(rho, ux, uy + tau * G_Y, T + tau * (1.0 - tau) * (G_Y * G_Y / 2.0))
    return [f[l] + (eq(l) - f[l]) / tau for l in range(37)]


def _rt_start(P):
    ly = P.shape[1]
    y = torch.arange(ly, dtype=torch.float64, device=P.device)[None, :]
    T = 1.0 - torch.tanh((y - (ly - 1) / 2.0 - P) / 2.0) / 3.0
    z = torch.zeros_like(T)
    eq = _Eq((8.0 / 9.0) / T, z, z, T)
    return [eq(l) for l in range(37)]


def _totals(f):
    return torch.stack([m.sum() for m in _moments(f)])


def _gradient(case, P, gT_of):
    """T_N, lambda_0 and the gradients by autograd, a step recomputed at a time."""
    P = P.detach().requires_grad_()
    tau = torch.tensor(case["tau"], dtype=torch.float64, device=P.device, requires_grad=True)
    f0 = torch.stack(_rt_start(P))

    def one(f, tau):
        return torch.stack(_step(list(f.unbind(0)), tau, True))

    f = f0
    for _ in range(case["n"]):
        f = _recompute(one, f, tau, use_reentrant=False)
    T = _macros(list(f.unbind(0)))[3]
    dP, dtau, lam = torch.autograd.grad(T, (P, tau, f0), gT_of(T.detach()))
    return T.detach(), dP, dtau, lam


def exact(case, seed):
    kind, n, tau, walls = case["kind"], case["n"], case["tau"], case["ybc"] == "walls"
    g = _gen(seed)
    shift = 0.0 if case["precision"] == "fp64" else 1.0
    if kind == "rollout":
        P = _interface(case, g)
        gT = torch.rand((case["lx"], case["ly"]), generator=g, device=DEV, dtype=torch.float64) * 0.2 - 0.1
        T, dP, dtau, _ = _gradient(case, P, lambda T: gT)
        return {"T": T, "dP": dP, "dtau": dtau}
    if kind == "reverse":
        P = _interface(case, g)
        target = 0.9 + 0.2 * torch.rand((case["lx"], case["ly"]), generator=g, device=DEV, dtype=torch.float64)
        T, dP, dtau, lam = _gradient(case, P, lambda T: T - target)
        return {"loss": 0.5 * (T - target).square().sum(), "dtau": dtau, "dP": dP, "lambda": lam}
    with torch.no_grad():
        if kind == "rt":
            f = _rt_start(_interface(case, g))
        else:
            f = [p.double() + shift * W[l] for l, p in enumerate(_populations(case, g))]
        totals = []
        for _ in range(n):
            f = _step(f, tau, walls)
            if kind == "watch":
                totals.append(_totals(f))
        if kind == "rt":
            return list(_macros(f))
        if kind == "watch":
            return {"fields": list(_macros(f)), "totals": totals}
        pops = torch.stack([p - shift * W[l] for l, p in enumerate(f)])
        return pops if kind == "kernels" else {"f": pops, "totals": _totals(f)}
