"""The work that users of this framework have it do, as cases that can be
timed and compared: Adam solves of unit-commitment grids, single gradient
evaluations, screened and batched solves, and the warm-start network.

A case is a dict of plain values; ``prepare`` makes what a program holds
before the call (the built grid, the point and the Adam moments of a solve
under way, the network's weights), ``run`` makes one pass through the public
entry points, ``work`` says what a pass cannot do without, and ``exact``
computes the same outputs in plain 64-bit torch from the definitions.

Sizes: the repository's own grids (14, 617 and 2,000 buses; 4 to 48 periods;
1.4 branches and 0.15 generators per bus; every outage that does not island
the grid) and network (11,124 -> 3 x 512 -> 29,412, batches of up to 64), and
odd sizes between them.
"""
import functools
import math

import numpy as np
import torch

from paper_2310_06650_amd import qg, synth

DEV = "cuda"
HORIZON = 5000                      # steps of the whole solve a pass is a part of
ALPHA = (1e-3, 1e-5)                # step sizes at its two ends
EPS = (1e-1, 1e-4)                  # soft-function widths
RAMP = (0.1, 1.0)                   # penalty scales (beta and rho)
FLAGS = {"fp64": 0, "fp32": qg.QG_FLAG_CTG_FP32, "bf16": qg.QG_FLAG_CTG_BF16}
FACTOR_BYTES = {"fp64": 8, "fp32": 4, "bf16": 2}


def grid(n_bus, n_branch, n_gen, n_period, n_ctg, grid_seed, tree):
    return dict(n_bus=n_bus, n_branch=n_branch, n_gen=n_gen, n_period=n_period, n_ctg=n_ctg,
                grid_seed=grid_seed, tree=tree)


SMALL = grid(14, 20, 5, 4, 0, 1, "recursive")
MIDDLE = grid(617, 850, 100, 18, 560, 2, "recursive")
LARGE = grid(2000, 2800, 300, 48, 2500, 3, "prufer")


def listed():
    return [
        # a toy grid: latency and launches alone
        dict(name="grid14-solve", kind="solve", steps=100, final=True, factors="fp64", **SMALL),
        # a small grid of ragged sizes, solved to its score
        dict(name="grid131-solve", kind="solve", steps=80, final=True, factors="fp64",
             **grid(131, 183, 20, 7, 0, 31, "prufer")),
        # the benchmark's grid: a stretch of a long solve, the score left for later
        dict(name="grid617-solve", kind="solve", steps=100, final=False, factors="fp64", **MIDDLE),
        # a caller's own loop on it: the gradient, then one Adam step
        dict(name="grid617-eval-adam", kind="eval", adam=True, factors="fp64", **MIDDLE),
        # objective and gradient with FP32 outage factors on a ragged grid
        dict(name="grid1009-eval-fp32", kind="eval", adam=False, factors="fp32",
             **grid(1009, 1413, 151, 31, 0, 37, "prufer")),
        # the largest grid
        dict(name="grid2000-solve", kind="solve", steps=64, final=False, factors="fp64", **LARGE),
        # two refresh cycles of contingency screening on the largest grid
        dict(name="grid2000-screened", kind="screen", steps=50, refresh=25, top=0.05, rand=0.05,
             factors="fp64", **LARGE),
        # independent grids of uneven size in one batched solve
        dict(name="batch12-solve", kind="batch", scenarios=12, steps=64, lo_bus=100, hi_bus=1000,
             lo_period=12, hi_period=48, grid_seed=4000),
        # the warm-start network: a training step, inference in both precisions
        dict(name="net-train-64", kind="net_train", d_in=11124, width=512, depth=3, d_out=29412,
             batch=64),
        dict(name="net-bf16-64", kind="net_bf16", d_in=11124, width=512, depth=3, d_out=29412,
             batch=64),
        # a smaller network on an odd batch in FP32
        dict(name="net-fp32-17", kind="net_fp32", d_in=2703, width=200, depth=2, d_out=7353,
             batch=17),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _drawn_grid(rng):
    n = _log_int(rng, 14, 2000)
    return grid(n, int(round(1.4 * n)), max(2, int(round(0.15 * n))), _log_int(rng, 4, 48), 0,
                rng.randrange(1 << 20), "prufer")


def draw(rng):
    u = rng.random()
    if u < 0.45:
        return dict(kind="solve", steps=rng.randint(16, 64), final=rng.random() < 0.5,
                    factors=rng.choice(("fp64", "fp64", "fp64", "fp32", "bf16")), **_drawn_grid(rng))
    if u < 0.65:
        return dict(kind="eval", adam=rng.random() < 0.5,
                    factors=rng.choice(("fp64", "fp64", "fp64", "fp32", "bf16")), **_drawn_grid(rng))
    if u < 0.73:
        return dict(kind="screen", steps=rng.randint(10, 50), refresh=rng.randint(5, 25),
                    top=rng.uniform(0.02, 0.1), rand=rng.uniform(0.02, 0.1), factors="fp64",
                    **_drawn_grid(rng))
    if u < 0.8:
        lo = rng.randint(20, 100)
        return dict(kind="batch", scenarios=rng.randint(2, 12), steps=rng.randint(16, 64),
                    lo_bus=lo, hi_bus=lo + rng.randint(0, 800), lo_period=rng.randint(4, 12),
                    hi_period=rng.randint(12, 48), grid_seed=rng.randrange(1 << 20))
    return dict(kind=rng.choice(("net_train", "net_bf16", "net_fp32")),
                d_in=_log_int(rng, 60, 11124), width=rng.choice((64, 200, 256, 384, 512)),
                depth=rng.randint(1, 3), d_out=_log_int(rng, 190, 29412),
                batch=rng.choice((1, 5, 17, 32, 48, 64)))


# ------------------------------------------------------------------ inputs

@functools.lru_cache(maxsize=64)
def _grid(n_bus, n_branch, n_gen, n_period, n_ctg, grid_seed, tree):
    """The grid a program works on (the loads of a day are drawn later)."""
    return synth.make_case(seed=grid_seed, n_bus=n_bus, n_branch=n_branch, n_gen=n_gen,
                           n_period=n_period, n_ctg=n_ctg or None, tree=tree, mesh=3.0)


def _grids(case):
    """The grids of a case: one, or the scenarios of a batch."""
    if case["kind"] != "batch":
        return [_grid(*(case[k] for k in ("n_bus", "n_branch", "n_gen", "n_period", "n_ctg",
                                          "grid_seed", "tree")))]
    rng = np.random.default_rng(case["grid_seed"])
    out = []
    for i in range(case["scenarios"]):
        n = int(rng.integers(case["lo_bus"], case["hi_bus"] + 1))
        t = int(rng.integers(case["lo_period"], case["hi_period"] + 1))
        out.append(_grid(n, int(round(1.4 * n)), max(2, int(round(0.15 * n))), t, 0,
                         case["grid_seed"] + 1 + i, "prufer"))
    return out


def _laplacian(g):
    y = g.br_x / (g.br_r ** 2 + g.br_x ** 2)
    Y = np.zeros((g.n_bus, g.n_bus))
    np.add.at(Y, (g.br_from, g.br_from), y)
    np.add.at(Y, (g.br_to, g.br_to), y)
    np.subtract.at(Y, (g.br_from, g.br_to), y)
    np.subtract.at(Y, (g.br_to, g.br_from), y)
    return y, Y


def _day(g, seed):
    """A day's loads on the grid, and a point and Adam moments of a solve
    under way: generators near their share of the load, angles that carry
    the power there, everything else near its place in the box."""
    g = synth.with_loads(g, synth.load_draw(g, seed))
    rng = np.random.default_rng(seed + 1)
    T, N, G = g.n_period, g.n_bus, g.n_gen
    share = g.load_p.sum(axis=1) / g.gen_pmax.sum()
    p = np.clip(share[:, None] * rng.uniform(0.7, 1.3, (T, G)), 0.02, 0.98) * g.gen_pmax
    inj = -g.load_p.copy()
    np.add.at(inj, (slice(None), g.gen_bus), p)
    inj -= inj.mean(axis=1, keepdims=True)
    th = np.zeros((T, N))
    th[:, 1:] = np.linalg.solve(_laplacian(g)[1][1:, 1:], inj[:, 1:].T).T
    q = rng.uniform(0.1, 0.9, (T, G)) * g.gen_qmax
    r = rng.uniform(0.1, 0.9, (T, G)) * g.gen_rmax
    u = rng.uniform(0.8, 0.99, (T, G))
    vm = rng.uniform(0.98, 1.02, (T, N))
    x = np.concatenate([a.reshape(-1) for a in (vm, th, p, q, r, u)])
    size = rng.lognormal(math.log(1e6), 1.0, x.size)  # of the gradients so far
    return g, x, 0.3 * size * rng.normal(size=x.size), size * size


def _begin(case):
    """Steps taken before the pass: a fifth of the horizon (whole refresh
    cycles of a screened solve)."""
    cycle = case.get("refresh", 1)
    return HORIZON // 5 // cycle * cycle


def _schedule(case):
    final = case.get("final", False)
    return dict(n_steps=case["steps"], alpha0=ALPHA[0], alphaf=ALPHA[1], iter0=_begin(case),
                n_total=HORIZON, eps0=EPS[0], epsf=EPS[1], beta0=RAMP[0], betaf=RAMP[1],
                rho0=RAMP[0], rhof=RAMP[1], skip_final=0 if final else 1)


def _net_inputs(case, seed):
    """Weights, moments and a batch, on the GPU, as flat layers
    [W_1, b_1, ..., W_out, b_out]."""
    gen = torch.Generator(device=DEV).manual_seed(seed)
    rnd = lambda *s: torch.randn(*s, generator=gen, device=DEV)  # noqa: E731
    sizes = [case["d_in"]] + [case["width"]] * case["depth"] + [case["d_out"]]
    layers = []
    for a, b in zip(sizes[:-1], sizes[1:]):
        layers += [rnd(a, b) * math.sqrt(2.0 / a), rnd(b) * 0.1]
    size = [3e-6 * torch.exp(0.5 * rnd(*w.shape)) for w in layers]  # of the gradients so far
    return dict(layers=layers, m=[0.3 * s * rnd(*s.shape) for s in size],
                v=[s * s for s in size], x=rnd(case["batch"], case["d_in"]),
                t=rnd(case["batch"], case["d_out"]))


NET_ITER, NET_LR = 500, 1e-3


def prepare(case, seed):
    kind = case["kind"]
    if kind.startswith("net"):
        given = _net_inputs(case, seed)
        net = qg.MLP(case["d_in"], case["width"], case["depth"], case["d_out"],
                     max_batch=case["batch"], device=DEV)
        for i in range(case["depth"] + 1):
            for part, o in enumerate(net.offsets(i)):
                for flat, name in ((net.params, "layers"), (net.m, "m"), (net.v, "v")):
                    a = given[name][2 * i + part].reshape(-1)
                    flat[o:o + a.numel()] = a
        net.iter = NET_ITER
        if kind == "net_bf16":
            net.to_bf16()
        return dict(kind=kind, net=net, x=given["x"], t=given["t"])
    state = dict(kind=kind, case=case, probs=[], x=[], m=[], v=[], start=[])
    for i, g in enumerate(_grids(case)):
        g, x, m, v = _day(g, seed + 1000 * i)
        prob = qg.Problem(g, device=DEV, flags=FLAGS[case.get("factors", "fp64")])
        if kind == "batch" and prob.K > 0:
            prob.set_tile("s4x4")
        if kind == "screen":
            prob.set_screening(case["top"], case["rand"], refresh=case["refresh"], seed=seed)
        state["probs"].append(prob)
        for name, a in (("x", x), ("m", m), ("v", v)):
            state[name].append(prob.new_vector(a))
        state["start"].append([state[name][-1].clone() for name in ("x", "m", "v")])
    if kind == "eval":
        eps, beta, rho, state["lr"] = _params(_begin(case) + 1)
        state["hom"] = dict(eps=eps, beta=beta, rho_scale=rho)
    else:
        state["opts"] = qg.solve_opts(**_schedule(case))
    return state


def run(state):
    kind = state["kind"]
    if kind == "net_train":
        net = state["net"]
        loss = net.train_step(state["x"], state["t"], NET_LR)
        return dict(params=net.params, m=net.m, v=net.v, loss=loss)
    if kind == "net_bf16":
        return state["net"].forward_bf16(state["x"])
    if kind == "net_fp32":
        return state["net"].forward(state["x"])
    probs, xs, ms, vs = (state[k] for k in ("probs", "x", "m", "v"))
    if kind == "eval":
        terms, grad = probs[0].eval_grad(xs[0], **state["hom"])
        if not state["case"]["adam"]:
            return dict(terms=terms, grad=grad)
        probs[0].adam_step(xs[0], ms[0], vs[0], grad, _begin(state["case"]) + 1, state["lr"])
        return dict(terms=terms, grad=grad, x=xs[0], m=ms[0], v=vs[0])
    # a solve from its start, as every solve begins: the vectors set, then the call
    for x, m, v, (x0, m0, v0) in zip(xs, ms, vs, state["start"]):
        x.copy_(x0)
        m.copy_(m0)
        v.copy_(v0)
    out = dict(x=xs, m=ms, v=vs)
    if kind == "batch":
        qg.solve_batch(probs, xs, ms, vs, state["opts"])
        return out
    rep = probs[0].solve(xs[0], ms[0], vs[0], state["opts"])
    if state["case"].get("final"):
        out.update(loss=rep.final_loss, score=rep.final_score, terms=np.array(list(rep.terms)))
    return out


def _grid_work(g, elem, scored):
    """One step: x, m, v read and written, the loads, the branch and
    generator data, the shift factors and the scored outage factors read."""
    T, N, L, G, K = g.n_period, g.n_bus, g.n_branch, g.n_gen, scored
    nbytes = 48 * g.n_x + 16 * T * N + 8 * (8 * L + 24 * G + L * G) + elem * L * K
    return nbytes, 8.0 * T * L * K + 4.0 * T * L * G + 150.0 * T * L


def work(case):
    kind = case["kind"]
    if kind.startswith("net"):
        sizes = [case["d_in"]] + [case["width"]] * case["depth"] + [case["d_out"]]
        n = sum(a * b + b for a, b in zip(sizes[:-1], sizes[1:]))
        macs = sum(a * b for a, b in zip(sizes[:-1], sizes[1:])) * case["batch"]
        io = 4 * case["batch"] * (case["d_in"] + case["d_out"])
        if kind == "net_train":
            return dict(bytes=24 * n + io, flops=2.0 * (3 * macs - case["batch"] * sizes[0] * sizes[1]))
        return dict(bytes=(2 if kind == "net_bf16" else 4) * n + io, flops=2.0 * macs)
    steps = case.get("steps", 1)
    nbytes = flops = 0.0
    for g in _grids(case):
        b, f = _grid_work(g, FACTOR_BYTES[case.get("factors", "fp64")], g.n_ctg)
        if kind == "screen":  # an exact step each cycle, the scored set in the others
            na = math.ceil(case["top"] * g.n_ctg) + math.ceil(case["rand"] * g.n_ctg)
            bs, fs = _grid_work(g, 8, min(na, g.n_ctg))
            full = math.ceil(steps / case["refresh"])
            b, f = full * b + (steps - full) * bs, full * f + (steps - full) * fs
        else:
            b, f = b * steps, f * steps
        nbytes, flops = nbytes + b, flops + f
    return dict(bytes=nbytes, flops=flops)


# ------------------------------------------------------------------ 64-bit values

def _params(i):
    """eps, beta, rho scale and step size at 1-based iteration i."""
    e = math.exp(4.0 * (2.0 * i / HORIZON - 1.0))
    s = e / (0.6 + e)
    curve = lambda a, b: a * 10.0 ** (s * math.log10(b / a))  # noqa: E731
    ramp = RAMP[0] + (RAMP[1] - RAMP[0]) * i / HORIZON
    return curve(*EPS), ramp, ramp, curve(*ALPHA)


class _Exact:
    """The penalised objective of one grid in plain FP64 torch, its gradient
    by autograd."""

    def __init__(self, g):
        self.g = g
        f64 = lambda a: torch.as_tensor(np.asarray(a, dtype=np.float64), device=DEV)  # noqa: E731
        i64 = lambda a: torch.as_tensor(np.asarray(a, dtype=np.int64), device=DEV)  # noqa: E731
        y, Y = _laplacian(g)
        inv = np.zeros_like(Y)
        inv[1:, 1:] = np.linalg.inv(Y[1:, 1:])
        isf = y[:, None] * (inv[g.br_from] - inv[g.br_to])
        fr, to, ctg = g.br_from, g.br_to, g.ctg_list
        ptdf = isf[:, fr[ctg]] - isf[:, to[ctg]]
        lodf = ptdf / (1.0 - ptdf[ctg, np.arange(ctg.size)])
        self.isf, self.lodf = f64(isf), f64(lodf)
        self.fr, self.to, self.ctg, self.gbus = i64(fr), i64(to), i64(ctg), i64(g.gen_bus)
        z2 = g.br_r ** 2 + g.br_x ** 2
        self.bg, self.bb, self.bh = f64(g.br_r / z2), f64(-g.br_x / z2), f64(0.5 * g.br_bch)
        self.pcum = np.concatenate([np.zeros((g.n_gen, 1)), np.cumsum(g.gen_seg_size, axis=1)], axis=1)
        self.lo = f64(self.pcum[:, :-1])
        self.c = {k: f64(getattr(g, k)) for k in (
            "br_smax", "br_smax_ctg", "gen_pmin", "gen_pmax", "gen_qmin", "gen_qmax", "gen_rmax",
            "gen_ru", "gen_rd", "gen_ru_su", "gen_rd_sd", "gen_p0", "gen_u0", "gen_c_on",
            "gen_c_su", "gen_c_sd", "gen_c_r", "gen_seg_cost", "gen_seg_size", "load_p", "load_q",
            "reserve_req", "dt", "v_min", "v_max")}
        T, inf = g.n_period, float("inf")
        n, m = g.n_bus, g.n_gen
        full = lambda k, v: torch.full((k,), v, dtype=torch.float64, device=DEV)  # noqa: E731
        c = self.c
        self.box = [torch.cat([a.repeat(T) for a in s]) for s in (
            (c["v_min"], full(n, -inf), full(m, 0.0), c["gen_qmin"], full(m, 0.0), full(m, 0.0)),
            (c["v_max"], full(n, inf), c["gen_pmax"], c["gen_qmax"], c["gen_rmax"], full(m, 1.0)))]

    def _outages(self, dt, F, q2, eps, beta, cols):
        """[t, k] penalties of the outages of some periods (every outage, or
        positions cols)."""
        out = self.ctg if cols is None else self.ctg[cols]
        lodf = self.lodf if cols is None else self.lodf[:, cols]
        other = torch.ones_like(lodf)
        other[out, torch.arange(out.numel(), device=DEV)] = 0.0
        P = F[:, :, None] + lodf * F[:, out][:, None, :]
        over = torch.relu(torch.sqrt(P * P + q2[:, :, None]) - self.c["br_smax_ctg"][:, None])
        sig = torch.sqrt(over * over + eps * eps)
        return (dt * self.g.c_s * beta)[:, None] * (sig * other).sum(dim=1)

    def __call__(self, x, eps, beta, rho_scale, cols=None, want_z=False):
        """(terms, gradient) and, asked for, the penalties [T, K]."""
        g, c = self.g, self.c
        T, N, G, L, K = g.n_period, g.n_bus, g.n_gen, g.n_branch, self.ctg.numel()
        x = x.detach().clone().requires_grad_(True)
        V, TH, P, Q, R, U = torch.split(x, [T * N, T * N] + [T * G] * 4)
        V, TH, P, Q, R, U = V.view(T, N), TH.view(T, N), P.view(T, G), Q.view(T, G), R.view(T, G), U.view(T, G)
        dt = c["dt"][:, None]
        soft = lambda e: torch.sqrt(torch.relu(e) ** 2 + eps * eps)  # noqa: E731
        # devices
        a = P[:, :, None] - self.lo
        size = c["gen_seg_size"]
        used = torch.where(a > 0.0, torch.where(a <= size, a, size.expand_as(a)), torch.zeros_like(a))
        before = lambda X, x0: torch.cat([x0[None, :], X[:-1]])  # noqa: E731
        du = U - before(U, c["gen_u0"])
        dev = (dt * ((c["gen_seg_cost"] * used).sum(dim=2) + c["gen_c_on"] * U + c["gen_c_r"] * R)
               + c["gen_c_su"] * torch.relu(du) + c["gen_c_sd"] * torch.relu(-du)).sum()
        dP = P - before(P, c["gen_p0"])
        up = dt * (c["gen_ru"] * U + c["gen_ru_su"] * (1.0 - U))
        dn = dt * (c["gen_rd"] * U + c["gen_rd_sd"] * (1.0 - U))
        rows = (P + R - c["gen_pmax"] * U, c["gen_pmin"] * U - P, dP - up, -dP - dn,
                Q - c["gen_qmax"] * U, c["gen_qmin"] * U - Q, R - c["gen_rmax"] * U)
        pen = sum((rho_scale * g.rho * beta * dt * soft(r)).sum() for r in rows)
        rsv = (c["dt"] * g.c_rsv * beta * soft(c["reserve_req"] - R.sum(dim=1))).sum()
        # branches
        vf, vt = V[:, self.fr], V[:, self.to]
        d = TH[:, self.fr] - TH[:, self.to]
        cs, sn, vv, bg, bb, bh = torch.cos(d), torch.sin(d), vf * vt, self.bg, self.bb, self.bh
        pf = bg * vf * vf + vv * (-bg * cs - bb * sn)
        qf = -(bb + bh) * vf * vf + vv * (bb * cs - bg * sn)
        pt = bg * vt * vt + vv * (-bg * cs + bb * sn)
        qt = -(bb + bh) * vt * vt + vv * (bb * cs + bg * sn)
        sf, st = torch.sqrt(pf * pf + qf * qf), torch.sqrt(pt * pt + qt * qt)
        br = (dt * g.c_s * beta * soft(torch.where(sf >= st, sf, st) - c["br_smax"])).sum()
        ang = (dt * g.c_ang * beta * soft(d.abs() - g.ang_max)).sum()
        q2 = torch.where(qf * qf >= qt * qt, qf * qf, qt * qt)
        # balance
        dp = c["load_p"].index_add(1, self.fr, pf).index_add(1, self.to, pt).index_add(1, self.gbus, -P)
        dq = c["load_q"].index_add(1, self.fr, qf).index_add(1, self.to, qt).index_add(1, self.gbus, -Q)
        bal = (dt * beta * (g.c_p * torch.sqrt(dp * dp + eps * eps)
                            + g.c_q * torch.sqrt(dq * dq + eps * eps))).sum()
        # outages, some periods at a time
        inj = (-c["load_p"]).index_add(1, self.gbus, P)
        F = (inj - inj.mean(dim=1, keepdim=True)) @ self.isf.T
        Fd, q2d = F.detach().requires_grad_(True), q2.detach().requires_grad_(True)
        cmax = cmean = 0.0
        zs = []
        some = max(1, (1 << 24) // max(1, L * (K if cols is None else cols.numel())))
        for t in range(0, T if K else 0, some):
            sl = slice(t, t + some)
            z = self._outages(c["dt"][sl], Fd[sl], q2d[sl], eps, beta, cols)
            rest = K - z.shape[1]
            floor = c["dt"][sl] * g.c_s * beta * (L - 1) * eps
            worst = z.max(dim=1).values
            if rest:
                worst = torch.where(worst < floor, floor, worst)
            mean = (z.sum(dim=1) + rest * floor) / K
            (worst + mean).sum().backward()
            cmax, cmean = cmax + worst.detach().sum(), cmean + mean.detach().sum()
            if want_z:
                zs.append(z.detach())
        smooth = dev + bal + br + ang + pen + rsv
        outer = smooth if Fd.grad is None else smooth + (F * Fd.grad).sum() + (q2 * q2d.grad).sum()
        outer.backward()
        value = (c["dt"] * g.load_value * c["load_p"].sum(dim=1)).sum()
        parts = [float(torch.as_tensor(v).detach())
                 for v in (dev, bal, br, ang, pen, rsv, cmax, cmean, value)]
        parts.append(sum(parts[:8]) - parts[8])
        terms = torch.tensor(parts, dtype=torch.float64, device=DEV)
        return (terms, x.grad, torch.cat(zs)) if want_z else (terms, x.grad)

    def adam(self, x, m, v, grad, i, lr):
        m = 0.9 * m + 0.1 * grad
        v = 0.999 * v + 0.001 * grad * grad
        step = lr * (m / (1.0 - 0.9 ** i)) / (torch.sqrt(v / (1.0 - 0.999 ** i)) + 1e-8)
        return torch.minimum(torch.maximum(x - step, self.box[0]), self.box[1]), m, v


def _selected(z, floor, top, rand, seed, refresh_index):
    """Positions of the contingencies a screened step scores: the worst ones
    and a uniform draw by SplitMix64 keys from the rest."""
    K = z.shape[1]
    n_top = min(K, math.ceil(top * K))
    n_act = min(K, n_top + math.ceil(rand * K))
    sev = torch.clamp((z - floor[:, None]).max(dim=0).values, min=0.0).cpu().numpy()
    worst = [int(k) for k in np.lexsort((np.arange(K), -sev)) if sev[k] > 0.0][:n_top]
    mask, keys = (1 << 64) - 1, []
    for k in range(K):
        s = (seed + 0x9E3779B97F4A7C15 * ((refresh_index << 32) + k + 1)) & mask
        s = ((s ^ (s >> 30)) * 0xBF58476D1CE4E5B9) & mask
        s = ((s ^ (s >> 27)) * 0x94D049BB133111EB) & mask
        keys.append(s ^ (s >> 31))
    rest = sorted(set(range(K)) - set(worst), key=lambda k: (keys[k], k))
    chosen = sorted(worst + rest[:n_act - len(worst)])
    return torch.as_tensor(chosen, device=DEV)


def _exact_solve(case, g, x, m, v, seed):
    model = _Exact(g)
    x, m, v = (torch.as_tensor(a, device=DEV) for a in (x, m, v))
    cols, last = None, None
    for i in range(_begin(case) + 1, _begin(case) + 1 + case["steps"]):
        eps, beta, rho, lr = _params(i)
        if case["kind"] == "screen" and (i - 1) % case["refresh"] == 0:
            last, grad, z = model(x, eps, beta, rho, want_z=True)
            floor = model.c["dt"] * g.c_s * beta * (g.n_branch - 1) * eps
            cols = _selected(z, floor, case["top"], case["rand"], seed,
                             (i - 1) // case["refresh"])
        else:
            last, grad = model(x, eps, beta, rho, cols)
        x, m, v = model.adam(x, m, v, grad, i, lr)
    out = dict(x=x, m=m, v=v)
    if case.get("final"):
        # at eps = 0 the kinks have no derivative; only the values are used
        terms = model(x, 0.0, 1.0, RAMP[1])[0]
        out.update(loss=float(last[9]), score=-float(terms[9]), terms=terms)
    return out


def _exact_net(case, seed):
    d64 = lambda ts: [a.double() for a in ts]  # noqa: E731
    given = _net_inputs(case, seed)
    layers, x = given["layers"], given["x"]
    if case["kind"] == "net_bf16":
        layers, x = [w.bfloat16() for w in layers], x.bfloat16()
    train = case["kind"] == "net_train"
    layers = [w.requires_grad_(train) for w in d64(layers)]
    h = x.double()
    for i in range(case["depth"]):
        h = torch.nn.functional.gelu(h @ layers[2 * i] + layers[2 * i + 1])
    y = h @ layers[-2] + layers[-1]
    if not train:
        return y
    loss = ((y - given["t"].double()) ** 2).mean()
    grads = torch.autograd.grad(loss, layers)
    it = NET_ITER + 1
    b1, b2 = 1.0 - 0.9 ** it, 1.0 - 0.999 ** it
    up = lambda n: -(-n // 64) * 64  # noqa: E731  each array starts at a multiple of 64 floats
    flat = {k: [] for k in ("params", "m", "v")}
    for w, m, v, gr in zip(layers, d64(given["m"]), d64(given["v"]), grads):
        m = 0.9 * m + 0.1 * gr
        v = 0.999 * v + 0.001 * gr * gr
        w = w.detach() - NET_LR * (m / b1) / (torch.sqrt(v / b2) + 1e-8)
        for k, a in (("params", w), ("m", m), ("v", v)):
            flat[k] += [a.reshape(-1), a.new_zeros(up(a.numel()) - a.numel())]
    return dict(loss=loss.detach(), **{k: torch.cat(a) for k, a in flat.items()})


def exact(case, seed):
    kind = case["kind"]
    if kind.startswith("net"):
        return _exact_net(case, seed)
    outs = []
    for i, g in enumerate(_grids(case)):
        g, x, m, v = _day(g, seed + 1000 * i)
        if kind == "eval":
            model = _Exact(g)
            x, m, v = (torch.as_tensor(a, device=DEV) for a in (x, m, v))
            eps, beta, rho, lr = _params(_begin(case) + 1)
            terms, grad = model(x, eps, beta, rho)
            if not case["adam"]:
                return dict(terms=terms, grad=grad)
            x, m, v = model.adam(x, m, v, grad, _begin(case) + 1, lr)
            return dict(terms=terms, grad=grad, x=x, m=m, v=v)
        outs.append(_exact_solve(case, g, x, m, v, seed))
    merged = {k: [o[k] for o in outs] for k in ("x", "m", "v")}
    merged.update({k: outs[0][k] for k in ("loss", "score", "terms") if k in outs[0]})
    return merged
