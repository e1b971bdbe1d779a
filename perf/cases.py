"""The work that is timed: what programs that use this library have it do.

A case is one call pattern at one size.  Grid cases (`call` "run") restore a
state and advance it by `steps` Runge-Kutta steps through Solver.run, as a
parameter study or an ensemble does; `call` "rhs" evaluates the operator once,
as a program with its own time integrator does; batch cases advance many
uneven tubes through one plan; the training case is one step of the
learned-weight training loop.

States are synthetic and drawn from the seed:
  start      the workloads' initial conditions: a body (bubble, cylinder,
             droplet) at rest in a fluid and a planar shock, piecewise constant
  developed  the same some hundred steps on: the interface spread over three
             cells and waves around the body, which die out to rounding size at
             `reach` of the domain's height from its surface; beyond, the flow
             is still uniform.  In runs of the 2D workloads the share of cells
             equal to their neighbours falls from nearly all to about two
             thirds in 50 steps at 512 x 256 and to a third on average over
             the benchmark's run; reach is set near that average
  dense      two phases with waves in every field everywhere: no cell is like
             its neighbour

`exact` evaluates the method in 64 bits with plain torch operations.
"""
import math
import random

import torch

from paper_1707_00592_amd import isweno

# (rho, u, p, gamma, Pinf): fluid ahead of the shock, behind it, and the body
SETUPS = {
    # air bubble in water, 1 GPa water shock moving right
    "bubble": ((1000.0, 0.0, 1e5, 4.4, 6e8), (1230.377, 432.692, 1e9, 4.4, 6e8),
               (1.0, 0.0, 1e5, 1.4, 0.0)),
    # R22 cylinder in air, Ms = 1.22 shock (mirrored to move right)
    "cylinder": ((1.4, 0.0, 1e5, 1.4, 0.0), (1.927, 114.42, 1.57e5, 1.4, 0.0),
                 (4.415, 0.0, 1e5, 1.249, 0.0)),
    # water droplet in air, Mach 2.4 air shock
    "droplet": ((1.0, 0.0, 1e5, 1.4, 0.0), (3.2119, 618.49, 6.5533e5, 1.4, 0.0),
                (1000.0, 0.0, 1e5, 4.4, 6e8)),
}
BC = {"open": 0, "periodic": 1, "wall": 2}
PRECISION = {"f64": isweno.FP64, "f32": isweno.FP32}
WEIGHTS = {"modified": isweno.W_MODIFIED, "basic": isweno.W_BASIC,
           "cutoff": isweno.W_CUTOFF, "learned": isweno.W_MLP}
EPS = 1e-40


def _grid(nx, ny=1, nz=1, *, setup="bubble", state="developed", precision="f64",
          weights="modified", mood=True, bc="open", call="run", steps=1, reach=0.5):
    return {"kind": "grid", "nx": nx, "ny": ny, "nz": nz, "setup": setup, "state": state,
            "precision": precision, "weights": weights, "mood": mood, "bc": bc, "call": call,
            "steps": steps, "reach": reach}


def _batch(problems, nmin, nmax, *, state="start", precision="f64", tuned=True, steps=5):
    return {"kind": "batch", "problems": problems, "nmin": nmin, "nmax": nmax, "state": state,
            "precision": precision, "tuned": tuned, "steps": steps}


def listed():
    return [
        # the gas-liquid shock tube: a program that runs one small 1D problem
        dict(_grid(200, state="start", steps=20), name="tube_200"),
        # the 2D benchmark as it begins
        dict(_grid(1024, 512, state="start", steps=8), name="bubble_1024x512_start"),
        # the 2D benchmark under way
        dict(_grid(1024, 512, steps=4), name="bubble_1024x512"),
        # the float form on the finer grid
        dict(_grid(2048, 1024, precision="f32", steps=4), name="bubble_2048x1024_f32"),
        # the gas cylinder in a channel with walls, cascade off as in the paper
        dict(_grid(3000, 1000, setup="cylinder", mood=False, bc="wall", steps=2, reach=0.6),
             name="cylinder_3000x1000"),
        # one operator evaluation on a periodic box, odd sizes, cut-off weights
        dict(_grid(611, 397, state="dense", weights="cutoff", bc="periodic", call="rhs"),
             name="rhs_611x397_cutoff"),
        # the 3D shock-droplet interaction at its configured size
        dict(_grid(256, 256, 256, setup="droplet", steps=1, reach=0.35), name="droplet_256"),
        # a ragged 3D box with flow everywhere, float form
        dict(_grid(150, 97, 131, setup="droplet", state="dense", precision="f32", steps=2),
             name="dense_150x97x131_f32"),
        # thousands of uneven tubes in one plan, some tens of steps on
        dict(_batch(4096, 128, 4096, state="developed"), name="batch_4096"),
        # a few hundred tubes as drawn, float form, default launch configuration
        dict(_batch(300, 50, 1500, precision="f32", tuned=False),
             name="batch_300_f32"),
        # the learned weights in the solver
        dict(_grid(1024, 512, precision="f32", weights="learned", steps=2),
             name="learned_1024x512"),
        # one training step of the learned weights at the training loop's batch size
        {"kind": "train", "samples": 65536, "name": "train_65536"},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["1d", "2d", "2d", "2d", "3d", "3d", "batch", "batch", "learned", "train"])
    state = rng.choice(["start", "developed", "developed", "dense"])
    precision = rng.choice(["f64", "f64", "f32"])
    weights = rng.choice(["modified", "modified", "cutoff", "basic"])
    bc = rng.choice(["open", "open", "wall", "periodic"])
    call = rng.choice(["run", "run", "rhs"])
    mood = rng.random() < 0.7
    reach = rng.uniform(0.3, 0.7)
    if kind == "1d":
        return _grid(_log(rng, 50, 20000), setup=rng.choice(["bubble", "droplet"]),
                     state=rng.choice(["start", "developed"]), precision=precision,
                     weights=weights, mood=True, call="run", steps=rng.randint(5, 20), reach=reach)
    if kind == "2d":
        return _grid(_log(rng, 60, 3000), _log(rng, 30, 1000), setup=rng.choice(list(SETUPS)),
                     state=state, precision=precision, weights=weights, mood=mood, bc=bc,
                     call=call, steps=rng.randint(1, 3), reach=reach)
    if kind == "3d":
        return _grid(_log(rng, 30, 200), _log(rng, 30, 200), _log(rng, 30, 200),
                     setup=rng.choice(["droplet", "cylinder"]), state=state, precision=precision,
                     weights=weights, mood=mood, bc=bc, call=call, reach=reach)
    if kind == "batch":
        nmin = _log(rng, 20, 300)
        return _batch(_log(rng, 20, 4096), nmin, nmin + _log(rng, 50, 3000),
                      state=rng.choice(["start", "developed"]), precision=precision,
                      tuned=rng.random() < 0.5, steps=rng.randint(1, 5))
    if kind == "learned":
        return _grid(_log(rng, 100, 1200), _log(rng, 60, 600), state=rng.choice(["start", "developed"]),
                     precision="f32", weights="learned", reach=reach)
    return {"kind": "train", "samples": _log(rng, 2000, 100000)}


# ------------------------------------------------------------------ states
def _conservative(rho, vel, p, G, P):
    ke = sum(v * v for v in vel)
    return torch.stack([rho, *[rho * v for v in vel], G * p + P + 0.5 * rho * ke, G, P])


def _material(gamma, pinf):
    return 1.0 / (gamma - 1.0), gamma * pinf / (gamma - 1.0)


def _waves(rng, coords, count=5, shortest=0.06):
    """A sum of plane waves with periods on the unit box, between -1 and 1."""
    out = 0.0
    for _ in range(count):
        ks = [rng.randint(-int(1 / shortest), int(1 / shortest)) for _ in coords]
        ks[0] = ks[0] or 1
        out = out + torch.sin(2 * math.pi * (sum(k * x for k, x in zip(ks, coords)) + rng.random()))
    return out / count


def _state(case, seed):
    """(U, dx): the initial conservative state (nc, N) and the cell sizes."""
    rng = random.Random(seed)
    n = [case["nx"], case["ny"], case["nz"]]
    ndim = 1 + (n[1] > 1) + (n[2] > 1)
    n = n[:ndim]
    h = 1.0 / n[-1]  # square cells, the last axis of length 1
    ax = [(torch.arange(m, dtype=torch.float64, device="cuda") + 0.5) * h for m in n]
    X = [x.view([1] * (ndim - 1 - a) + [-1] + [1] * a).expand(n[::-1]) for a, x in enumerate(ax)]
    ahead, behind, body = SETUPS[case["setup"]]
    L = n[0] * h  # all positions in units of the domain's length and height
    centre = [(0.45 + 0.04 * rng.uniform(-1, 1)) * L] + [0.5 * n[a] * h for a in range(1, ndim)]
    radius = 0.25 * min(n) * h * (1 + 0.1 * rng.uniform(-1, 1))
    if ndim == 1:
        radius = 0.3 * L
    if ndim == 3:
        radius *= 0.5
    strength = 1 + 0.05 * rng.uniform(-1, 1)
    x_shock = centre[0] - radius * (1.5 if case["state"] == "start" else 0.8) - 0.02 * L * rng.random()
    r = torch.sqrt(sum((x - c) ** 2 for x, c in zip(X, centre)))
    unit = [x / (m * h) for x, m in zip(X, n)]
    post = X[0] < x_shock
    if case["state"] == "start":
        a = (r < radius).double()
    else:  # the interface spread over three cells, exactly 0 and 1 beyond them
        a = ((radius - r) / (3 * h) + 0.5).clamp(0.0, 1.0)
    if case["state"] == "dense":
        a = (0.5 + 0.02 / h / 3 * _waves(rng, unit, 3, 0.5)).clamp(0.0, 1.0)
        post = torch.ones_like(post)
    pick = [torch.where(post, torch.full_like(r, behind[k] * (strength if k == 1 else 1.0)),
                        torch.full_like(r, ahead[k])) for k in range(3)]
    Gs, Ps = _material(ahead[3], ahead[4])
    Gb, Pb = _material(body[3], body[4])
    # the size of pressure and velocity waves: a few percent of rho c^2 and c
    # of the fluid a cell is in (of the softer one where the two are mixed)
    def stiffness(f):
        return f[3] * (f[2] + f[4])
    outer = torch.where(post, torch.full_like(r, stiffness(behind)), torch.full_like(r, stiffness(ahead)))
    inner = torch.full_like(r, stiffness(body))
    mixed = (a > 0) & (a < 1)
    K = torch.where(mixed, torch.minimum(outer, inner), torch.where(a > 0.5, inner, outer))
    rho = a * body[0] + (1 - a) * pick[0]
    c_sound = (K / rho).sqrt()
    p = a * body[2] + (1 - a) * pick[2]
    vel = [(1 - a) * pick[1]] + [torch.zeros_like(r)] * (ndim - 1)
    if case["state"] == "dense":  # one pressure and velocity level through both phases
        p, vel[0] = pick[2], pick[1]
        window = torch.ones_like(r)
    elif case["state"] == "developed":
        # full waves near the body's surface, dying out to rounding size where
        # the scheme's own stencil has carried them, and nothing beyond
        height = min(n) * h if ndim > 1 else L
        far = (r - radius).abs() / (case["reach"] * height)
        window = torch.exp(-36 * (far - 0.3).clamp(min=0.0) / 0.7) * (far < 1)
    if case["state"] != "start":
        rho = rho * (1 + 0.02 * window * _waves(rng, unit))
        p = p + 0.02 * K * window * _waves(rng, unit)
        vel = [v + 0.03 * c_sound * window * _waves(rng, unit) for v in vel]
    U = _conservative(rho, vel, p, a * Gb + (1 - a) * Gs, a * Pb + (1 - a) * Ps)
    return U.reshape(4 + ndim, -1).contiguous(), (h,) * ndim


def _tubes(case, seed):
    """(U, offsets, dx) of independent two-phase shock tubes of uneven length."""
    rng = random.Random(seed)
    lengths = random.Random(case["problems"])  # the same lengths whatever the seed
    sizes = [lengths.randint(case["nmin"], case["nmax"]) for _ in range(case["problems"])]
    count = torch.tensor(sizes, device="cuda")
    offsets = torch.zeros(len(sizes) + 1, dtype=torch.int64, device="cuda")
    offsets[1:] = torch.cumsum(count, 0)
    problem = torch.repeat_interleave(torch.arange(len(sizes), device="cuda"), count)
    cell = torch.arange(int(offsets[-1]), device="cuda") - offsets[problem]
    left, right = [], []
    for _ in sizes:  # liquid and gas as drawn, the velocities kept from cavitating
        for side in (left, right):
            gamma, pinf = rng.choice([(4.4, 6e8), (1.4, 0.0)])
            rho = 10 ** rng.uniform(2.5, 3) if pinf else 10 ** rng.uniform(0, 1.5)
            side.append((rho, rng.uniform(-20, 20), 10 ** rng.uniform(5, 9 if pinf else 7), gamma, pinf))
    both = torch.tensor([left, right], dtype=torch.float64, device="cuda")
    x0 = torch.tensor([rng.uniform(0.3, 0.7) for _ in sizes], dtype=torch.float64, device="cuda")
    x = (cell + 0.5) / count[problem]
    f = torch.where((x < x0[problem]).unsqueeze(1), both[0][problem], both[1][problem])
    rho, u, p = f[:, 0], f[:, 1], f[:, 2]
    if case["state"] == "developed":  # waves around the interface, of rounding size 400 cells off
        d = (x - x0[problem]) * count[problem]
        w = torch.exp(-0.1 * (d.abs() - 40).clamp(min=0.0)) * (d.abs() < 400)
        phase = rng.random() * 6
        rho = rho * (1 + 0.05 * w * torch.sin(0.35 * d + phase))
        p = p * (1 + 0.1 * w * torch.sin(0.27 * d + phase))
        u = u + 10 * w * torch.sin(0.31 * d)
    G, P = _material(f[:, 3], f[:, 4])
    U = _conservative(rho, [u], p, G, P).contiguous()
    return U, offsets.cpu().numpy(), (1.0 / count.double()).cpu().numpy()


def _network(seed):
    """Float parameters of a network that does what training arrives at: weights
    near the optimal ones, and confidence where the stencil has no kinks (eight
    hidden units carry its second differences to the confidence head)."""
    gen = torch.Generator().manual_seed(seed)

    def rand(size, *shape):
        return size * torch.randn(*shape, generator=gen)

    W1, W2, W3 = rand(0.3, 32, 8), rand(0.05, 32, 32), rand(0.05, 9, 32)
    W1[:8] = 0.0
    for k in range(4):
        W1[k, k:k + 3] = torch.tensor([1.0, -2.0, 1.0])
        W1[4 + k, k:k + 3] = torch.tensor([-1.0, 2.0, -1.0])
    W2[:8] = torch.eye(32)[:8]
    W3[8] = 0.0
    W3[8, :8] = -8.0
    b3 = torch.tensor([math.log(d) for d in (0.4, 0.2, 0.3, 0.1)] * 2 + [2.0])
    b1, b2 = rand(0.1, 32), rand(0.1, 32)
    b1[:8] = b2[:8] = 0.0
    return torch.cat([t.reshape(-1) for t in (W1, b1, W2, b2, W3, b3)]).float().cuda()


def _samples(count, seed):
    """Normalised six-cell stencils, smooth ones and ones with a jump, and the
    weights of eq. (28) of both sides."""
    gen = torch.Generator(device="cuda").manual_seed(seed)

    def rand(*shape):
        return torch.rand(*shape, generator=gen, device="cuda", dtype=torch.float64)

    j = torch.arange(6, device="cuda", dtype=torch.float64)
    smooth = torch.sin(rand(count, 1) * 6.28 + j * (0.05 + 0.6 * rand(count, 1)))
    jump = torch.where(j < (rand(count, 1) * 7).floor(), rand(count, 1), rand(count, 1)) \
        + 0.02 * rand(count, 6)
    w = torch.where(rand(count, 1) < 0.3, jump, smooth)
    lo, hi = w.amin(1, keepdim=True), w.amax(1, keepdim=True)
    w = (w - lo) / (hi - lo)
    water = rand(count, 1) < 0.5
    mat = torch.cat([torch.where(water, 0.85, 0.1), torch.where(water, 0.945, 0.0)], 1)
    v = list(w.unbind(1))
    Y = torch.stack(_omega(*v[:5], "modified", False) + _omega(*v[:0:-1], "modified", False), 1)
    return torch.cat([w, mat.double()], 1).float().contiguous(), Y.float().contiguous()


# ------------------------------------------------------- what a program holds
def prepare(case, seed):
    s = {"case": case, "ctx": isweno.Context(0)}
    if case["kind"] == "train":
        gen = torch.Generator().manual_seed(seed + 1)
        s["X"], s["Y"] = _samples(case["samples"], seed)
        s["P"] = _network(seed)
        # the moments of a training run under way
        s["m"] = (1e-2 * torch.randn(isweno.MLP_NPARAM, generator=gen)).cuda()
        s["v"] = (1e-3 * torch.rand(isweno.MLP_NPARAM, generator=gen) + 1e-4).cuda()
        s["grad"] = torch.zeros_like(s["P"])
        s["loss"] = torch.zeros(1, device="cuda")
        return s
    opts = dict(precision=PRECISION[case["precision"]], cfl=0.5, eps=EPS)
    if case["kind"] == "batch":
        s["U0"], offsets, dx = _tubes(case, seed)
        s["U"] = s["U0"].clone()
        s["plan"] = s["ctx"].batch_plan(offsets, dx, 0, 0)
        s["opts"] = isweno.make_opts(mood=True, **opts)
        s["dt"] = torch.zeros(case["problems"], dtype=torch.float64, device="cuda")
        if case["tuned"]:
            s["plan"].autotune(s["U0"], s["opts"])
        s["plan"].status  # the plan's status array, allocated once
    else:
        s["U0"], dx = _state(case, seed)
        n = [case["nx"], case["ny"], case["nz"]][:len(dx)]
        bc = [BC["periodic" if case["bc"] == "periodic" else "open"]] + [BC[case["bc"]]] * (len(n) - 1)
        grid = isweno.make_grid(n, dx, bc, bc)
        if case["weights"] == "learned":
            s["net"] = torch.zeros(isweno.MLP_NPARAM, dtype=torch.int16, device="cuda")
            s["ctx"].mlp_pack(_network(seed), s["net"])
            opts["mlp_params"] = s["net"]
        s["solver"] = isweno.Solver(
            grid, isweno.make_opts(weights=WEIGHTS[case["weights"]], mood=case["mood"], **opts), s["ctx"])
        s["U"] = s["U0"].clone()
    s["stats"] = isweno.new_stats()
    return s


def run(s):
    case = s["case"]
    if case["kind"] == "train":
        s["ctx"].mlp_loss_grad(s["P"], s["X"], s["Y"], None, s["loss"], s["grad"])
        s["ctx"].mlp_adam(s["P"], s["grad"], s["m"], s["v"], 100, 3e-3)
        return {"loss": s["loss"], "grad": s["grad"], "P": s["P"], "m": s["m"], "v": s["v"]}
    if case["kind"] == "batch":
        s["U"].copy_(s["U0"])
        s["plan"].step(s["U"], s["opts"], s["dt"], case["steps"], s["stats"])
        return {"U": s["U"], "dt": s["dt"], "status": s["plan"].status,
                "stats": s["stats"].view(torch.int64)}
    solver = s["solver"]
    if case["call"] == "rhs":
        solver.ctx.rhs(s["U0"], solver.grid, solver.opts, s["U"], s["stats"])
        return {"dUdt": s["U"], "stats": s["stats"].view(torch.int64)}
    s["U"].copy_(s["U0"])
    solver.run(s["U"], nsteps=case["steps"], stats=s["stats"])
    return {"U": s["U"], "stats": s["stats"].view(torch.int64)}


def work(case):
    """Bytes: every step reads and writes the state once (its stages could stay
    on the chip); operations: those of the method at every face and cell, as
    the formulas count them."""
    if case["kind"] == "train":
        per = 2 * (8 * 32 + 32 * 32 + 32 * 9)
        return {"bytes": case["samples"] * 16 * 4, "flops": 3 * per * case["samples"]}
    if case["kind"] == "batch":
        cells, ndim = case["problems"] * (case["nmin"] + case["nmax"]) / 2, 1
    else:
        cells = case["nx"] * case["ny"] * case["nz"]
        ndim = 1 + (case["ny"] > 1) + (case["nz"] > 1)
    nc = 4 + ndim
    stage = ndim * (1160 + 109 * (ndim - 1) + 3 * nc + 7) - nc + 4 + 3 * ndim
    if case.get("call") == "rhs":
        return {"bytes": 16 * nc * cells, "flops": stage * cells}
    return {"bytes": case["steps"] * 16 * nc * cells,
            "flops": case["steps"] * (3 * stage + 12 * nc - 2) * cells}


# ------------------------------------------------ the method in 64 bits, torch
def _omega(a, b, c, d, e, weights, order3):
    """Nonlinear weights of the four candidates, eqs. (21), (24), (25), (28)."""
    k = 13.0 / 12.0
    t1 = (e - a) - 2 * (d - b)
    t2 = ((e + a) - 4 * (d + b)) + 6 * c
    tau = 0.25 * t1 * t1 + k * t2 * t2
    b1, b2 = (d - c) ** 2, (c - b) ** 2
    b3 = k * (c - 2 * d + e) ** 2 + 0.25 * (3 * c - 4 * d + e) ** 2
    b4 = k * (a - 2 * b + c) ** 2 + 0.25 * (a - 4 * b + 3 * c) ** 2
    r1, r2, r3, r4 = (tau / (x + EPS) for x in (b1, b2, b3, b4))
    if weights != "basic":
        r12 = tau / (k * (b - 2 * c + d) ** 2 + 0.25 * (b - d) ** 2 + EPS)
        r1, r2 = r1 * r12, r2 * r12
    if weights == "cutoff":
        g = [1 + r for r in ((r1, r2) if order3 else (r1, r2, r3, r4))]
        top = g[0]
        for x in g[1:]:
            top = torch.maximum(top, x)
        share = [(x / top) ** 6 for x in g]
        kept = [(x >= 1e-5 * sum(share)).double() for x in share]
        al = [d_k * x for d_k, x in zip((4, 2, 3, 1), kept)]
    else:
        al = [0.4 * (1 + r1), 0.2 * (1 + r2)]
        if not order3:
            al += [0.3 * (1 + r3), 0.1 * (1 + r4)]
    total = sum(al)
    return [x / total for x in al]


def _value(a, b, c, d, e, weights, order3):
    """Eq. (19) on the candidates of eq. (20)."""
    om = _omega(a, b, c, d, e, weights, order3)
    cand = [0.5 * c + 0.5 * d, -0.5 * b + 1.5 * c, c / 3 + 5 * d / 6 - e / 6,
            a / 3 - 7 * b / 6 + 11 * c / 6]
    return sum(w * q for w, q in zip(om, cand))


def _star(q, Sk, Ss):
    """Star flux and velocity of one side, eqs. (15), (18)."""
    rho, un, ut, p, G, P = q[0], q[1], q[2:-3], q[-3], q[-2], q[-1]
    E = G * p + P + 0.5 * rho * (un * un + sum(t * t for t in ut))
    Uk = [rho, rho * un, *[rho * t for t in ut], E, G, P]
    Fk = [rho * un, rho * un * un + p, *[rho * un * t for t in ut], (E + p) * un, G * un, P * un]
    den = Sk - Ss
    same, den = den == 0, torch.where(den == 0, torch.ones_like(den), den)
    pk = p + rho * (Sk - un) * (Ss - un)
    F = []
    for k in range(len(Uk)):
        D = 1.0 if k == 1 else Ss if k == len(Uk) - 3 else 0.0
        F.append(torch.where(same, Fk[k], (Ss * (Sk * Uk[k] - Fk[k]) + Sk * pk * D) / den))
    return F, torch.where(same, un, Ss * (Sk - un) / den)


def _hllc(l, r):
    """Eqs. (14)-(18)."""
    cl2, cr2 = (((q[-2] + 1) * q[-3] + q[-1]) / (q[-2] * q[0]) for q in (l, r))
    sl, sr, ul, ur = l[0].sqrt(), r[0].sqrt(), l[1], r[1]
    ubar = (sl * ul + sr * ur) / (sl + sr)
    cbar = ((sl * cl2 + sr * cr2) / (sl + sr)
            + 0.5 * sl * sr / (sl + sr) ** 2 * (ur - ul) ** 2).sqrt()
    Sl = torch.minimum(ubar - cbar, ul - cl2.sqrt()).clamp(max=0)
    Sr = torch.maximum(ubar + cbar, ur + cr2.sqrt()).clamp(min=0)
    ml, mr = l[0] * (Sl - ul), r[0] * (Sr - ur)
    Ss = (r[-3] - l[-3] + ml * ul - mr * ur) / (ml - mr)
    Fl, usl = _star(l, Sl, Ss)
    Fr, usr = _star(r, Sr, Ss)
    wl = 0.5 * (1 + torch.sign(Ss))
    return [wl * x + (1 - wl) * y for x, y in zip(Fl, Fr)], wl * usl + (1 - wl) * usr


def _admissible(q):
    return (q[0] > 0) & (q[-2] > 0) & ((q[-2] + 1) * q[-3] + q[-1] > 0)


def _face(st, weights, mood):
    """Flux and interface velocity from six cells' face-order primitives."""
    mean = [0.5 * (x + y) for x, y in zip(st[2], st[3])]
    c2 = ((mean[-2] + 1) * mean[-3] + mean[-1]) / (mean[-2] * mean[0])
    c = c2.sqrt()
    rc = mean[0] * c

    def states(order3):
        fields = [[-0.5 * rc * q[1] + 0.5 * q[-3] for q in st], [q[0] - q[-3] / c2 for q in st]]
        fields += [[q[k] for q in st] for k in [*range(2, len(st[0]) - 3), len(st[0]) - 2, len(st[0]) - 1]]
        fields += [[0.5 * rc * q[1] + 0.5 * q[-3] for q in st]]
        sides = []
        for rev in (False, True):
            v = [_value(*(w[:0:-1] if rev else w[:5]), weights, order3) for w in fields]
            sides.append([v[0] / c2 + v[1] + v[-1] / c2, (v[-1] - v[0]) / rc, *v[2:-3],
                          v[0] + v[-1], v[-3], v[-2]])
        return sides

    sides = states(False)
    if mood:
        bad = [~_admissible(q) for q in sides]
        if bool(bad[0].any() | bad[1].any()):
            for k, q3 in enumerate(states(True)):
                ok3 = _admissible(q3)
                sides[k] = [torch.where(bad[k], torch.where(ok3, y, z), x)
                            for x, y, z in zip(sides[k], q3, st[2 + k])]
    return _hllc(*sides)


def _exact_rhs(U, lines, dx, weights, mood, part=1 << 22):
    """dU/dt; lines[d][j]: the cell that stands at distance j - 3 along axis d
    of every cell, and whether its normal velocity is mirrored."""
    ndim = U.shape[0] - 4
    vel = [U[1 + a] / U[0] for a in range(ndim)]
    p = (U[-3] - 0.5 * U[0] * sum(v * v for v in vel) - U[-1]) / U[-2]
    out = torch.zeros_like(U)
    for d in range(ndim):
        order = [d] + [a for a in range(ndim) if a != d]
        for s in range(0, U.shape[1], part):
            cells = []
            for at, flip in lines(d, s, min(U.shape[1], s + part)):
                un = vel[d][at]
                cells.append([U[0][at], torch.where(flip, -un, un), *[vel[a][at] for a in order[1:]],
                              p[at], U[-2][at], U[-1][at]])
            Fa, ua = _face(cells[:6], weights, mood)
            Fb, ub = _face(cells[1:], weights, mood)
            h = dx[d] if not torch.is_tensor(dx[d]) else dx[d][s:s + part]
            rows = [0, *[1 + a for a in order], 1 + ndim, 2 + ndim, 3 + ndim]
            for k, row in enumerate(rows):
                r = (Fa[k] - Fb[k]) / h
                if row >= 2 + ndim:
                    r = r + U[row, s:s + part] * (ub - ua) / h
                out[row, s:s + part] += r
    speed = 0.0
    c = (((U[-2] + 1) * p + U[-1]) / (U[-2] * U[0])).sqrt()
    for d in range(ndim):
        speed = speed + (vel[d].abs() + c) / dx[d]
    return out, speed


def _exact_steps(U, lines, dx, case, top):
    """top(speed): every cell's largest wave speed of the problem it is in."""
    def rhs(V):
        return _exact_rhs(V, lines, dx, case.get("weights", "modified"), case.get("mood", True))

    for _ in range(case["steps"]):
        L, speed = rhs(U)
        dt = 0.5 / top(speed)
        U1 = U + dt * L
        U2 = 0.75 * U + 0.25 * (U1 + dt * rhs(U1)[0])
        U = U / 3 + (2 / 3) * (U2 + dt * rhs(U2)[0])
    return U, dt


def _grid_lines(n, bc):
    n3 = list(n) + [1] * (3 - len(n))
    strides = [1, n3[0], n3[0] * n3[1]]

    def lines(d, s, t):
        cell = torch.arange(s, t, device="cuda")
        l = cell // strides[d] % n3[d]
        m = n3[d]
        for j in range(-3, 4):
            k = l + j
            out = (k < 0) | (k >= m)
            if bc[d] == 1:
                to = k % m
            elif bc[d] == 2:
                to = torch.where(k < 0, -k - 1, torch.where(k >= m, 2 * m - 1 - k, k))
            else:
                to = k.clamp(0, m - 1)
            yield cell + (to - l) * strides[d], out & (bc[d] == 2)
    return lines


def _exact_train(case, seed):
    X, Y = (t.double() for t in _samples(case["samples"], seed))
    s = prepare(case, seed)
    P = s["P"].double().requires_grad_()
    W = torch.split(P, [256, 32, 1024, 32, 288, 9])
    h = torch.relu(X @ W[0].view(32, 8).T + W[1])
    h = torch.relu(h @ W[2].view(32, 32).T + W[3])
    z = h @ W[4].view(9, 32).T + W[5]
    loss, err = 0.0, 0.0
    for side in (0, 1):
        a, b, c, d, e = (X[:, k] for k in ((0, 1, 2, 3, 4) if side == 0 else (5, 4, 3, 2, 1)))
        cand = torch.stack([0.5 * c + 0.5 * d, -0.5 * b + 1.5 * c, c / 3 + 5 * d / 6 - e / 6,
                            a / 3 - 7 * b / 6 + 11 * c / 6], 1)
        off = ((torch.softmax(z[:, 4 * side:4 * side + 4], 1) - Y[:, 4 * side:4 * side + 4]) * cand).sum(1)
        loss = loss + (off / 0.01) ** 2
        err = torch.maximum(off.abs(), err) if side else off.abs()
    label = (err.detach() < 0.005).double()
    loss = (loss + torch.nn.functional.binary_cross_entropy_with_logits(z[:, 8], label, reduction="none")).mean()
    g, = torch.autograd.grad(loss, P)
    m = 0.9 * s["m"].double() + 0.1 * g
    v = 0.999 * s["v"].double() + 0.001 * g * g
    new = P.detach() - 3e-3 * (m / (1 - 0.9 ** 100)) / ((v / (1 - 0.999 ** 100)).sqrt() + 1e-8)
    return {"loss": loss.detach().reshape(1), "grad": g, "P": new, "m": m, "v": v}


def exact(case, seed):
    if case["kind"] == "train":
        return _exact_train(case, seed)
    if case["kind"] == "batch":
        U, offsets, dx = _tubes(case, seed)
        off = torch.from_numpy(offsets).cuda()
        problem = torch.repeat_interleave(torch.arange(len(dx), device="cuda"), off[1:] - off[:-1])
        lo, hi = off[problem], off[problem + 1] - 1

        def lines(d, s, t):
            cell = torch.arange(s, t, device="cuda")
            for j in range(-3, 4):
                to = torch.minimum(torch.maximum(cell + j, lo[s:t]), hi[s:t])
                yield to, torch.zeros_like(to, dtype=torch.bool)

        def top(speed):
            best = torch.zeros(len(dx), dtype=torch.float64, device="cuda")
            best.scatter_reduce_(0, problem, speed, "amax")
            return best[problem]

        U, dt = _exact_steps(U, lines, [torch.from_numpy(dx).cuda()[problem]], case, top)
        return {"U": U, "dt": dt[off[:-1]], "status": None, "stats": None}
    if case["weights"] == "learned":
        return None  # the network works in 16 bits and its fallbacks are yes-or-no decisions
    U, dx = _state(case, seed)
    n = [case["nx"], case["ny"], case["nz"]][:len(dx)]
    lines = _grid_lines(n, [1 if case["bc"] == "periodic" else 0] + [BC[case["bc"]]] * (len(n) - 1))
    if case["call"] == "rhs":
        return {"dUdt": _exact_rhs(U, lines, dx, case["weights"], case["mood"])[0], "stats": None}
    return {"U": _exact_steps(U, lines, dx, case, lambda speed: speed.max())[0], "stats": None}
