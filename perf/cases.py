"""Work that users of this library have it do, as cases that can be timed and compared.

Every case goes through the public binding (`hsf.Context`, `hsf.Net`,
`hsf.evaluate_static`) with device buffers, as the coupled runs, the inversions and the
warm-start training use it.  Sizes and parameters are those of `workloads.py` (16^3 A4B4
melt, 64^3 A8B8 melt pair, batches of A3B9 + S solutions, 128^3 vesicle solution) and of
the warm-start networks; `draw` varies boxes (odd and non-cubic ones among them), chains,
precision, replicas and options over the same ranges.

Inputs are made from the seed with torch alone.  `exact` evaluates the same formulas in
float64 with plain torch operations.
"""
import numpy as np
import torch

from paper_1204_2088_amd import hsf
from paper_1204_2088_amd import workloads as W

F64 = torch.float64


# ---- the cases -------------------------------------------------------------------------

def listed():
    return [
        # one evaluation of the density functional at given fields: the smallest box in use ...
        dict(name="eval_16_fp64", kind="eval", Lx=16, Ly=16, Lz=16, replicas=1, n_a=4, n_b=4, solvent=False,
             precision="fp64"),
        # ... the melt at two viscosities as two replicas of one context ...
        dict(name="eval_64x2_fp32", kind="eval", Lx=64, Ly=64, Lz=64, replicas=2, n_a=8, n_b=8, solvent=False,
             precision="fp32"),
        # ... a batch of solutions of mixed box sizes (32, 48, 64 in turn) ...
        dict(name="eval_batch12_fp32", kind="eval", Lx=0, Ly=0, Lz=0, replicas=12, n_a=3, n_b=9, solvent=True,
             precision="fp32"),
        # ... and the vesicle solution, the largest
        dict(name="eval_128_fp32", kind="eval", Lx=128, Ly=128, Lz=128, replicas=1, n_a=3, n_b=9, solvent=True,
             precision="fp32"),
        # the allocation-free evaluation of a serving loop, on a ragged box
        dict(name="static_40x36x30_fp32", kind="static", Lx=40, Ly=36, Lz=30, n_a=3, n_b=9, solvent=True,
             precision="fp32"),
        # one coupled step (inversion to 1e-8, force, LB, convection-diffusion): the small FP64 melt ...
        dict(name="step_16_fp64", kind="step", Lx=16, Ly=16, Lz=16, n_a=4, n_b=4, solvent=False, precision="fp64"),
        # ... and the vesicle solution: FP32 propagators, finished with FP64 evaluations
        dict(name="step_128_fp32", kind="step", Lx=128, Ly=128, Lz=128, n_a=3, n_b=9, solvent=True,
             precision="fp32"),
        # eight lattice-Boltzmann steps under a force field: FP32 population storage, BGK
        dict(name="lb_128_fp32", kind="lb", Lx=128, Ly=128, Lz=128, steps=8, lb="bgk", noise=False,
             precision="fp32"),
        # the fluctuating fluid: MRT collision with mode noise, FP64 populations
        dict(name="lb_noise_64_fp64", kind="lb", Lx=64, Ly=64, Lz=64, steps=4, lb="mrt", noise=True,
             precision="fp64"),
        # chemical potential and force, then the convection-diffusion update
        dict(name="dynamics_128", kind="dynamics", Lx=128, Ly=128, Lz=128, n_a=3, n_b=9, solvent=True, noise=False),
        # a warm-start prediction of the one-level network, two boxes at once
        dict(name="net_forward_64x2", kind="net_forward", L=64, batch=2, in_ch=4, depth=1, width=16),
        # loss and gradient of the four-level network (training)
        dict(name="net_grad_64x2", kind="net_grad", L=64, batch=2, in_ch=6, depth=4, width=8),
    ]


def _size(rng, lo, hi):
    """A box length, spread over the logarithm of the range, odd ones among them."""
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng):
    kind = rng.choice(["eval", "eval", "eval", "static", "step", "lb", "dynamics", "net_forward", "net_grad"])
    box = lambda lo, hi: dict(Lx=_size(rng, lo, hi), Ly=_size(rng, lo, hi), Lz=_size(rng, lo, hi))
    if kind == "eval":
        c = dict(kind=kind, replicas=rng.choice([1, 1, 2, 3]), solvent=rng.random() < 0.5,
                 precision=rng.choice(["fp32", "fp32", "fp64"]), **box(12, 100))
        c.update(zip(("n_a", "n_b"), rng.choice([(4, 4), (8, 8), (4, 12), (3, 9), (5, 11), (2, 8)])))
        return c
    if kind == "static":
        c = dict(kind=kind, solvent=rng.random() < 0.5, precision=rng.choice(["fp32", "fp64"]), **box(12, 48))
        c.update(zip(("n_a", "n_b"), rng.choice([(4, 4), (3, 9), (8, 8)])))
        return c
    if kind == "step":
        c = dict(kind=kind, solvent=rng.random() < 0.5, precision=rng.choice(["fp32", "fp64"]), **box(12, 56))
        c.update(zip(("n_a", "n_b"), rng.choice([(4, 4), (3, 9), (8, 8)])))
        return c
    if kind == "lb":
        return dict(kind=kind, steps=rng.randint(1, 8), lb=rng.choice(["bgk", "mrt"]), noise=rng.random() < 0.3,
                    precision=rng.choice(["fp32", "fp64"]), **box(16, 100))
    if kind == "dynamics":
        return dict(kind=kind, n_a=8, n_b=8, solvent=rng.random() < 0.5, noise=rng.random() < 0.3, **box(16, 112))
    depth = rng.choice([1, 2, 3, 4])
    q = 1 << (depth - 1)
    return dict(kind=kind, L=q * max(2, _size(rng, 16, 64) // q), batch=rng.randint(1, 2), in_ch=rng.choice([2, 4, 6]),
                depth=depth, width=rng.choice([8, 12, 16]) if depth == 1 else 8)


def _boxes(c):
    if c["kind"] == "eval" and c["Lx"] == 0:
        return [((32, 48, 64)[r % 3],) * 3 for r in range(c["replicas"])]
    return [(c["Lx"], c["Ly"], c["Lz"])] * c.get("replicas", 1)


def _workload(c, L, r=0):
    n_a, n_b, solvent = c.get("n_a", 8), c.get("n_b", 8), c.get("solvent", False)
    N = n_a + n_b
    chi = W.chi_matrix(ab=25 / N, bs=35 / N) if solvent else W.chi_matrix(ab=20 / N)
    tau = 0.8 + 0.2 * (r % 3)
    return W.Workload(name=c["kind"], L=tuple(L), types=W.chain(n_a, n_b), has_solvent=solvent, chi=chi, tau=tau,
                      noise=0.005, seed=r, phi_p=0.12 if solvent else 1.0, precision=c.get("precision", "fp64"),
                      lb=c.get("lb", "bgk"),
                      gammas=W.mrt_gammas(tau) if c.get("lb") == "mrt" else (0.0, 0.0, 0.0))


def _workloads(c):
    return [_workload(c, L, r) for r, L in enumerate(_boxes(c))]


# ---- inputs ----------------------------------------------------------------------------

def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(1000003 * int(seed) + 17)
    return g


def _smooth(g, n, shape, rounds=3):
    """Smooth random fields [n][Lz][Ly][Lx] of mean 0 and rms 1."""
    x = torch.rand((n,) + tuple(shape), dtype=F64, device="cuda", generator=g) - 0.5
    for _ in range(rounds):
        for d in (1, 2, 3):
            x = (x + x.roll(1, d) + x.roll(-1, d)) / 3
    x = x - x.mean(dim=(1, 2, 3), keepdim=True)
    return x / x.square().mean(dim=(1, 2, 3), keepdim=True).sqrt().clamp_min(1e-12)


def _phi(g, wl, contrast=0.3):
    """Compositions with exact bulk amounts: a melt or a dilute solution that is segregating."""
    f = sum(1 for t in wl.types if t == W.A) / wl.N
    a, b = _smooth(g, 2, wl.shape).clamp(-3, 3)
    fluct = lambda x: (lambda y: y / y.mean())(1 + contrast * x / 3)
    if not wl.has_solvent:
        pa = f * fluct(a)
        return torch.stack([pa, 1 - pa])
    pa, pb = wl.phi_p * f * fluct(a), wl.phi_p * (1 - f) * fluct(b)
    return torch.stack([pa, pb, 1 - pa - pb])


def _eval_inputs(c, seed):
    """Per replica: fields of a segregated state (a few kT) and the current densities."""
    g = _gen(seed)
    return [(0.8 * _smooth(g, wl.nsp, wl.shape), _phi(g, wl)) for wl in _workloads(c)]


def _cat(parts):
    return torch.cat([p.reshape(-1) for p in parts]).contiguous()


def _velocity_set():
    cx = [0, 1, -1, 0, 0, 0, 0, 1, -1, 1, -1, 1, -1, 1, -1, 0, 0, 0, 0]
    cy = [0, 0, 0, 1, -1, 0, 0, 1, -1, -1, 1, 0, 0, 0, 0, 1, -1, 1, -1]
    cz = [0, 0, 0, 0, 0, 1, -1, 0, 0, 0, 0, 1, -1, -1, 1, 1, -1, -1, 1]
    w = [1 / 3] + [1 / 18] * 6 + [1 / 36] * 12
    return list(zip(cx, cy, cz)), w


def _populations(g, shape):
    """A slowly moving fluid: density 1 to a part in a thousand, velocities of a few 1e-3."""
    cs, w = _velocity_set()
    rho = 1 + 1e-3 * _smooth(g, 1, shape)[0]
    u = 2e-3 * _smooth(g, 3, shape)
    return torch.stack([w[q] * rho * (1 + 3 * (cs[q][0] * u[0] + cs[q][1] * u[1] + cs[q][2] * u[2]))
                        for q in range(19)])


def _lb_inputs(c, seed):
    g = _gen(seed)
    shape = (c["Lz"], c["Ly"], c["Lx"])
    return _populations(g, shape), 1e-5 * _smooth(g, 3, shape)


def _dynamics_inputs(c, seed):
    g = _gen(seed)
    wl = _workloads(c)[0]
    return 0.8 * _smooth(g, wl.nsp, wl.shape), _phi(g, wl), 2e-3 * _smooth(g, 3, wl.shape)


def _step_inputs(c, seed):
    g = _gen(seed)
    wl = _workloads(c)[0]
    phi0 = _phi(g, wl, contrast=0.1)   # early after the quench
    change = 1 + 0.002 * _smooth(g, 2, wl.shape).clamp(-3, 3)
    # the next step's densities: a small change that keeps every species' amount
    p = phi0[:2] * change
    p = p * (phi0[:2].mean(dim=(1, 2, 3), keepdim=True) / p.mean(dim=(1, 2, 3), keepdim=True))
    if wl.has_solvent:
        p = torch.cat([p, (1 - p.sum(0))[None]])
    return phi0, p, _populations(g, wl.shape)


def _net_widths(c):
    return tuple(c["width"] * (k + 1) for k in range(c["depth"]))


def _net_layers(c):
    w, shapes, prev = _net_widths(c), [], c["in_ch"]
    for v in w:
        shapes += [(prev, v), (v, v)]
        prev = v
    for l in range(len(w) - 2, -1, -1):
        shapes += [(w[l + 1], w[l]), (w[l], w[l])]
    return shapes + [(w[0], 2)]


def _net_inputs(c, seed):
    """Flat FP32 parameters (He-like), the network's input and a training target."""
    g = _gen(seed)
    parts = []
    for ci, co in _net_layers(c):
        parts.append(torch.randn(co * ci * 27, device="cuda", generator=g) * (2.0 / (27 * ci)) ** 0.5)
        parts.append(torch.randn(co, device="cuda", generator=g) * 0.05)
    L, B = c["L"], c["batch"]
    x = torch.stack([_smooth(g, c["in_ch"], (L, L, L), 1) for _ in range(B)]).float().contiguous()
    y = torch.stack([_smooth(g, 2, (L, L, L), 2) for _ in range(B)]).float().contiguous()
    return torch.cat(parts).contiguous(), x, y


# ---- what a user's program has in hand ------------------------------------------------

def _context(c, tune=True):
    ctx = hsf.Context(_workloads(c), stream=torch.cuda.current_stream())
    if c.get("solvent"):
        ctx.set_solver(precond=True, refine=c.get("kind") == "step" and c["precision"] == "fp32")
    elif c.get("kind") == "step" and c["precision"] == "fp32":
        ctx.set_solver(refine=True)
    if tune:
        ctx.autotune(reps=3)
    return ctx


def prepare(case, seed):
    c, kind = case, case["kind"]
    s = {"case": c}
    empty = lambda n: torch.empty(n, dtype=F64, device="cuda")
    if kind == "eval":
        inputs = _eval_inputs(c, seed)
        s["ctx"] = ctx = _context(c)
        ctx.set_densities(_cat([p for _, p in inputs]))
        s.update(w=_cat([w for w, _ in inputs]), out=empty(ctx.nsp * ctx.T))
    elif kind == "static":
        (w, phi), = _eval_inputs(c, seed)
        s.update(wl=_workloads(c)[0], w=w.contiguous(), phi=phi.contiguous(), out=torch.empty_like(w), q=empty(1))
    elif kind == "step":
        phi0, phi1, n = _step_inputs(c, seed)
        s["ctx"] = ctx = _context(c)
        # the fields of the step before, converged; the step starts from them
        ctx.set_densities(_cat([phi0]))
        ctx.invert(tol=1e-10, max_iter=4000, warm=hsf.WARM_LOCAL, allow_noconv=True)
        w = empty(ctx.nsp * ctx.T)
        ctx.get_fields(out=w)
        s.update(phi=_cat([phi1]), w=w, n=_cat([n]), out=empty(ctx.nsp * ctx.T), out_n=empty(19 * ctx.T))
    elif kind == "lb":
        n, f = _lb_inputs(c, seed)
        s["ctx"] = ctx = _context(c, tune=False)
        s.update(n=_cat([n]), f=_cat([f]), out=empty(19 * ctx.T), rho=empty(ctx.T), u=empty(3 * ctx.T), seed=int(seed))
    elif kind == "dynamics":
        w, phi, u = _dynamics_inputs(c, seed)
        s["ctx"] = ctx = _context(c, tune=False)
        ctx.set_fields(_cat([w]))
        n = ctx.nsp * ctx.T
        s.update(phi=_cat([phi]), u=_cat([u]), mu=empty(n), f=empty(3 * ctx.T), out=empty(n), seed=int(seed))
    else:
        p, x, y = _net_inputs(c, seed)
        s["net"] = net = hsf.Net(c["in_ch"], 2, _net_widths(c), stream=torch.cuda.current_stream())
        net.set_params(p)
        s.update(x=x, y=y, out=torch.empty_like(y))
    return s


def run(state):
    s, c = state, state["case"]
    kind, ctx = c["kind"], state.get("ctx")
    if kind == "eval":
        ctx.set_fields(s["w"])
        phi, q = ctx.evaluate(out=s["out"])
        return {"phi": phi, "Q": q}
    if kind == "static":
        if hsf.evaluate_static(s["wl"], s["w"], s["phi"], s["out"], s["q"]) != hsf.HSF_OK:
            raise RuntimeError("evaluate_static refused the case")
        return {"phi": s["out"], "Q": s["q"]}
    if kind == "step":
        ctx.set_densities(s["phi"])
        ctx.set_fields(s["w"])
        ctx.set_lb(s["n"])
        ctx.step(1, tol=1e-8, max_iter=4000)
        return {"phi": ctx.get_densities(out=s["out"]), "n": ctx.get_lb(out=s["out_n"])}
    if kind == "lb":
        if c["noise"]:
            ctx.set_noise(cd=False, lb=True, omega=400.0, seed=s["seed"], step=0)
        ctx.set_lb(s["n"])
        ctx.lb_advance(c["steps"], s["f"])
        rho, u = ctx.get_flow(s["rho"], s["u"])
        return {"n": ctx.get_lb(out=s["out"]), "rho": rho, "u": u}
    if kind == "dynamics":
        if c["noise"]:
            ctx.set_noise(cd=True, lb=False, omega=400.0, seed=s["seed"], step=0)
        ctx.set_densities(s["phi"])
        ctx.mu_force(s["mu"], s["f"])
        ctx.cd_advance(s["mu"], s["u"])
        return {"mu": s["mu"], "force": s["f"], "phi": ctx.get_densities(out=s["out"])}
    if kind == "net_forward":
        return s["net"].forward(s["x"], c["batch"], c["L"], out=s["out"])
    loss, grad = s["net"].loss_grad(s["x"], s["y"], c["batch"], c["L"])
    return {"loss": loss, "grad": grad}


# ---- what a pass cannot do without ----------------------------------------------------

def work(case):
    c, kind = case, case["kind"]
    nsp = 3 if c.get("solvent") else 2
    if kind in ("eval", "static"):
        # fields and densities in, densities out; a separable stencil and a product per step
        V = sum(a * b * d for a, b, d in _boxes(c))
        N = c["n_a"] + c["n_b"]
        return {"bytes": 3 * 8 * nsp * V, "flops": 2 * N * 10 * V}
    if kind == "step":
        # one evaluation at the least, densities and populations in and out
        V, N = c["Lx"] * c["Ly"] * c["Lz"], c["n_a"] + c["n_b"]
        return {"bytes": (3 * 8 * nsp + 2 * 8 * 19) * V, "flops": (2 * N * 10 + 250) * V}
    if kind == "lb":
        V = c["Lx"] * c["Ly"] * c["Lz"]
        return {"bytes": 8 * (2 * 19 + 3 + 4) * V, "flops": 250 * c["steps"] * V}
    if kind == "dynamics":
        V = c["Lx"] * c["Ly"] * c["Lz"]
        return {"bytes": 8 * (2 * nsp + 3 + 2 * nsp + 3) * V, "flops": nsp * 80 * V}
    V = c["batch"] * c["L"] ** 3
    flops, size = 0, sum(27 * ci * co + co for ci, co in _net_layers(c))
    w = _net_widths(c)
    at = [0]
    for l in range(len(w)):
        at += [l, l]
    for l in range(len(w) - 2, -1, -1):
        at += [l, l]
    at = at[1:] + [0]
    for (ci, co), l in zip(_net_layers(c), at):
        flops += 2 * 27 * ci * co * V // 8 ** l
    if kind == "net_forward":
        return {"bytes": 4 * (c["in_ch"] + 2) * V + 4 * size, "flops": flops}
    return {"bytes": 4 * (c["in_ch"] + 2) * V + 8 * size, "flops": 3 * flops}


# ---- the same in 64 bits with torch ---------------------------------------------------

def _sigma(x, a=1.1543):
    al = a * a / 6.0
    for d in (-1, -2, -3):
        x = (1 - 2 * al) * x + al * (x.roll(1, d) + x.roll(-1, d))
    return x


def _evaluate(wl, w, phi):
    E, N = torch.exp(-w), wl.N
    G = [E[wl.types[0]] * _sigma(torch.ones_like(w[0]))]
    for s in range(1, N):
        G.append(E[wl.types[s]] * _sigma(G[-1]))
    Q = float(G[-1].mean())
    out = torch.zeros_like(w)
    back = torch.ones_like(w[0])
    for s in range(N - 1, -1, -1):
        sig = _sigma(back)
        out[wl.types[s]] += G[s] * sig
        back = E[wl.types[s]] * sig
    out[:2] *= float((phi[0] + phi[1]).mean()) / (N * Q)
    if wl.has_solvent:
        out[2] = phi[2].mean() * E[2] / E[2].mean()
    return out, Q


def _mu_force(wl, w, phi):
    sp = [_sigma(p) for p in phi]
    mu = torch.stack([-w[i] + sum(float(wl.chi[i, j]) * sp[j] for j in range(wl.nsp)) + wl.kappa * (phi.sum(0) - 1)
                      for i in range(wl.nsp)])
    f = torch.stack([-wl.dt ** 2 * sum(phi[i] * 0.5 * (mu[i].roll(-1, d) - mu[i].roll(1, d)) for i in range(wl.nsp))
                     for d in (2, 1, 0)])
    return mu, f


def _cd(wl, phi, mu, u):
    out = phi.clone()
    for i in range(wl.nsp):
        for a, d in enumerate((2, 1, 0)):
            p, m, v = phi[i], mu[i], u[a]
            pe, me, ve = p.roll(-1, d), m.roll(-1, d), v.roll(-1, d)
            J = -wl.dt * 0.5 * (p + pe) * (me - m) + (0.5 * (p + pe) - 0.5 * (pe * ve - p * v)) * 0.5 * (v + ve)
            out[i] -= J - J.roll(1, d)
    return out


def _lb_bgk(n, f, tau, steps):
    cs, w = _velocity_set()
    for _ in range(steps):
        rho = n.sum(0)
        j = [sum(cs[q][a] * n[q] for q in range(19)) for a in range(3)]
        u = torch.stack([(j[a] + 0.5 * f[a]) / rho for a in range(3)])
        uu, uf = (u * u).sum(0), (u * f).sum(0)
        new = torch.empty_like(n)
        for q in range(19):
            cu = sum(cs[q][a] * u[a] for a in range(3))
            cf = sum(cs[q][a] * f[a] for a in range(3))
            eq = w[q] * rho * (1 + 3 * cu + 4.5 * cu * cu - 1.5 * uu)
            F = (1 - 0.5 / tau) * w[q] * (3 * (cf - uf) + 9 * cu * cf)
            new[q] = (n[q] - (n[q] - eq) / tau + F).roll((cs[q][2], cs[q][1], cs[q][0]), (0, 1, 2))
        n = new
    return n, rho, u


def _conv(x, Wt, b):
    """Periodic 3x3x3 convolution by 27 shifted products, float64."""
    B, C, L = x.shape[0], x.shape[1], x.shape[-1]
    out = b.reshape(1, -1, 1, 1, 1).expand(B, -1, L, L, L).clone()
    for k in range(27):
        dz, dy, dx = k // 9 - 1, (k // 3) % 3 - 1, k % 3 - 1
        xs = x.roll((-dz, -dy, -dx), (2, 3, 4)).reshape(B, C, -1)
        out = out + torch.stack([Wt[:, :, k] @ xs[i] for i in range(B)]).reshape(out.shape)
    return out


def _net(c, p, x):
    layers, off = [], 0
    for ci, co in _net_layers(c):
        layers.append((p[off:off + 27 * ci * co].reshape(co, ci, 27), p[off + 27 * ci * co:off + 27 * ci * co + co]))
        off += 27 * ci * co + co
    F = torch.nn.functional
    conv = lambda i, h: F.silu(_conv(h, *layers[i]))
    up = lambda h: h.repeat_interleave(2, 2).repeat_interleave(2, 3).repeat_interleave(2, 4)

    def pool(h):
        B, C, L = h.shape[0], h.shape[1], h.shape[-1] // 2
        return h.reshape(B, C, L, 2, L, 2, L, 2).mean(dim=(3, 5, 7))

    D, enc, h = c["depth"], [], x
    for l in range(D):
        h = conv(2 * l + 1, conv(2 * l, h if l == 0 else pool(h)))
        enc.append(h)
    i = 2 * D
    for l in range(D - 2, -1, -1):
        h = conv(i + 1, conv(i, up(h)) + enc[l])
        i += 2
    return _conv(h, *layers[i])


def exact(case, seed):
    c, kind = case, case["kind"]
    if kind in ("eval", "static"):
        done = [_evaluate(wl, w, phi) for wl, (w, phi) in zip(_workloads(c), _eval_inputs(c, seed))]
        q = np.array([Q for _, Q in done])
        if kind == "static":
            return {"phi": done[0][0], "Q": torch.from_numpy(q)}
        return {"phi": _cat([p for p, _ in done]), "Q": q}
    if kind == "lb" and not c["noise"] and c["lb"] == "bgk":
        n, f = _lb_inputs(c, seed)
        n, rho, u = _lb_bgk(n, f, _workloads(c)[0].tau, c["steps"])
        return {"n": _cat([n]), "rho": _cat([rho]), "u": _cat([u])}
    if kind == "dynamics":
        wl = _workloads(c)[0]
        w, phi, u = _dynamics_inputs(c, seed)
        mu, f = _mu_force(wl, w, phi)
        return {"mu": _cat([mu]), "force": _cat([f]), "phi": None if c["noise"] else _cat([_cd(wl, phi, mu, u)])}
    if kind in ("net_forward", "net_grad"):
        p, x, y = _net_inputs(c, seed)
        p, x, y = p.double(), x.double(), y.double()
        if kind == "net_forward":
            return _net(c, p, x)
        p.requires_grad_(True)
        loss = ((_net(c, p, x) - y) ** 2).mean()
        loss.backward()
        return {"loss": float(loss.detach()), "grad": p.grad.detach().cpu().numpy()}
    return None   # the inversion's result is defined by its tolerance; the noise by its generator
