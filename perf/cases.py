"""Performance cases of libsfrde: the calls that a program makes once its plan exists.

A case is one call (or a forward call and its adjoint) through the public
``paper_2003_13569_amd.torch_api.Plan``: ``step``, ``integrate`` or
``integrate`` with checkpoints followed by ``backward``. ``listed()`` holds
the repository's own configurations (single problems, the paper's
applications, an ensemble, the two adjoint configurations) and the grids
between them; ``draw()`` spreads the same kinds of call over their ranges of
sizes, boundary conditions, reactions, schemes and types.

``exact()`` is an independent plain-torch implementation of the same step in
64 bits: dense per-axis transform products, the coefficients from their
closed forms, gradients by autograd.
"""
import math

import torch

from paper_2003_13569_amd.torch_api import Plan

TORCH = {"f32": torch.float32, "f64": torch.float64}

# Constants of each reaction's problem: domain length, diffusion coefficients,
# reaction parameters, time step, and the mean of the start fields and the
# spread of their noise (the repository's benchmark recipes).
PROBLEM = {
    "fhn": dict(length=2.5, kappa=(1e-4, 0.0), params=(0.1, 0.01, 0.5, 1.0, 0.0), dt=0.1,
                mean=(0.5, 0.05), spread=(0.05, 0.03)),
    "gray_scott": dict(length=2.0, kappa=(2e-5, 1e-5), params=(0.04, 0.06), dt=1.0,
                       mean=(1.0, 0.0), spread=(0.01, 0.01)),
    "schnakenberg": dict(length=1.0, kappa=(0.05, 1.0), params=(1.0, 0.1305, 0.7695), dt=0.005,
                         mean=(0.9, 0.9), spread=(0.01, 0.01)),
    "gierer_meinhardt": dict(length=2.0, kappa=(1e-3, 0.05), params=(0.1, 1.0, 1.0, 1.0, 1.0),
                             dt=0.05, mean=(1.1, 1.21), spread=(0.01, 0.01)),
}


def _case(call, bc, reaction, dtype, shape, steps, alpha=1.5, beta=None, scheme="p13", batch=0,
          every=0, name=None):
    """shape: slowest axis first; steps of one pass; every: steps between
    checkpoints of an adjoint pass; batch: ensemble members (0: a single plan);
    alpha, beta: the fractional orders of the two species."""
    nz, ny, nx = (0,) * (3 - len(shape)) + tuple(shape)
    case = dict(call=call, bc=bc, reaction=reaction, dtype=dtype, nz=nz, ny=ny, nx=nx, steps=steps,
                alpha=alpha, beta=alpha if beta is None else beta, scheme=scheme, batch=batch,
                every=every)
    return dict(case, name=name) if name else case


def listed():
    return [
        # One step of the 64^2 FitzHugh-Nagumo configuration: a program that looks at the field
        # after every step. All latency.
        _case("step", "neumann", "fhn", "f64", (64, 64), 1, name="fhn64_step_f64"),
        # The paper's Gierer-Meinhardt application, 64 intervals (65 Neumann unknowns), two
        # orders; it runs thousands of steps, here a stretch of them.
        _case("integrate", "neumann", "gierer_meinhardt", "f64", (65, 65), 20, alpha=2.0, beta=1.9,
              name="gm65_f64"),
        # A parameter sweep: 64 members of the 64^2 configuration in one plan.
        _case("integrate", "neumann", "fhn", "f64", (64, 64), 10, batch=64,
              name="fhn64_ensemble64_f64"),
        # The 256^2 Gierer-Meinhardt adjoint configuration, shortened: forward with checkpoints,
        # backward with every gradient.
        _case("adjoint", "neumann", "gierer_meinhardt", "f32", (256, 256), 20, alpha=1.6, every=10,
              name="gm256_adjoint_f32"),
        # The 512^2 Gray-Scott configuration.
        _case("integrate", "periodic", "gray_scott", "f32", (512, 512), 20, alpha=1.7,
              name="grayscott512_f32"),
        # The paper's Gray-Scott application: 265 points per axis.
        _case("integrate", "periodic", "gray_scott", "f64", (265, 265), 10, alpha=2.0,
              name="grayscott265_f64"),
        # The paper's 3D Schnakenberg application, with the exponential scheme.
        _case("integrate", "periodic", "schnakenberg", "f64", (32, 32, 32), 20, alpha=2.0,
              scheme="exp", name="schnakenberg32_f64"),
        # A box with three different axes, none of them a round size.
        _case("integrate", "neumann", "schnakenberg", "f32", (101, 81, 65), 10, alpha=1.8,
              name="schnakenberg_box_f32"),
        # The 128^3 Schnakenberg configuration.
        _case("integrate", "dirichlet", "schnakenberg", "f32", (128, 128, 128), 10, alpha=1.8,
              name="schnakenberg128_f32"),
        # The same in FP64, with its adjoint: gradients that are checked against differences.
        _case("adjoint", "dirichlet", "schnakenberg", "f64", (128, 128, 128), 4, alpha=1.8, every=2,
              name="schnakenberg128_adjoint_f64"),
        # The headline configuration, 256^3.
        _case("integrate", "neumann", "schnakenberg", "f32", (256, 256, 256), 10,
              name="schnakenberg256_f32"),
        # Its adjoint, shortened.
        _case("adjoint", "neumann", "schnakenberg", "f32", (256, 256, 256), 8, every=4,
              name="schnakenberg256_adjoint_f32"),
    ]


def _log_int(rng, lo, hi):
    return min(hi, int(math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))))


def draw(rng):
    bc = rng.choice(("periodic", "dirichlet", "neumann"))
    reaction = rng.choice(tuple(PROBLEM))
    dtype = rng.choice(("f32", "f64"))
    scheme = "exp" if rng.random() < 0.2 else "p13"
    orders = dict(alpha=round(rng.uniform(1.2, 2.0), 3), beta=round(rng.uniform(1.2, 2.0), 3))
    kind = rng.choice(("small", "ensemble", "long", "mid", "big", "adjoint"))
    if kind == "small":  # 2D grids of the paper's examples and applications
        shape, steps = [_log_int(rng, 24, 192) for _ in range(2)], _log_int(rng, 1, 20)
        call = "step" if steps == 1 else "integrate"
        return _case(call, bc, reaction, dtype, shape, steps, scheme=scheme, **orders)
    if kind == "ensemble":
        shape = [_log_int(rng, 32, 96) for _ in range(2)]
        return _case("integrate", bc, reaction, dtype, shape, _log_int(rng, 2, 20), scheme=scheme,
                     batch=_log_int(rng, 8, 256), **orders)
    if kind == "long":  # axes past 256 points
        shape = [rng.choice((256, 512, rng.randint(200, 400))) for _ in range(2)]
        return _case("integrate", bc, reaction, dtype, shape, _log_int(rng, 2, 6), scheme=scheme,
                     **orders)
    if kind == "mid":
        shape = [rng.choice((64, 128, rng.randint(30, 140))) for _ in range(3)]
        return _case("integrate", bc, reaction, dtype, shape, _log_int(rng, 2, 10), scheme=scheme,
                     **orders)
    if kind == "big":
        shape = [rng.choice((192, 256, rng.randint(150, 256))) for _ in range(3)]
        bc = rng.choice(("dirichlet", "neumann"))
        return _case("integrate", bc, reaction, dtype, shape, rng.randint(1, 4), scheme=scheme,
                     **orders)
    if rng.random() < 0.5:
        shape = [rng.choice((64, 128, 256, rng.randint(48, 256))) for _ in range(2)]
        steps, every = _log_int(rng, 4, 20), rng.randint(2, 10)
    else:
        shape = [rng.choice((64, 128, rng.randint(30, 140))) for _ in range(3)]
        steps, every = rng.randint(2, 6), rng.randint(1, 4)
    return _case("adjoint", bc, reaction, dtype, shape, steps, every=min(steps, every),
                 scheme=scheme, **orders)


def _shape(case):
    return tuple(n for n in (case["nz"], case["ny"], case["nx"]) if n > 0)


def _spacing(case):
    length, bc = PROBLEM[case["reaction"]]["length"], case["bc"]
    return tuple(length / (n if bc == "periodic" else n + 1 if bc == "dirichlet" else n - 1)
                 for n in _shape(case))


def _members(case):
    """(alpha, kappa, params) of every member: an ensemble sweeps the orders and
    the first reaction parameter."""
    pr = PROBLEM[case["reaction"]]
    rows = []
    count = max(1, case["batch"])
    for b in range(count):
        f = b / count
        a = (case["alpha"] - 0.2 * f, case["beta"] - 0.2 * f)
        prm = (pr["params"][0] * (1.0 + 0.1 * f),) + pr["params"][1:]
        rows.append((a, pr["kappa"], prm))
    return rows


def _fields(case, seed):
    """Start fields and, for an adjoint, the cotangent of the result."""
    pr, dt = PROBLEM[case["reaction"]], TORCH[case["dtype"]]
    gen = torch.Generator(device="cuda").manual_seed(seed)
    lead = (case["batch"], 2) if case["batch"] else (2,)
    u = torch.randn(lead + _shape(case), generator=gen, device="cuda", dtype=dt)
    bump = torch.ones((), device="cuda", dtype=dt)  # noise on a smooth hill
    for n in _shape(case):
        x = (torch.arange(n, device="cuda", dtype=dt) + 0.5) / n - 0.4
        bump = bump.unsqueeze(-1) * torch.exp(-10.0 * x * x)
    u.add_(bump, alpha=8.0)
    for s in range(2):
        part = u[:, s] if case["batch"] else u[s]
        part.mul_(pr["spread"][s]).add_(pr["mean"][s])
        if case["reaction"] == "gray_scott":  # the disturbed square in the middle
            mid = part[(...,) + tuple(slice(n // 2 - n // 10, n // 2 + n // 10 + 1)
                                      for n in _shape(case))]
            mid.add_(-0.5 if s == 0 else 0.25)
    g = None
    if case["call"] == "adjoint":
        # as of a loss that weighs each species' mean and its square: one part in common, one along
        # the field's own deviation (a cotangent without relation to the field would leave the
        # gradients of the orders and diffusion coefficients as sums that cancel)
        g = torch.stack([(u[s] - pr["mean"][s]) / pr["spread"][s] + 1.0 for s in range(2)])
        g.add_(torch.randn(u.shape, generator=gen, device="cuda", dtype=dt), alpha=0.25)
        g.div_(u[0].numel())
    return u, g


def prepare(case, seed):
    u0, g = _fields(case, seed)
    pr, rows = PROBLEM[case["reaction"]], _members(case)
    alpha, kappa, params = [list(v) for v in zip(*rows)]
    if case["batch"]:
        plan = Plan(_shape(case), case["bc"], _spacing(case), alpha, kappa, pr["dt"],
                    case["reaction"], params, case["dtype"], case["scheme"], batch=case["batch"])
    else:
        plan = Plan(_shape(case), case["bc"], _spacing(case), alpha[0], kappa[0], pr["dt"],
                    case["reaction"], params[0], case["dtype"], case["scheme"])
    state = dict(case=case, plan=plan, u0=u0, u=torch.empty_like(u0))
    if g is not None:
        state.update(g=g, gu0=torch.empty_like(u0),
                     ckpt=plan.new_ckpt(case["steps"], case["every"]))
    return state


def run(state):
    case, plan, u = state["case"], state["plan"], state["u"]
    u.copy_(state["u0"])
    if case["call"] == "step":
        plan.step(u)
        return u
    if case["call"] == "integrate":
        plan.integrate(u, case["steps"])
        return u
    n, every, gu0 = case["steps"], case["every"], state["gu0"]
    plan.integrate(u, n, 0.0, every, state["ckpt"])
    gk, ga, gp = plan.backward(state["ckpt"], n, every, state["g"], 0.0, gu0)
    dt = TORCH[case["dtype"]]
    return {"u": u, "grad_u0": gu0, "grad_kappa": torch.tensor(gk, dtype=dt),
            "grad_alpha": torch.tensor(ga, dtype=dt), "grad_params": torch.tensor(gp, dtype=dt)}


def work(case):
    """Bytes: every step reads the state and writes the next one (an adjoint
    step also reads the state it is taken at and carries the cotangent).
    Operations: a forward and an inverse real fast transform per axis, stage
    and species (2.5 N log2 N each) and about 30 per point for the reaction
    and the stage combine; an adjoint step about three times a forward one."""
    shape = _shape(case)
    pts = math.prod(shape) * 2 * max(1, case["batch"])
    w = 4 if case["dtype"] == "f32" else 8
    step_flops = pts * 4 * (sum(5.0 * math.log2(n) for n in shape) + 30.0)
    if case["call"] == "adjoint":
        return {"bytes": case["steps"] * pts * w * 5.0, "flops": case["steps"] * step_flops * 3.0}
    return {"bytes": case["steps"] * pts * w * 2.0, "flops": case["steps"] * step_flops}


# ------------------------------------------------------------ 64-bit reference
def _axis(bc, n, h):
    """Transform matrix of one axis, its inverse's scale and the eigenvalues of
    the compact fourth-order operator."""
    k = torch.arange(n, dtype=torch.float64, device="cuda")
    kj = torch.outer(k, k)
    if bc == "periodic":
        th = 2 * math.pi * torch.remainder(kj, n) / n
        m, scale, s = torch.cos(th) + torch.sin(th), 1.0 / n, torch.sin(math.pi * k / n)
    elif bc == "dirichlet":
        kj = torch.outer(k + 1, k + 1)
        m = torch.sin(math.pi * torch.remainder(kj, 2 * (n + 1)) / (n + 1))
        scale, s = 2.0 / (n + 1), torch.sin(math.pi * (k + 1) / (2 * (n + 1)))
    else:
        m = torch.cos(math.pi * torch.remainder(kj, 2 * (n - 1)) / (n - 1))
        m[:, 0] *= 0.5
        m[:, -1] *= 0.5
        scale, s = 2.0 / (n - 1), torch.sin(math.pi * k / (2 * (n - 1)))
    return m, scale, 4 * s * s / (h * h * (1 - s * s / 3))


def _along(x, m, axis):
    y = x.movedim(axis, -1)
    return (y.reshape(-1, y.shape[-1]) @ m.T).reshape(y.shape).movedim(-1, axis)


def _phis(z):
    """phi_1, phi_2, phi_3 of z <= 0: Taylor series near 0, else the recurrence."""
    small = z > -2.0
    zs = torch.where(small, z, torch.zeros_like(z))
    zl = torch.where(small, torch.full_like(z, -2.0), z)
    series = []
    for k in (1, 2, 3):
        acc, term = torch.zeros_like(z), torch.full_like(z, 1.0 / math.factorial(k))
        for j in range(1, 36):
            acc = acc + term
            term = term * zs / (k + j)
        series.append(acc)
    p1 = torch.expm1(zl) / zl
    p2 = (p1 - 1) / zl
    p3 = (p2 - 0.5) / zl
    return [torch.where(small, a, b) for a, b in zip(series, (p1, p2, p3))]


def _coefficients(scheme, L, tau):
    if scheme == "p13":
        d, dh = 24 + L * (18 + L * (6 + L)), 192 + L * (72 + L * (12 + L))
        return ((24 - 6 * L) / d, (192 - 24 * L) / dh, tau * (96 + L * (12 + L)) / dh,
                tau * (4 - L) / d, tau * (8 + 2 * L) / d, tau * (4 + L * (3 + L)) / d)
    p1, p2, p3 = _phis(-L)
    h1 = _phis(-0.5 * L)[0]
    return (torch.exp(-L), torch.exp(-0.5 * L), 0.5 * tau * h1, tau * (p1 - 3 * p2 + 4 * p3),
            2 * tau * (p2 - 2 * p3), tau * (4 * p3 - p2))


def _reaction(kind, p, w):
    """p: parameters [members][...] broadcast over the grid; w: [members][2][grid]."""
    u, v = w[:, 0], w[:, 1]
    if kind == "fhn":
        f = (u * (1 - u) * (u - p[0]) - v, p[1] * (p[2] * u - p[3] * v - p[4]))
    elif kind == "gray_scott":
        f = (-u * v * v + p[0] * (1 - u), u * v * v - (p[0] + p[1]) * v)
    elif kind == "schnakenberg":
        f = (p[0] * (p[1] - u + u * u * v), p[0] * (p[2] - u * u * v))
    else:
        f = (p[0] - p[1] * u + p[2] * u * u / v, p[3] * u * u - p[4] * v)
    return torch.stack(f, dim=1)


def exact(case, seed):
    from torch.utils.checkpoint import checkpoint

    u0, g = _fields(case, seed)
    pr, rows, shape = PROBLEM[case["reaction"]], _members(case), _shape(case)
    d, tau = len(shape), pr["dt"]
    grad = case["call"] == "adjoint"

    def leaf(v):
        return torch.tensor(v, dtype=torch.float64, device="cuda").requires_grad_(grad)

    alpha, kappa, params = leaf([r[0] for r in rows]), leaf([r[1] for r in rows]), leaf([r[2] for r in rows])
    axes = [_axis(case["bc"], n, h) for n, h in zip(shape, _spacing(case))]
    lam = sum(a[2].reshape([-1 if i == j else 1 for j in range(d)]) for i, a in enumerate(axes))
    live = lam > 0
    safe = torch.where(live, lam, torch.ones_like(lam))
    ones = (1,) * d

    def hat(x):
        for i, a in enumerate(axes):
            x = _along(x, a[0], 2 + i)
        return x

    def back(x):
        for i, a in enumerate(axes):
            x = _along(x, a[0] * a[1], 2 + i)
        return x

    def step(u, alpha, kappa, params):
        power = torch.where(live, safe ** (0.5 * alpha).reshape(alpha.shape + ones), torch.zeros_like(lam))
        R, Q, phi, phi1, phi2, phi3 = _coefficients(case["scheme"], tau * kappa.reshape(kappa.shape + ones) * power, tau)
        prm = [params[:, k].reshape((-1,) + ones) for k in range(params.shape[1])]
        uh, fu = hat(u), hat(_reaction(case["reaction"], prm, u))
        ah = Q * uh + phi * fu
        fa = hat(_reaction(case["reaction"], prm, back(ah)))
        fb = hat(_reaction(case["reaction"], prm, back(Q * uh + phi * fa)))
        fc = hat(_reaction(case["reaction"], prm, back(Q * ah + phi * (2 * fb - fu))))
        return back(R * uh + phi1 * fu + phi2 * (fa + fb) + phi3 * fc)

    u = u0.double().reshape((len(rows), 2) + shape)
    if not grad:
        with torch.no_grad():
            for _ in range(case["steps"]):
                u = step(u, alpha, kappa, params)
        return u.reshape(u0.shape)
    start = u.clone().requires_grad_(True)
    u = start
    for _ in range(case["steps"]):
        u = checkpoint(step, u, alpha, kappa, params, use_reentrant=False)
    u.backward(g.double().reshape(u.shape))
    return {"u": u.detach().reshape(u0.shape), "grad_u0": start.grad.reshape(u0.shape),
            "grad_kappa": kappa.grad.reshape(-1).cpu(), "grad_alpha": alpha.grad.reshape(-1).cpu(),
            "grad_params": params.grad.reshape(-1).cpu()}
