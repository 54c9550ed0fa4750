"""The workloads that the speed of this library is judged by.

`listed()` names them, `draw(rng)` gives more of the same ranges; a case is a
dict of plain values:

  path     "flow" (one component), "two_phase" (phase field and capillary
           force) or "adjoint" (gradient through a run)
  nx, ny, nz, lattice, storage, tau, steps
  walls    halfway bounce-back at both ends of y (else periodic)
  force    "none", "uniform" or "field" (per site)
  contrast (two_phase) densities 0.5 / 1.5 and relaxation times 0.65 / 1.7
  every, m0_grad (adjoint) checkpoint interval; gradient of the initial state

A pass of "flow" and "two_phase" advances `steps` steps from where the last
pass left the state and reads the state out, as a program does that writes a
snapshot or a statistic every so many steps; a pass of "adjoint" is a whole
forward run and its gradient.
"""
import math

import torch

DEVICE = "cuda"
SIGMA, WIDTH, DIFFUSIVITY = 0.03, 4.0, 0.1      # droplet workload
RHO, TAU = (0.5, 1.5), (0.65, 1.7)              # layered-channel phases
GRAVITY = (1e-6, 0.0, 0.0)
WORD = {"f64": 8, "f32": 4, "f16s": 2, "bf16s": 2, "f16su": 2}


def _case(name, path, shape, lattice, storage, steps, tau=0.6, walls=False, force="none", **more):
    nx, ny, nz = shape
    case = {"path": path, "nx": nx, "ny": ny, "nz": nz, "lattice": lattice, "storage": storage,
            "steps": steps, "tau": tau, "walls": walls, "force": force}
    case.update(more)
    if name:
        case["name"] = name
    return case


def listed():
    return [
        # the validation vortex's grid and precision: a call of many tiny steps
        _case("vortex_32_f64", "flow", (32, 32, 32), 19, "f64", 50, tau=0.8),
        # a small box, as in a parameter study: steps of a few microseconds
        _case("box_64_f32", "flow", (64, 64, 64), 19, "f32", 50),
        # the layered channel of two phases in its own size, the smallest grid there is in use
        _case("layered_8x128x8_f32", "two_phase", (8, 128, 8), 19, "f32", 50, tau=0.65, walls=True,
              force="uniform", contrast=True),
        # a grid cut to a measured geometry (odd in every direction), with a
        # per-site force, on the larger velocity set
        _case("odd_201x97x113_27_f32", "flow", (201, 97, 113), 27, "f32", 20, force="field"),
        # the channel run: walls and a uniform force
        _case("channel_256_f32", "flow", (256, 256, 256), 19, "f32", 20, tau=0.9, walls=True,
              force="uniform"),
        # the largest runs: single precision, and 16-bit storage
        _case("flow_512_f32", "flow", (512, 512, 512), 19, "f32", 10),
        _case("flow_512_f16s", "flow", (512, 512, 512), 19, "f16s", 10),
        # 16-bit storage that keeps the velocity's precision, a size that is no power of two
        _case("flow_300_f16su", "flow", (300, 300, 300), 19, "f16su", 20),
        # double precision in three dimensions
        _case("flow_250_f64", "flow", (250, 250, 250), 19, "f64", 10),
        # the high-order set
        _case("flow_256_27h_f32", "flow", (256, 256, 256), "27h", "f32", 10),
        # optimisation: force gradient of a run, checkpoints and recomputation
        _case("adjoint_192_f32", "adjoint", (192, 192, 192), 19, "f32", 40, tau=0.8, force="field",
              every=10, m0_grad=False),
        # the droplet run, equal densities
        _case("droplet_256_f32", "two_phase", (256, 256, 256), 19, "f32", 20, tau=1.0,
              contrast=False),
    ]


def _extent(rng, lo, hi):
    n = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    kind = rng.random()
    if kind < 0.35:
        return n | 1                              # odd
    if kind < 0.7:
        return max(8, (n + 4) // 8 * 8)           # multiple of 8
    return n


def draw(rng):
    path = rng.choices(["flow", "two_phase", "adjoint"], [0.6, 0.25, 0.15])[0]
    hi = 320 if path == "flow" else 224
    nx, ny, nz = (_extent(rng, 8, hi) for _ in range(3))
    nx = max(nx, rng.choice([8, 32, 32, 64]))
    walls = rng.random() < 0.3
    if path == "two_phase":
        storage = rng.choices(["f32", "f64", "f16s"], [0.7, 0.2, 0.1])[0]
        contrast = rng.random() < 0.5
        return _case(None, path, (nx, ny, nz), rng.choice([19, 19, 27]), storage,
                     rng.randint(5, 20), tau=TAU[0] if contrast else 1.0, walls=walls,
                     force="uniform" if contrast else "none", contrast=contrast)
    if path == "adjoint":
        return _case(None, path, (nx, ny, nz), rng.choice([19, 19, 27]),
                     rng.choice(["f32", "f32", "f64"]), rng.randint(6, 24), tau=0.8, walls=walls,
                     force="field", every=rng.choice([1, 4, 10]), m0_grad=rng.random() < 0.5)
    lattice = rng.choices([19, 27, "27h"], [0.6, 0.25, 0.15])[0]
    storage = rng.choices(["f32", "f64", "f16s", "bf16s", "f16su"], [0.45, 0.2, 0.15, 0.05, 0.15])[0]
    force = rng.choices(["none", "uniform", "field"], [0.6, 0.2, 0.2])[0]
    return _case(None, path, (nx, ny, nz), lattice, storage, rng.randint(5, 40),
                 tau=round(rng.uniform(0.55, 1.2), 3), walls=walls, force=force)


# -- inputs ----------------------------------------------------------------------

def _axes(case):
    n = (case["nx"], case["ny"], case["nz"])
    return [torch.arange(n[a], dtype=torch.float64, device=DEVICE).view([-1 if d == 2 - a else 1
                                                                         for d in range(3)])
            for a in range(3)]


def _dtype(case):
    return torch.float64 if case["storage"] == "f64" else torch.float32


def _generator(seed):
    return torch.Generator(device=DEVICE).manual_seed(seed)


def _flow_state(case, seed):
    """[10, nz, ny, nx]: a divergence-free flow of random Fourier modes, rms
    0.02 (between walls it is weak), with a2 = u u and p* = 0."""
    g = torch.Generator().manual_seed(seed)
    x = _axes(case)
    n = (case["nx"], case["ny"], case["nz"])
    shape = (case["nz"], case["ny"], case["nx"])
    u = torch.zeros((3,) + shape, dtype=torch.float64, device=DEVICE)
    modes, amp = 6, (0.004 if case["walls"] else 0.02)
    for _ in range(modes):
        k = [int(torch.randint(-3, 4, (1,), generator=g)) for _ in range(3)]
        if k == [0, 0, 0]:
            k = [1, 2, -1]
        q = torch.tensor([2.0 * math.pi * k[a] / n[a] for a in range(3)], dtype=torch.float64)
        a = torch.randn(3, dtype=torch.float64, generator=g)
        a = a - q * (a @ q) / (q @ q)
        a = a / a.norm() * amp * math.sqrt(2.0 / modes)
        phase = float(torch.rand(1, generator=g)) * 2.0 * math.pi
        wave = torch.cos(float(q[0]) * x[0] + float(q[1]) * x[1] + float(q[2]) * x[2] + phase)
        for c in range(3):
            u[c].add_(wave, alpha=float(a[c]))
        del wave
    m = torch.empty((10,) + shape, dtype=_dtype(case), device=DEVICE)
    m[0] = 0.0
    for c in range(3):
        m[1 + c] = u[c]
    for k, (a, b) in enumerate(_PAIRS):
        m[4 + k] = u[a] * u[b]
    return m


def _force_field(case, seed):
    return 1e-6 * torch.randn((3, case["nz"], case["ny"], case["nx"]), generator=_generator(seed),
                              dtype=_dtype(case), device=DEVICE)


def _phase_field(case, seed):
    """Two layers (between walls) or a droplet, a little off a random place."""
    g = torch.Generator().manual_seed(seed + 1)
    x, y, z = _axes(case)
    n = (case["nx"], case["ny"], case["nz"])
    d = [float(v) for v in torch.rand(3, generator=g) - 0.5]
    if case["walls"]:
        dist = (y - (n[1] / 2.0 + d[1])) + 0.0 * (x + z)
    else:
        r = torch.sqrt(sum(torch.minimum((v - c).abs(), e - (v - c).abs()) ** 2
                           for v, c, e in zip((x, y, z), (n[a] / 2.0 + d[a] for a in range(3)), n)))
        dist = max(4.0, 40.0 * min(n) / 256.0) - r
    return (0.5 * (1.0 + torch.tanh(2.0 * dist / WIDTH))).to(_dtype(case)).contiguous()


def _uniform(case):
    return GRAVITY if case["force"] == "uniform" else (0.0, 0.0, 0.0)


def prepare(case, seed):
    from paper_2609_09160_amd import Solver
    shape = (case["nx"], case["ny"], case["nz"])
    s = Solver(shape, case["tau"], lattice=case["lattice"], storage=case["storage"],
               bc=(0, 1 if case["walls"] else 0, 0), force=_uniform(case))
    m0 = _flow_state(case, seed)
    state = {"case": case, "solver": s}
    if case["path"] == "adjoint":
        state["F"] = _force_field(case, seed).requires_grad_()
        state["m0"] = m0.requires_grad_(case["m0_grad"])
        state["dJ"] = torch.randn(m0.shape, generator=_generator(seed + 2), dtype=m0.dtype,
                                  device=DEVICE)
        return state
    s.set_moments(m0)
    if case["path"] == "two_phase":
        if case["contrast"]:
            s.enable_two_phase(SIGMA, WIDTH, DIFFUSIVITY, rho=RHO, tau=TAU)
        else:
            s.enable_two_phase(SIGMA, WIDTH, DIFFUSIVITY)
        s.set_phase(_phase_field(case, seed))
    elif case["force"] == "field":
        s.set_force_field(_force_field(case, seed))
    state["out"] = m0  # read back into the same array
    return state


def run(state):
    case, s = state["case"], state["solver"]
    if case["path"] == "adjoint":
        from paper_2609_09160_amd.adjoint import simulate
        F, m0 = state["F"], state["m0"]
        mT = simulate(F, m0, case["tau"], case["steps"], every=case["every"], solver=s)
        wanted = [F, m0] if case["m0_grad"] else [F]
        return [mT.detach()] + list(torch.autograd.grad(mT, wanted, state["dJ"]))
    s.step(case["steps"])
    m = s.moments(out=state["out"])
    if case["path"] == "two_phase":
        return [m, s.phase(dtype=m.dtype)]
    return [m]


def work(case):
    """Bytes: every state read once and written once per step (and the forces
    and phase fields that go with it), and the read-out; operations: source,
    pull and projection of each site, about 8 per direction."""
    sites = case["nx"] * case["ny"] * case["nz"]
    w = WORD[case["storage"]]
    c = 8 if case["storage"] == "f64" else 4
    planes = 13 if case["storage"] == "f16su" else 10
    q = 19 if case["lattice"] == 19 else 27
    field = 3 * c if case["force"] == "field" else 0
    step = 2 * planes * w + field
    flops = q * (24 if case["lattice"] == "27h" else 8)
    read = planes * w + 10 * c                        # state in, user array out
    if case["path"] == "two_phase":
        # phase update: phi, u in, phi out; flow: also F in and out, phi in
        step += 2 * c + 3 * w + 7 * c + (c if case["contrast"] else 0)
        return {"bytes": sites * (case["steps"] * step + read + 2 * c),
                "flops": sites * case["steps"] * (flops + 150)}
    if case["path"] == "adjoint":
        # forward; recomputation of all but the stored ends; adjoint sweep:
        # lambda in and out, F, u(t), u(t + 1), dJ/dF in and out; checkpoints
        n, k = case["steps"], case["every"]
        segments = -(-n // k)
        sweep = n * (20 + 3 + 6 + 6) * c
        copies = segments * 20 * c if k > 1 else 20 * c
        return {"bytes": sites * ((2 * n - segments + 1) * step + sweep + copies + 3 * read),
                "flops": sites * flops * (3 * n - segments + 1)}
    return {"bytes": sites * (case["steps"] * step + read), "flops": sites * case["steps"] * flops}


# -- the same in plain torch, 64 bits ----------------------------------------------

_PAIRS = ((0, 0), (1, 1), (2, 2), (0, 1), (0, 2), (1, 2))


def _velocities(lattice):
    got = []
    for cz in (-1, 0, 1):
        for cy in (-1, 0, 1):
            for cx in (-1, 0, 1):
                n = abs(cx) + abs(cy) + abs(cz)
                if lattice == 19:
                    if n < 3:
                        got.append(((cx, cy, cz), (1 / 3, 1 / 18, 1 / 36)[n]))
                else:
                    got.append(((cx, cy, cz), (8 / 27, 2 / 27, 1 / 54, 1 / 216)[n]))
    return got


def _second_order(m, F, om1):
    """Post-collision coefficients p*, u + F/2 and the six of second order."""
    u = m[1:4]
    P2 = [u[a] * u[b] + om1 * (m[4 + k] - u[a] * u[b]) + 0.5 * (u[a] * F[b] + u[b] * F[a])
          for k, (a, b) in enumerate(_PAIRS)]
    p0 = m[0] - 1.5 * (P2[0] + P2[1] + P2[2])
    p1 = [u[a] + 0.5 * F[a] for a in range(3)]

    def population(c, w, rows):
        f = p0[:, rows].clone()
        for a in range(3):
            if c[a]:
                f = f + (3.0 * c[a]) * p1[a][:, rows]
        for k, (a, b) in enumerate(_PAIRS):
            if c[a] * c[b]:
                f = f + (4.5 if a == b else 9.0) * (c[a] * c[b]) * P2[k][:, rows]
        return w * f
    return population


def _full_basis(m, F, om1):
    """The complete D3Q27 basis: a product of one-dimensional equilibria, and
    its second derivatives contracted with the relaxed part."""
    u = m[1:4]

    def g(c, v):
        return 2 / 3 - v * v if c == 0 else 1 / 6 + 0.5 * c * v + 0.5 * v * v

    def dg(c, v):
        return -2.0 * v if c == 0 else 0.5 * c + v

    def population(c, w, rows):
        v = [u[a][:, rows] for a in range(3)]
        G = [g(c[a], v[a]) for a in range(3)]
        d = [dg(c[a], v[a]) for a in range(3)]
        dd = [-2.0 if c[a] == 0 else 1.0 for a in range(3)]
        f = w * (m[0][:, rows] - 1.0) + G[0] * G[1] * G[2]
        for k, (a, b) in enumerate(_PAIRS):
            B = om1 * (m[4 + k][:, rows] - v[a] * v[b])
            o = 3 - a - b
            if a == b:
                e, h = [q for q in range(3) if q != a]
                f = f + 0.5 * B * dd[a] * G[e] * G[h]
            else:
                f = f + B * d[a] * d[b] * G[o]
        cu = sum(c[a] * v[a] for a in range(3))
        cF = sum(c[a] * F[a][:, rows] for a in range(3))
        uF = sum(v[a] * F[a][:, rows] for a in range(3))
        return f + 0.5 * w * (3.0 * cF - 3.0 * uF + 9.0 * cu * cF)
    return population


def _exact_step(m, lattice, omega, walls, F, F_next):
    """One step: pull the populations, project them, correct with F_next."""
    om1 = 1.0 - omega
    pop = _full_basis(m, F, om1) if lattice == "27h" else _second_order(m, F, om1)
    whole = slice(None)
    s0, s1, s2 = 0.0, [0.0] * 3, [0.0] * 6
    for c, w in _velocities(lattice):
        f = torch.roll(pop(c, w, whole), (c[2], c[1], c[0]), (0, 1, 2))
        if walls and c[1]:
            row = slice(0, 1) if c[1] == 1 else slice(-1, None)
            back = pop(tuple(-v for v in c), w, row)
            f = torch.cat([back, f[:, 1:]] if c[1] == 1 else [f[:, :-1], back], 1)
        s0 = s0 + f
        for a in range(3):
            if c[a]:
                s1[a] = s1[a] + c[a] * f
        for k, (a, b) in enumerate(_PAIRS):
            h = c[a] * c[b] - (1 / 3 if a == b else 0.0)
            if h:
                s2[k] = s2[k] + h * f
    u = [s1[a] + 0.5 * F_next[a] for a in range(3)]
    a2 = [s2[k] + 0.5 * (F_next[a] * u[b] + F_next[b] * u[a]) for k, (a, b) in enumerate(_PAIRS)]
    return torch.stack([s0] + u + a2)


def _neighbour(v, c, walls, sign=1.0):
    """v(x + c); beyond a wall the mirror row, times sign."""
    if walls and c[1]:
        ghost = sign * (v[:, -1:] if c[1] == 1 else v[:, :1])
        v = torch.cat([v[:, 1:], ghost] if c[1] == 1 else [ghost, v[:, :-1]], 1)
        return torch.roll(v, (-c[2], -c[0]), (0, 2))
    return torch.roll(v, (-c[2], -c[1], -c[0]), (0, 1, 2))


def _gradient(v, walls):
    g, lap = [0.0] * 3, 0.0
    for c, w in _velocities(27):
        if c == (0, 0, 0):
            continue
        n = _neighbour(v, c, walls)
        lap = lap + 6.0 * w * (n - v)
        for a in range(3):
            if c[a]:
                g[a] = g[a] + 3.0 * w * c[a] * n
    return g, lap


def _phase_update(phi, u, walls):
    g, lap = _gradient(phi, walls)
    norm = torch.sqrt(sum(v * v for v in g)) + 1e-12
    lam = 4.0 * DIFFUSIVITY / WIDTH
    V = [phi * u[a] + lam * phi * (1.0 - phi) * g[a] / norm for a in range(3)]
    div = 0.0
    for c, w in _velocities(27):
        for a in range(3):
            if c[a]:
                div = div + 3.0 * w * c[a] * _neighbour(V[a], c, walls, -1.0 if a == 1 else 1.0)
    return phi - div + DIFFUSIVITY * lap


def _blend(pair, phi):
    return pair[0] + phi * (pair[1] - pair[0])


def _capillary(phi, m, rho, tau, gravity, walls):
    g, lap = _gradient(phi, walls)
    beta, kappa = 12.0 * SIGMA / WIDTH, 1.5 * SIGMA * WIDTH
    mu = 4.0 * beta * phi * (phi - 1.0) * (phi - 0.5) - kappa * lap
    r = _blend(rho, phi)
    F = [mu * g[a] + r * gravity[a] for a in range(3)]
    if rho[0] != rho[1]:
        nu = _blend([(t - 0.5) / 3.0 for t in tau], phi)
        cv = 3.0 * nu / (3.0 * nu + 0.5)
        gr = [(rho[1] - rho[0]) * v for v in g]
        for a in range(3):
            F[a] = F[a] - m[0] / 3.0 * gr[a]
        for k, (a, b) in enumerate(_PAIRS):
            neq = cv * (m[4 + k] - m[1 + a] * m[1 + b])
            F[a] = F[a] - neq * gr[b]
            if a != b:
                F[b] = F[b] - neq * gr[a]
    return F


def _exact_two_phase(case, seed):
    m = _flow_state(case, seed).double()
    phi = _phase_field(case, seed).double()
    walls, gravity = case["walls"], _uniform(case)
    rho, tau = (RHO, TAU) if case["contrast"] else ((1.0, 1.0), (case["tau"],) * 2)
    nu = [(t - 0.5) / 3.0 for t in tau]
    F = _capillary(phi, m, rho, tau, gravity, walls)
    for _ in range(case["steps"]):
        after = _phase_update(phi, m[1:4], walls)
        F_next = _capillary(after, m, rho, tau, gravity, walls)
        omega = 1.0 / (3.0 * _blend(nu, phi) + 0.5)
        r, r_next = _blend(rho, phi), _blend(rho, after)
        m = _exact_step(m, case["lattice"], omega, walls, [v / r for v in F],
                        [v / r_next for v in F_next])
        phi, F = after, F_next
    return [m, phi]


def exact(case, seed):
    if case["path"] == "two_phase":
        return _exact_two_phase(case, seed)
    m = _flow_state(case, seed).double()
    omega = 1.0 / case["tau"]
    if case["path"] == "adjoint":
        from torch.utils.checkpoint import checkpoint
        F = _force_field(case, seed).double().requires_grad_()
        m0 = m.requires_grad_(case["m0_grad"])
        m = m0
        for _ in range(case["steps"]):
            m = checkpoint(_exact_step, m, case["lattice"], omega, case["walls"], F, F,
                           use_reentrant=False)
        dJ = torch.randn(m.shape, generator=_generator(seed + 2), dtype=_dtype(case),
                         device=DEVICE).double()
        wanted = [F, m0] if case["m0_grad"] else [F]
        return [m.detach()] + list(torch.autograd.grad(m, wanted, dJ))
    shape = m.shape[1:]
    if case["force"] == "field":
        F = _force_field(case, seed).double()
    else:
        F = torch.tensor(_uniform(case), dtype=torch.float64, device=DEVICE).view(3, 1, 1, 1)
        F = F.expand((3,) + shape)
    for _ in range(case["steps"]):
        m = _exact_step(m, case["lattice"], omega, case["walls"], F, F)
    return [m]
