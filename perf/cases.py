"""The work that a user of this library has it do, as cases that can be timed.

Every case is one call, or one forward and backward, or one time step, through
the Python entry points (`forces`, `TreeForces`, `leapfrog_step`) on particles
drawn from a seed on the GPU.  Sizes, opening angles and softenings are those
of the workloads, tests and benchmark of this repository, or lie between them:
tens of thousands of particles while a set-up is being tried out, 1e5..1e6 in
a simulation's steps, 2^18 in a fit, 1e7 in the headline evaluation.
"""
import math

import torch

import paper_2412_01733_amd as tc

_DT = {"f32": torch.float32, "f64": torch.float64}
_WALK_DT = {"f32c": torch.float32, "f64": torch.float64}


def listed():
    return [
        # trying a set-up out, or a small cluster: the call's latency
        dict(name="forces-f32c-1000", kind="forces", dist="plummer", n=1000, dtype="f32", walk="f32c", theta=0.7, eps=0.01),
        # the size that the accuracy of a set-up is checked at, in double precision throughout
        dict(name="forces-f64-4096", kind="forces", dist="plummer", n=4096, dtype="f64", walk="f64", theta=0.7, eps=0.01),
        # double-precision particles, compensated FP32 walk: the evaluation's smallest workload
        dict(name="forces-f32c-16384", kind="forces", dist="plummer", n=16384, dtype="f64", walk="f32c", theta=0.7, eps=0.01),
        # theta = 0: the direct sum that approximations are compared with; an odd size
        dict(name="direct-f32c-12345", kind="forces", dist="plummer", n=12345, dtype="f32", walk="f32c", theta=0.0, eps=0.01),
        # a differentiable force in double precision, as in a gradient check or a small fit
        dict(name="grad-f64-20000", kind="grad", dist="lognormal", n=20000, dtype="f64", walk="f64", theta=0.6, eps=0.01),
        # a time step of a disc galaxy in double precision
        dict(name="kdk-f64-100000", kind="kdk", dist="disc", n=100000, dtype="f64", walk="f64", theta=0.5, eps=0.02),
        # the fitting workload: forward and backward, masses of every size, 2^18 particles
        dict(name="grad-f32c-262144", kind="grad", dist="lognormal", n=262144, dtype="f32", walk="f32c", theta=0.5, eps=0.01),
        # the simulation workload: one kick-drift-kick step of a disc and halo
        dict(name="kdk-f32c-1000000", kind="kdk", dist="disc", n=1000000, dtype="f32", walk="f32c", theta=0.5, eps=0.02),
        # the same set at the paper's own opening angle: a short walk, the tree counts; an odd size
        dict(name="forces-f32c-999999-theta1", kind="forces", dist="disc", n=999999, dtype="f32", walk="f32c", theta=1.0, eps=0.02),
        # the headline evaluation, in both precisions
        dict(name="forces-f32c-10000000", kind="forces", dist="plummer", n=10000000, dtype="f32", walk="f32c", theta=0.5, eps=0.005),
        dict(name="forces-f64-10000000", kind="forces", dist="plummer", n=10000000, dtype="f32", walk="f64", theta=0.5, eps=0.005),
        # forward and backward at the headline size
        dict(name="grad-f32c-10000000", kind="grad", dist="lognormal", n=10000000, dtype="f32", walk="f32c", theta=0.5, eps=0.005),
    ]


def _interactions(case):
    """Interactions of one evaluation: n (n - 1) for the direct sum; otherwise the
    count per target that the walk reports for Plummer spheres, 2030 at 1e7 and
    theta = 0.5, growing by 85 for each doubling of n, and as theta^-2.55 between
    theta = 0.3 and 0.8."""
    n, th = case["n"], case["theta"]
    per = n - 1.0
    if th > 0:
        per = min(per, (2030.0 + 85.0 * math.log2(n / 1e7)) * (0.5 / th) ** 2.55)
    return n * per


def _cost(case):
    return _interactions(case) * {"forces": 1.0, "kdk": 1.0, "grad": 3.0}[case["kind"]] * (1.9 if case["walk"] == "f64" else 1.0)


def draw(rng):
    most = max(_cost(c) for c in listed())
    while True:
        kind = rng.choice(["forces", "forces", "kdk", "grad"])
        walk = rng.choice(["f32c", "f32c", "f64"])
        n = int(round(10 ** rng.uniform(math.log10(500.0), 7.0)))
        theta = rng.choice([0.3, 0.5, 0.6, 0.7, 0.8, 1.0])
        if kind == "forces" and rng.random() < 0.1:
            n, theta = int(round(10 ** rng.uniform(math.log10(500.0), math.log10(20000.0)))), 0.0
        case = dict(kind=kind, dist={"kdk": "disc", "grad": "lognormal"}.get(kind) or rng.choice(["plummer", "disc"]), n=n,
                    dtype="f64" if walk == "f64" else rng.choice(["f32", "f32", "f64"]), walk=walk, theta=theta,
                    eps=rng.choice([0.005, 0.01, 0.02, 0.05]))
        if _cost(case) <= most:
            return case


def work(case):
    """Positions and masses read once, accelerations and potentials written once
    (and velocities read and written by a step; upstream gradients read and
    gradients written by a backward pass); 20 operations an interaction, 40 more
    for its derivative."""
    n, b, w = case["n"], _DT[case["dtype"]].itemsize, _WALK_DT[case["walk"]].itemsize
    by, fl = n * 4 * (b + w), 20.0
    if case["kind"] == "kdk":
        by += n * (9 * b + 3 * w)
    elif case["kind"] == "grad":
        by += n * 4 * (w + b)
        fl += 40.0
    return {"bytes": float(by), "flops": fl * _interactions(case)}


# -- inputs ----------------------------------------------------------------------


def _isotropic(r, u, v):
    ct = 2 * u - 1
    st = (1 - ct * ct).clamp_min(0).sqrt()
    return torch.stack([r * st * torch.cos(2 * math.pi * v), r * st * torch.sin(2 * math.pi * v), r * ct], 1)


def _plummer(n, rand):
    u = rand(n, 3)
    ft = 1000.0 / 101.0 ** 1.5  # the sphere ends at r = 10
    r = ((u[:, 0] * ft).clamp_min(1e-30) ** (-2.0 / 3.0) - 1).rsqrt()
    return _isotropic(r, u[:, 1], u[:, 2])


def _disc(n, rand, randn):
    """An exponential disc (four fifths of the particles, mass 1) in a Hernquist halo (mass 4), rotating."""
    nd = n * 4 // 5
    u = rand(nd, 3)
    f = u[:, 0] * (1 - 11.0 * math.exp(-10.0))
    R = torch.full_like(f, 1.5)
    for _ in range(60):
        R = (R - (1 - (1 + R) * torch.exp(-R) - f) / (R * torch.exp(-R)).clamp_min(1e-300)).clamp(1e-12, 10.0)
    z = 0.1 * torch.atanh((2 * u[:, 1] - 1) * math.tanh(10.0))
    ph = 2 * math.pi * u[:, 2]
    xd = torch.stack([R * torch.cos(ph), R * torch.sin(ph), z], 1)
    c = (100.0 / 105.0) ** 2
    w = rand(n - nd, 3)
    s = (w[:, 0] * c).sqrt()
    rh = 5.0 * s / (1 - s)
    xh = _isotropic(rh, w[:, 1], w[:, 2])

    def inside(r):
        return 1 - (1 + r) * torch.exp(-r) + 4.0 * r * r / (r + 5.0) ** 2 / c

    vc = (inside(R) / R).sqrt()
    g = randn(nd, 3) * vc[:, None]
    vr, vt = 0.1 * g[:, 0], vc + 0.1 * g[:, 1]
    vd = torch.stack([vr * torch.cos(ph) - vt * torch.sin(ph), vr * torch.sin(ph) + vt * torch.cos(ph), 0.05 * g[:, 2]], 1)
    vh = randn(n - nd, 3) * (inside(rh) / (3 * rh.clamp_min(1e-12))).sqrt()[:, None]
    m = torch.cat([torch.full_like(R, 1.0 / nd), torch.full_like(rh, 4.0 / (n - nd))])
    return torch.cat([xd, xh]), torch.cat([vd, vh]), m


def _inputs(case, seed):
    """Positions, velocities (a step only), masses, and upstream gradients of acc and pot (a backward pass only)."""
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev).manual_seed(int(seed))
    f8 = torch.float64

    def rand(*s):
        return torch.rand(*s, generator=gen, device=dev, dtype=f8)

    def randn(*s):
        return torch.randn(*s, generator=gen, device=dev, dtype=f8)

    n, dt, wd = case["n"], _DT[case["dtype"]], _WALK_DT[case["walk"]]
    vel = None
    if case["dist"] == "disc":
        pos, vel, mass = _disc(n, rand, randn)
    else:
        pos = _plummer(n, rand)
        mass = torch.full((n,), 1.0 / n, device=dev, dtype=f8)
        if case["dist"] == "lognormal":
            mass = mass * torch.exp(0.2 * randn(n) - 0.02)
    up = (randn(n, 3).to(wd), randn(n).to(wd)) if case["kind"] == "grad" else (None, None)
    return pos.to(dt), vel.to(dt) if case["kind"] == "kdk" else None, mass.to(dt), up


_TAU = 1e-3


def prepare(case, seed):
    pos, vel, mass, up = _inputs(case, seed)
    s = dict(case=case, pos=pos, mass=mass)
    if case["kind"] == "grad":
        pos.requires_grad_(True)
        mass.requires_grad_(True)
        s["up"] = up
    else:
        s["tree"] = tc.Tree()  # a program that calls again keeps the handle
    if case["kind"] == "kdk":  # a step starts from the last one's accelerations
        acc, pot, _ = tc.forces(pos, mass, case["theta"], case["eps"], walk=case["walk"], tree=s["tree"])
        s.update(vel=vel, acc=acc, pot=pot)
    return s


def run(state):
    c = state["case"]
    if c["kind"] == "forces":
        acc, pot, _ = tc.forces(state["pos"], state["mass"], c["theta"], c["eps"], walk=c["walk"], tree=state["tree"])
        return acc, pot
    if c["kind"] == "kdk":
        tc.leapfrog_step(state["pos"], state["vel"], state["mass"], state["acc"], _TAU, c["theta"], c["eps"], walk=c["walk"],
                         pot=state["pot"], tree=state["tree"])
        return state["pos"], state["vel"], state["acc"], state["pot"]
    acc, pot = tc.TreeForces.apply(state["pos"], state["mass"], c["theta"], c["eps"], 1.0, c["walk"])
    gpos, gmass = torch.autograd.grad((acc, pot), (state["pos"], state["mass"]), state["up"])
    return acc.detach(), pot.detach(), gpos, gmass


# -- the same in 64 bits, in plain torch ----------------------------------------------


class _Octree:
    """The octree's cells level by level, as arrays: cells of particles that share 3 l leading key bits."""

    def __init__(self, pos, mass):
        n, dev = pos.shape[0], pos.device
        lo = pos.amin(0)
        ext = float((pos.amax(0) - lo).max())
        f, e = math.frexp(ext)
        self.L = 2.0 ** (e - 1 if f == 0.5 else e) if ext > 0 else 1.0
        q = torch.floor((pos - lo) * (2.0 ** 21 / self.L)).clamp(0, 2 ** 21 - 1).long()
        key = torch.zeros(n, dtype=torch.long, device=dev)
        for b in range(21):
            for k in range(3):
                key |= ((q[:, k] >> b) & 1) << (3 * b + 2 - k)
        key, self.perm = torch.sort(key, stable=True)
        self.x, self.m = pos[self.perm], mass[self.perm]
        self.cell, self.start, self.count, self.X, self.M, self.kids = [], [], [], [], [], []
        for lv in range(22):
            _, inv, cnt = torch.unique_consecutive(key >> (3 * (21 - lv)), return_inverse=True, return_counts=True)
            M, *S = (torch.segment_reduce(v, "sum", lengths=cnt, unsafe=True)
                     for v in (self.m, *(self.m * w for w in self.x.unbind(1))))
            S = torch.stack(S, 1)
            self.cell.append(inv)
            self.count.append(cnt)
            self.start.append(cnt.cumsum(0) - cnt)
            self.M.append(M)
            self.X.append(torch.where((cnt == 1)[:, None], self.x[self.start[-1]], S / M[:, None]))
        for lv in range(22):  # first child (at the last level: first particle) of each cell, and how many
            first, end = self.start[lv], self.start[lv] + self.count[lv]
            if lv < 21:
                first, end = (torch.searchsorted(self.start[lv + 1], v) for v in (first, end))
            self.kids.append((first, end - first))

    def terms(self, a, b, theta):
        """For the targets a .. b-1 (sorted positions): tuples (level, target, cell) of accepted cells and (None, target,
        particle) of direct terms, targets ascending in each."""
        t = torch.arange(a, b, device=self.x.device)
        c = torch.zeros_like(t)
        for lv in range(22):
            d2 = ((self.X[lv][c] - self.x[t]) ** 2).sum(1)
            inside = self.cell[lv][t] == c
            one = self.count[lv][c] == 1
            take = ~inside & (one | (self.L * 0.5 ** lv < theta * d2.sqrt()))
            yield lv, t[take], c[take]
            go = ~take & ~one
            t, c = t[go], c[go]
            first, kids = self.kids[lv]
            k = kids[c]
            t = torch.repeat_interleave(t, k)
            c = torch.repeat_interleave(first[c] - (k.cumsum(0) - k), k) + torch.arange(t.shape[0], device=t.device)
            if lv == 21:
                yield None, t[t != c], c[t != c]


def _sums(t, a, b, vals):
    """Sums of each column of vals over the rows of each target (ascending t)."""
    if not t.shape[0]:
        return torch.zeros(b - a, vals.shape[1], dtype=vals.dtype, device=vals.device)
    lens = torch.bincount(t - a, minlength=b - a)
    return torch.stack([torch.segment_reduce(v.contiguous(), "sum", lengths=lens, unsafe=True) for v in vals.unbind(1)], 1)


def _forces64(pos, mass, theta, eps, up=None):
    """(acc, pot[, gpos, gmass]) of Eq.(1) with the opening rule, G = 1, every interaction set held fixed in the gradients."""
    n, dev = pos.shape[0], pos.device
    T = _Octree(pos, mass)
    out = torch.zeros(n, 4, dtype=pos.dtype, device=dev)
    if up is not None:
        ga, gp = up[0].to(pos.dtype)[T.perm], up[1].to(pos.dtype)[T.perm]
        gx, gm = torch.zeros_like(T.x), torch.zeros_like(T.m)
        gX, gM = [torch.zeros_like(X) for X in T.X], [torch.zeros_like(M) for M in T.M]
    chunk = max(256, int(3e7 / max(1.0, _interactions(dict(n=n, theta=theta)) / n)))
    for a in range(0, n, chunk):
        b = min(n, a + chunk)
        for lv, t, c in T.terms(a, b, theta):
            X, M = (T.x, T.m) if lv is None else (T.X[lv], T.M[lv])
            d, M = X[c] - T.x[t], M[c]
            ri = ((d * d).sum(1) + eps * eps).rsqrt()
            w = M * ri ** 3
            out[a:b] += _sums(t, a, b, torch.cat([w[:, None] * d, -(M * ri)[:, None]], 1))
            if up is not None:
                g, h = ga[t], gp[t]
                dg = (d * g).sum(1)
                src = w[:, None] * g + (w * (h - 3 * ri * ri * dg))[:, None] * d
                gx[a:b] -= _sums(t, a, b, src)
                o = torch.argsort(c)
                g = _sums(c[o], 0, X.shape[0], torch.cat([src, (dg * ri ** 3 - h * ri)[:, None]], 1)[o])
                if lv is None:
                    gx, gm = gx + g[:, :3], gm + g[:, 3]
                else:
                    gX[lv] += g[:, :3]
                    gM[lv] += g[:, 3]
    res = torch.empty_like(out)
    res[T.perm] = out
    ans = [res[:, :3].contiguous(), res[:, 3].contiguous()]
    if up is not None:
        for lv in range(22):
            u = (gX[lv] / T.M[lv][:, None])[T.cell[lv]]
            gx += T.m[:, None] * u
            gm += gM[lv][T.cell[lv]] + (u * (T.x - T.X[lv][T.cell[lv]])).sum(1)
        for g in (gx, gm):
            r = torch.empty_like(g)
            r[T.perm] = g
            ans.append(r)
    return ans


def exact(case, seed):
    if _cost(case) > 3e9:
        return None
    pos, vel, mass, up = _inputs(case, seed)
    dt, wd = pos.dtype, _WALK_DT[case["walk"]]
    f8 = torch.float64
    th, eps = case["theta"], case["eps"]
    if case["kind"] != "kdk":
        return tuple(_forces64(pos.to(f8), mass.to(f8), th, eps, up if case["kind"] == "grad" else None))
    # positions and velocities are stored in their own type between the operations
    acc = _forces64(pos.to(f8), mass.to(f8), th, eps)[0].to(wd).to(f8)
    v = (vel.to(f8) + 0.5 * _TAU * acc).to(dt).to(f8)
    x = (pos.to(f8) + _TAU * v).to(dt).to(f8)
    acc, pot = _forces64(x, mass.to(f8), th, eps)
    return x, v + 0.5 * _TAU * acc, acc, pot
