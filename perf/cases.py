"""Workloads of the hydro step whose speed is watched, with a plain 64-bit evaluation of each.

A case is a level (a domain cut into boxes), a flow and the way a program
advances it.  Kinds:
  step     an eager time loop: ghost fill, one step, the next dt left on the
           device by the update
  graph    whole steps [fill, step] replayed from a HIP graph
  jet      the inflowing jet of a planar slab (an inflow face, outflow
           elsewhere), its steps replayed from a HIP graph
  grad     one step and its vector-Jacobian product through autograd
  rollout  a checkpointed differentiable roll-out and its gradient
  species  a step with passive species
  amr      one coarse step of a two-level hierarchy (one coarse and two fine
           steps, flux register, reflux, average down)

`exact` evaluates the same thing in float64 with whole-array torch
expressions of the method's definition (PPM with the Colella-Woodward
limiter and flattening, characteristic tracing, the two-shock solver, the
12-solve corner-transport-upwind scheme), gradients by torch's autograd.
"""
import math
import random

import torch

from paper_1008_2801_amd import inputs as I
from paper_1008_2801_amd import ppm as P

NG = 4
PERIODIC, OUTFLOW, REFLECT, INFLOW = 0, 1, 2, 4
BCS = {"periodic": (PERIODIC,) * 6, "outflow": (OUTFLOW,) * 6,
       "walls": (PERIODIC,) * 4 + (REFLECT,) * 2}
# algorithmic operations of one zone update (add, mul, div, sqrt once each)
FLOPS_ZONE = 4300.0


# ------------------------------------------------------------------ cases --
def listed():
    return [
        # the smallest loops: what a step costs when only its launches count
        dict(name="step 16^3", kind="step", nx=16, ny=16, nz=16, box=16, bc="periodic", flow="smooth", prec=0),
        dict(name="graph 32^3 x10", kind="graph", nx=32, ny=32, nz=32, box=32, bc="periodic", flow="smooth", prec=0,
             steps=10),
        # a planar problem: many short steps of a thin slab
        dict(name="jet 256x256x4 x10", kind="jet", n=256, nz=4, prec=0, steps=10),
        # a small level of several boxes with walls and gravity
        dict(name="rt 8 boxes of 64^3", kind="step", nx=128, ny=128, nz=128, box=64, bc="walls", flow="rt", prec=0),
        # one large box, in both precisions
        dict(name="step 256^3", kind="step", nx=256, ny=256, nz=256, box=256, bc="periodic", flow="jump", prec=0),
        dict(name="step 256^3 fp32", kind="step", nx=256, ny=256, nz=256, box=256, bc="periodic", flow="jump",
             prec=1),
        # many unequal boxes
        dict(name="tiling 512 boxes", kind="step", nper=8, lseed=3, bc="periodic", flow="smooth", prec=0),
        # the largest: a level of equal boxes with walls and gravity, whole steps in a graph
        dict(name="graph rt 216 boxes x2", kind="graph", nx=384, ny=384, nz=384, box=64, bc="walls", flow="rt",
             prec=0, steps=2),
        # differentiation: one step, and a roll-out with checkpoints
        dict(name="grad 128^3", kind="grad", nx=128, ny=128, nz=128, box=128, bc="periodic", flow="smooth", prec=0),
        dict(name="rollout 64^3 x8", kind="rollout", nx=64, ny=64, nz=64, box=64, bc="periodic", flow="smooth",
             prec=0, steps=8, every=4),
        # passive species
        dict(name="species 128^3 x3", kind="species", nx=128, ny=128, nz=128, box=128, bc="periodic", flow="smooth",
             prec=0, ns=3),
        # two levels, several boxes on each
        dict(name="amr 96^3+96^3", kind="amr", n=96, cbox=48, fbox=48, prec=0),
    ]


def _size(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["step", "step", "step", "graph", "graph", "tiling", "jet", "grad", "rollout", "species",
                       "amr"])
    prec = 1 if rng.random() < 0.3 else 0
    if kind == "jet":
        return dict(kind="jet", n=_size(rng, 48, 400), nz=rng.choice([4, 5, 6]), prec=prec,
                    steps=rng.choice([4, 8, 10]))
    if kind == "amr":
        return dict(kind="amr", n=4 * _size(rng, 6, 32), cbox=_size(rng, 16, 64), fbox=2 * _size(rng, 8, 32), prec=prec)
    if kind == "tiling":
        return dict(kind="step", nper=rng.randrange(2, 8), lseed=rng.randrange(100), bc="periodic", flow="smooth",
                    prec=prec)
    top = {"step": 288, "graph": 256, "grad": 128, "rollout": 80, "species": 128}[kind]
    nx, ny, nz = (_size(rng, 12, top) for _ in range(3))
    box = rng.choice([max(nx, ny, nz), 64, 48, 32])
    bc = rng.choice(["periodic", "walls", "outflow"]) if kind in ("step", "graph") else "periodic"
    flow = "smooth" if kind in ("grad", "rollout") else "rt" if bc == "walls" else rng.choice(["smooth", "jump"])
    c = dict(kind=kind, nx=nx, ny=ny, nz=nz, box=box, bc=bc, flow=flow, prec=prec)
    if kind == "graph":
        c["steps"] = rng.choice([1, 2, 4])
    if kind == "rollout":
        c.update(steps=rng.choice([4, 6, 8]), every=rng.choice([2, 3, 4]))
    if kind == "species":
        c["ns"] = rng.randrange(1, 6)
    return c


# ----------------------------------------------------------------- levels --
def _split(total, size):
    k = -(-total // size)
    return [total // k + (1 if i < total % k else 0) for i in range(k)]


def _layout(case):
    """The level's boxes; its spacing makes the longest edge 1."""
    if "nper" in case:
        lay, _ = I.cfg3_layout(case["lseed"], nper=case["nper"])
        n = [hi + 1 for hi in lay.domain_hi]
    else:
        n = [case["nx"], case["ny"], case["nz"]]
        lay = I.tensor_tiling(*[_split(v, case["box"]) for v in n], bc=BCS[case["bc"]])
    h = 1.0 / max(n)
    return lay, tuple(n), (h, h, h)


def _params(case, cls=None):
    grav = (0.0, 0.0, -1.0) if case.get("flow") == "rt" else (0.0, 0.0, 0.0)
    kw = dict(gamma=5.0 / 3.0 if case.get("flow") == "jump" else 1.4, grav=grav)
    return kw if cls is None else cls(precision=case["prec"], **kw)


def _centres(n, h, dev, lo=(0, 0, 0)):
    x = [(torch.arange(n[d], device=dev, dtype=torch.float64) + lo[d] + 0.5) * h[d] for d in range(3)]
    return x[0][None, None, :], x[1][None, :, None], x[2][:, None, None]


def _modes(r, X, L, count, K):
    """Random-phase mode sum in [-1, 1], periodic over the lengths L."""
    amp = [r.random() for _ in range(count)]
    out = 0.0
    for a in amp:
        while True:
            k = [r.randint(-K, K) for _ in range(3)]
            if 1 <= sum(v * v for v in k) <= K * K:
                break
        ph = r.uniform(0.0, 2.0 * math.pi)
        arg = sum(2.0 * math.pi * k[d] / L[d] * X[d] for d in range(3)) + ph
        out = out + a / sum(amp) * torch.cos(arg)
    return out


def _cons(q, gamma):
    r, u, v, w, p = torch.broadcast_tensors(*[torch.as_tensor(t, dtype=torch.float64) for t in q])
    return torch.stack([r, r * u, r * v, r * w, p / (gamma - 1.0) + 0.5 * r * (u * u + v * v + w * w)])


def _flow(flow, seed, n, h, dev, lo=(0, 0, 0), L=None):
    """Conserved state (5, nz, ny, nx) at the centres of zones lo .. lo + n."""
    r = random.Random(1000003 * seed + 17)
    L = [n[d] * h[d] for d in range(3)] if L is None else L
    X = _centres(n, h, dev, lo)
    zero = torch.zeros((n[2], n[1], n[0]), device=dev, dtype=torch.float64)
    if flow == "rt":  # heavy over light at rest, the interface perturbed, hydrostatic pressure
        delta, mid = 2.0 * h[2], 0.5 * L[2]
        zi = mid + 0.01 * _modes(r, (X[0], X[1], torch.zeros_like(X[2])), L, 8, 8)
        rho = 1.5 + 0.5 * torch.tanh((X[2] - zi) / delta) + zero

        def lc(x):
            return x.abs() + torch.log1p(torch.exp(-2.0 * x.abs())) - math.log(2.0)
        p = 2.5 - (1.5 * X[2] + 0.5 * delta * (lc((X[2] - mid) / delta) - lc(torch.full_like(X[2], mid / delta))))
        return _cons([rho, zero, zero, zero, p + zero], 1.4)
    if flow == "jump":  # a planar jump in x under density modes, constant velocity
        left = X[0] < 0.5 * L[0]
        rho = torch.where(left, 1.0, 0.125).double() * (1.0 + 0.1 * _modes(r, X, L, 8, 8)) + zero
        vel = [r.uniform(-0.5, 0.5) for _ in range(3)]
        p = torch.where(left, 1.0, 0.1).double() + zero
        return _cons([rho] + [v + zero for v in vel] + [p], 5.0 / 3.0)
    s = [_modes(r, X, L, 6, 3) for _ in range(5)]  # smooth, a bulk flow and moderate amplitudes
    vel = [r.uniform(-0.4, 0.4) for _ in range(3)]
    return _cons([1.25 + 0.4 * s[0]] + [vel[d] + 0.3 * s[1 + d] for d in range(3)] + [1.25 + 0.4 * s[4]], 1.4)


def _pack(lay, V, ghosts=None):
    """Arena of a level from its domain's valid zones V (components, nz, ny,
    nx); the boxes' ghost zones are zero, or those of the padded domain
    `ghosts` (components, nz + 8, ny + 8, nx + 8)."""
    parts = []
    for b in range(lay.nbox):
        x, y, z = (int(lay.lo[b][d] - lay.domain_lo[d]) for d in range(3))
        nx, ny, nz = lay.n(b)
        own = V[:, z:z + nz, y:y + ny, x:x + nx]
        if ghosts is None:
            own = torch.nn.functional.pad(own, (NG,) * 6)
        else:
            box = ghosts[:, z:z + nz + 8, y:y + ny + 8, x:x + nx + 8].clone()
            _core(box).copy_(own)
            own = box
        parts.append(own.reshape(-1))
    return torch.cat(parts)


def _cotangent(seed, V):
    g = torch.Generator(device=V.device)
    g.manual_seed(seed + 99)
    return torch.randn(V.shape, generator=g, device=V.device, dtype=torch.float64)


def _fractions(seed, n, h, ns, dev):
    r = random.Random(7919 * seed + 5)
    X, L = _centres(n, h, dev), [n[d] * h[d] for d in range(3)]
    w = [1.0 + 0.8 * _modes(r, X, L, 4, 3) + torch.zeros((n[2], n[1], n[0]), device=dev, dtype=torch.float64)
         for _ in range(ns)]
    tot = 2.0 * sum(w)
    return torch.stack([v / tot for v in w])


def _jet(case, seed):
    """The jet's workload, its inflow speed varied by the seed."""
    wl = I.jet(case["n"], case["nz"])
    f = wl.meta["inflow"][2]
    s = 0.8 + 0.4 * random.Random(seed).random()
    f[4] += 0.5 * f[2] ** 2 / f[0] * (s * s - 1.0)
    f[2] *= s
    return wl, torch.from_numpy(f)


def _hierarchy(case, seed, dev):
    n = case["n"]
    lo, fe = n // 4, 2 * (n // 2)
    cl = I.tensor_tiling(*[_split(n, case["cbox"])] * 3)
    even = [2 * v for v in _split(fe // 2, max(1, case["fbox"] // 2))]
    fl = I.tensor_tiling(even, even, even, bc=(3,) * 6, origin=(2 * lo,) * 3)
    h = 1.0 / n
    Gc = _flow("smooth", seed, (n,) * 3, (h,) * 3, dev, L=(1.0,) * 3)
    Gf = _flow("smooth", seed, (fe,) * 3, (h / 2,) * 3, dev, lo=(2 * lo,) * 3, L=(1.0,) * 3)
    return cl, fl, Gc, Gf, (h, h, h), lo, fe


def prepare(case, seed):
    dev = torch.device("cuda")
    kind = case["kind"]
    if kind == "amr":
        cl, fl, Gc, Gf, dx, _, _ = _hierarchy(case, seed, dev)
        t = P.TwoLevel(cl, fl)
        Uc, Uf = _pack(cl, Gc), _pack(fl, Gf)
        return dict(kind=kind, t=t, a=Uc, b=torch.zeros_like(Uc), f=Uf, ft=torch.zeros_like(Uf), dx=dx,
                    p=_params(case, P.params), dt=torch.zeros(2, dtype=torch.float64, device=dev))
    if kind == "jet":
        wl, face = _jet(case, seed)
        lev = P.Level(wl.layout)
        lev.set_inflow(2, face.to(dev))
        A = torch.nan_to_num(torch.from_numpy(wl.arena).to(dev))
        B = torch.zeros_like(A)
        g = lev.graph(A, B, wl.dx, _params(case, P.params), case["steps"])
        return dict(kind=kind, lev=lev, a=A, b=B, g=g, odd=case["steps"] % 2)
    lay, n, dx = _layout(case)
    V = _flow(case["flow"], seed, n, dx, dev)
    lev = P.Level(lay)
    p = _params(case, P.params)
    lev.ensure_workspace(p.precision)
    A = _pack(lay, V)
    s = dict(kind=kind, lev=lev, dx=dx, p=p, a=A)
    if kind == "rollout":
        s.update(steps=case["steps"], every=case["every"], w=_pack(lay, _cotangent(seed, V)))
        return s
    s["dt"] = lev.compute_dt(A, dx, p)
    if kind == "grad":
        lev.ensure_adjoint_workspace(p.precision)
        s["w"] = _pack(lay, _cotangent(seed, V))
        return s
    s["b"] = torch.zeros_like(A)
    if kind == "graph":
        s.update(g=lev.graph(A, s["b"], dx, p, case["steps"]), odd=case["steps"] % 2)
    if kind == "species":
        ns = case["ns"]
        lev.ensure_species_workspace(ns, p.precision)
        X = _fractions(seed, n, dx, ns, dev)
        s.update(ns=ns, x=_pack(lay, X * V[0]))
        s["y"] = torch.zeros_like(s["x"])
    return s


def run(s):
    kind = s["kind"]
    if kind == "step":  # the state advances from pass to pass, as in a time loop
        lev, a, b, dt = s["lev"], s["a"], s["b"], s["dt"]
        lev.fill_boundary(a)
        lev.hydro_step(a, b, s["dx"], s["p"], dt_dev=dt, dt_next=dt)
        s["a"], s["b"] = b, a
        return b, dt
    if kind in ("graph", "jet"):
        s["g"].launch()
        return s["b"] if s["odd"] else s["a"]
    if kind == "grad":
        U = s["a"].detach().requires_grad_()
        V = P.hydro_step_autograd(U, s["lev"], s["dt"], s["dx"], s["p"])
        return V.detach(), torch.autograd.grad(V, U, s["w"])[0]
    if kind == "rollout":
        U = s["a"].detach().requires_grad_()
        V = P.rollout(U, s["lev"], s["steps"], s["dx"], s["p"], checkpoint_every=s["every"])
        return V.detach(), torch.autograd.grad(V, U, s["w"])[0]
    if kind == "species":
        lev = s["lev"]
        lev.fill_boundary(s["a"])
        lev.fill_species(s["x"], s["ns"])
        lev.hydro_step_species(s["a"], s["b"], s["x"], s["y"], s["ns"], s["dx"], s["p"], dt_dev=s["dt"])
        return s["b"], s["y"]
    s["t"].step(s["a"], s["b"], s["f"], s["ft"], s["dx"], s["p"], dt_out=s["dt"])
    s["a"], s["b"] = s["b"], s["a"]
    return s["a"], s["f"], s["dt"]


def work(case):
    kind = case["kind"]
    if kind == "amr":
        z = float(case["n"]) ** 3
        return {"bytes": 80.0 * 2 * z, "flops": FLOPS_ZONE * 3 * z}
    if kind == "jet":
        z = float(case["n"]) ** 2 * case["nz"] * case["steps"]
    else:
        n = _layout(case)[1]
        z = float(n[0]) * n[1] * n[2] * (case["steps"] if kind == "graph" else 1)
    if kind == "grad":  # state and cotangent in, new state and gradient out; a reverse costs at least two forwards
        return {"bytes": 160.0 * z, "flops": 3 * FLOPS_ZONE * z}
    if kind == "rollout":
        return {"bytes": 160.0 * z, "flops": 3 * FLOPS_ZONE * z * case["steps"]}
    if kind == "species":
        return {"bytes": (80.0 + 16.0 * case["ns"]) * z, "flops": (FLOPS_ZONE + 300.0 * case["ns"]) * z}
    return {"bytes": 80.0 * z, "flops": FLOPS_ZONE * z}


# -------------------------------------------------- the method in 64 bits --
SMALL = 1e-12


def _sh(a, d, o):
    """Value at the zone o beyond along axis d (the last dimension is x); wraps."""
    return a if o == 0 else torch.roll(a, -o, -1 - d)


def _pad(V, bc, odd=True):
    """Ghost zones of a domain: 4 per side; odd: the normal momentum changes sign at a wall."""
    for d in range(3):
        n, dim = V.shape[-1 - d], V.dim() - 1 - d
        i = torch.arange(-NG, n + NG, device=V.device)
        lo, hi = i < 0, i >= n
        kl, kh = bc[2 * d], bc[2 * d + 1]
        idx = torch.where(lo, i + n if kl == PERIODIC else (-1 - i if kl == REFLECT else torch.zeros_like(i)), i)
        idx = torch.where(hi, i - n if kh == PERIODIC else (2 * n - 1 - i if kh == REFLECT
                                                           else torch.full_like(i, n - 1)), idx)
        if kl == PERIODIC:
            idx = i % n
        V = V.index_select(dim, idx)
        if odd and (kl == REFLECT or kh == REFLECT):
            sg = torch.where((lo & (kl == REFLECT)) | (hi & (kh == REFLECT)), -1.0, 1.0).double()
            shape = [1, 1, 1]
            shape[2 - d] = -1
            V = torch.cat([V[:1 + d], V[1 + d:2 + d] * sg.view(shape), V[2 + d:]])
    return V


def _core(A, g=NG):
    return A[..., g:-g, g:-g, g:-g]


def _prim(U, g):
    r = U[0]
    u, v, w = U[1] / r, U[2] / r, U[3] / r
    p = (g - 1.0) * (U[4] - 0.5 * r * (u * u + v * v + w * w))
    return [r, u, v, w, p.clamp_min(SMALL)]


def _speed(V, h, g):
    r, u, v, w, p = _prim(V, g)
    c = torch.sqrt(g * p / r)
    return max(float(((a.abs() + c) / h[d]).max()) for d, a in enumerate((u, v, w)))


def _flatten(q):
    p, out = q[4], None
    for d in range(3):
        dp = _sh(p, d, 1) - _sh(p, d, -1)
        dp2 = _sh(p, d, 2) - _sh(p, d, -2)
        u = q[1 + d]
        hit = ((_sh(u, d, -1) - _sh(u, d, 1)) > 0) & (dp.abs() > 0.33 * torch.minimum(_sh(p, d, 1), _sh(p, d, -1)))
        chi0 = torch.where(hit, (10.0 * (dp.abs() / dp2.abs().clamp_min(SMALL) - 0.75)).clamp(0.0, 1.0),
                           torch.zeros_like(p))
        lo, hi = _sh(chi0, d, -1), _sh(chi0, d, 1)
        zero = torch.zeros_like(p)
        chi = torch.maximum(chi0, torch.maximum(torch.where(dp < 0, zero, lo), torch.where(dp > 0, zero, hi)))
        out = 1.0 - chi if out is None else torch.minimum(out, 1.0 - chi)
    return out


def _parabola(a, d, phi):
    dl, dr = a - _sh(a, d, -1), _sh(a, d, 1) - a
    dc = 0.5 * (_sh(a, d, 1) - _sh(a, d, -1))
    m = torch.minimum(torch.minimum(dc.abs(), 2.0 * dl.abs()), 2.0 * dr.abs())
    s = torch.where(dl * dr > 0, m * torch.sign(dc), torch.zeros_like(a))
    aL = 0.5 * (_sh(a, d, -1) + a) - (s - _sh(s, d, -1)) / 6.0
    aR = 0.5 * (a + _sh(a, d, 1)) - (_sh(s, d, 1) - s) / 6.0
    aL, aR = phi * aL + (1.0 - phi) * a, phi * aR + (1.0 - phi) * a
    ext = (aR - a) * (a - aL) <= 0
    t, e = (aR - aL) * (a - 0.5 * (aL + aR)), (aR - aL) ** 2 / 6.0
    hi, lo = ~ext & (t > e), ~ext & (t < -e)
    L = torch.where(ext, a, torch.where(hi, 3.0 * a - 2.0 * aR, aL))
    R = torch.where(ext, a, torch.where(lo, 3.0 * a - 2.0 * aL, aR))
    return L, R, 6.0 * a - 3.0 * (L + R)


def _swept(par, sg, high):
    L, R, a6 = par
    if high:
        return R - 0.5 * sg * ((R - L) - (1.0 - 2.0 / 3.0 * sg) * a6)
    return L + 0.5 * sg * ((R - L) + (1.0 - 2.0 / 3.0 * sg) * a6)


def _trace(q, d, phi, dt, h, g, grav):
    """States at the high and the low d face of every zone."""
    r, p, un = q[0], q[4], q[1 + d]
    c = torch.sqrt(g * p / r)
    par = [_parabola(a, d, phi) for a in q]
    lam = [un - c, un, un + c]
    zero = torch.zeros_like(r)
    out = []
    for high in (True, False):
        sgn = 1.0 if high else -1.0
        s = [(sgn * v).clamp_min(0.0) * (dt / h[d]) for v in lam]
        on = [(sgn * v) > 0 for v in lam]
        ref = [_swept(a, s[2] if high else s[0], high) for a in par]

        def jump(m, k):
            return ref[m] - _swept(par[m], s[k], high)
        a1 = torch.where(on[0], (jump(4, 0) - r * c * jump(1 + d, 0)) / (2.0 * c * c), zero)
        a2 = torch.where(on[1], jump(0, 1) - jump(4, 1) / (c * c), zero)
        a3 = torch.where(on[2], (jump(4, 2) + r * c * jump(1 + d, 2)) / (2.0 * c * c), zero)
        e = list(ref)
        e[0] = ref[0] - (a1 + a2 + a3)
        e[1 + d] = ref[1 + d] + c / r * (a1 - a3)
        e[4] = ref[4] - c * c * (a1 + a3)
        for m in (1, 2, 3):
            if m != 1 + d:
                e[m] = ref[m] - torch.where(on[1], jump(m, 1), zero)
            if grav[m - 1] != 0.0:
                e[m] = e[m] + 0.5 * dt * grav[m - 1]
        e[0], e[4] = e[0].clamp_min(SMALL), e[4].clamp_min(SMALL)
        out.append(e)
    return out


def _sample(ro, uo, po, C, W, us, p, g):
    """State on the face on the left side of the contact."""
    v = 1.0 / ro - (p - po) / (W * W)
    bad = (v <= 0) | (1.0 / torch.where(v > 0, v, torch.ones_like(v)) < SMALL)
    rs = torch.where(bad, torch.full_like(v, SMALL), 1.0 / torch.where(bad, torch.ones_like(v), v))
    shock = p > po
    hd, tl = uo - C / ro, us - torch.sqrt(g * p / rs)
    star = torch.where(shock, (uo - W / ro) < 0, (hd < 0) & (tl <= 0))
    fan = ~shock & (hd < 0) & (tl > 0)
    w = torch.where(fan, -hd / torch.where(fan, tl - hd, torch.ones_like(hd)), torch.zeros_like(hd))
    w = torch.where(star, torch.ones_like(w), w)
    return [torch.where(star, s, torch.where(fan, (1.0 - w) * o + w * s, o))
            for o, s in ((ro, rs), (uo, us), (po, p))]


def _riemann(L, R, d, g, iters=3):
    beta = (g + 1.0) / (2.0 * g)
    rl, ul, pl, rr, ur, pr = L[0], L[1 + d], L[4], R[0], R[1 + d], R[4]
    cl, cr = torch.sqrt(g * pl * rl), torch.sqrt(g * pr * rr)
    p = (((cr * pl + cl * pr) + cl * cr * (ul - ur)) / (cl + cr)).clamp_min(SMALL)
    for _ in range(iters):
        wl, wr = (C * torch.sqrt(1.0 + beta * (p / po - 1.0)) for C, po in ((cl, pl), (cr, pr)))
        iz = (0.5 * (1.0 + (cl / wl) ** 2) / wl) + (0.5 * (1.0 + (cr / wr) ** 2) / wr)
        p = (p - ((ur + (p - pr) / wr) - (ul - (p - pl) / wl)) / iz).clamp_min(SMALL)
    wl, wr = (C * torch.sqrt(1.0 + beta * (p / po - 1.0)) for C, po in ((cl, pl), (cr, pr)))
    us = ((wl * ul + wr * ur) + (pl - pr)) / (wl + wr)
    a = _sample(rl, ul, pl, cl, wl, us, p, g)
    b = _sample(rr, -ur, pr, cr, wr, -us, p, g)
    b[1] = -b[1]
    t = [m for m in (1, 2, 3) if m != 1 + d]
    a, b = a + [L[t[0]], L[t[1]]], b + [R[t[0]], R[t[1]]]
    q0, q1, q2, q3, q4 = (torch.where(us > 0, x, torch.where(us < 0, y, 0.5 * (x + y))) for x, y in zip(a, b))
    m = q0 * q1
    F = [m, None, None, None, q1 * (q2 / (g - 1.0) + 0.5 * q0 * (q1 * q1 + q3 * q3 + q4 * q4) + q2)]
    F[1 + d] = m * q1 + q2
    F[t[0]], F[t[1]] = m * q3, m * q4
    return F


def _to_cons(q, g):
    r = q[0]
    return [r, r * q[1], r * q[2], r * q[3],
            q[4] / (g - 1.0) + 0.5 * r * (q[1] * q[1] + q[2] * q[2] + q[3] * q[3])]


def _to_prim(U, g):
    r = U[0].clamp_min(SMALL)
    u, v, w = U[1] / r, U[2] / r, U[3] / r
    p = (g - 1.0) * (U[4] - 0.5 * r * (u * u + v * v + w * w))
    return [r, u, v, w, p.clamp_min(SMALL)]


def _solve(hi, lo, d, g, walls):
    """Fluxes at every zone's low d face, from the high-face states of the
    zone below and its own low-face states; walls: positions (low, high) of
    wall faces along d or None."""
    L, R = [_sh(a, d, -1) for a in hi], list(lo)
    for k, x in enumerate(walls or ()):
        if x is None:
            continue
        at = torch.arange(R[0].shape[-1 - d], device=R[0].device) == x
        at = at.view([-1 if i == 2 - d else 1 for i in range(3)])
        for m in range(5):
            sg = -1.0 if m == 1 + d else 1.0
            l, r = L[m], R[m]
            if k == 0:
                L[m] = torch.where(at, sg * r, l)
            else:
                R[m] = torch.where(at, sg * l, r)
    return _riemann(L, R, d, g)


def _diff(F, d):
    return _sh(F, d, 1) - F


def _advance(U, dt, h, g, grav=(0.0, 0.0, 0.0), walls=(None, None, None), X=None):
    """One step of every zone of U (5, z, y, x); neighbours wrap, so a padded
    domain's result is right away from its edges.  X: mass fractions.
    Returns (U', fluxes at the zones' low faces[, rho X'])."""
    q = _prim(U, g)
    phi = _flatten(q)
    tr = [_trace(q, d, phi, dt, h, g, grav) for d in range(3)]
    F1 = [_solve(tr[d][0], tr[d][1], d, g, walls[d]) for d in range(3)]

    def corrected(d, side, terms):
        e = _to_cons(tr[d][side], g)
        for F, t, f in terms:
            e = [a - f * dt / h[t] * _diff(b, t) for a, b in zip(e, F)]
        return _to_prim(e, g)
    F2 = {}
    for d in range(3):
        for t in range(3):
            if t != d:
                F2[d, t] = _solve(*[corrected(d, s, [(F1[t], t, 1.0 / 3.0)]) for s in (0, 1)], d, g, walls[d])
    F3 = []
    for d in range(3):
        a, b = [t for t in range(3) if t != d]
        F3.append(_solve(*[corrected(d, s, [(F2[a, b], a, 0.5), (F2[b, a], b, 0.5)]) for s in (0, 1)], d, g,
                         walls[d]))
    un = [U[m] - sum(dt / h[d] * _diff(F3[d][m], d) for d in range(3)) for m in range(5)]
    if any(grav):
        def src(u):
            return [u[0] * grav[0], u[0] * grav[1], u[0] * grav[2], u[1] * grav[0] + u[2] * grav[1] + u[3] * grav[2]]
        s0 = src(U)
        us = [un[0]] + [un[m] + dt * s0[m - 1] for m in (1, 2, 3, 4)]
        s1 = src(us)
        un = [us[0]] + [us[m] + 0.5 * dt * (s1[m - 1] - s0[m - 1]) for m in (1, 2, 3, 4)]
    V = torch.stack(un)
    if X is None:
        return V, F3
    return V, F3, torch.stack([_species(X[s] * U[0], X[s], q, phi, tr, F1, F2, F3, dt, h, g)
                               for s in range(X.shape[0])])


def _species(RX, X, q, phi, tr, F1, F2, F3, dt, h, g):
    c = torch.sqrt(g * q[4] / q[0])
    zero = torch.zeros_like(X)
    xt = []
    for d in range(3):
        par, un = _parabola(X, d, phi), q[1 + d]
        k = dt / h[d]
        hi = torch.where(un > 0, _swept(par, un.clamp_min(0.0) * k, True),
                         _swept(par, (un + c).clamp_min(0.0) * k, True))
        lo = torch.where(un < 0, _swept(par, (-un).clamp_min(0.0) * k, False),
                         _swept(par, (c - un).clamp_min(0.0) * k, False))
        xt.append((hi, lo))

    def carry(F, hi, lo, d):
        return torch.where(F[0] > 0, F[0] * _sh(hi, d, -1), F[0] * lo)

    def corrected(d, s, terms):
        rx, r = tr[d][s][0] * xt[d][s], tr[d][s][0]
        for G, F, t, f in terms:
            rx, r = rx - f * dt / h[t] * _diff(G, t), r - f * dt / h[t] * _diff(F[0], t)
        return rx / r.clamp_min(SMALL)
    G1 = [carry(F1[d], *xt[d], d) for d in range(3)]
    G2 = {(d, t): carry(F2[d, t], *[corrected(d, s, [(G1[t], F1[t], t, 1.0 / 3.0)]) for s in (0, 1)], d)
          for d, t in F2}
    out = RX
    for d in range(3):
        a, b = [t for t in range(3) if t != d]
        G3 = carry(F3[d], *[corrected(d, s, [(G2[a, b], F2[a, b], a, 0.5), (G2[b, a], F2[b, a], b, 0.5)])
                            for s in (0, 1)], d)
        out = out - dt / h[d] * _diff(G3, d)
    return out + zero


def _walls(bc, n):
    return [(NG if bc[2 * d] == REFLECT else None, n[d] + NG if bc[2 * d + 1] == REFLECT else None)
            for d in range(3)]


def _steps(V, count, h, g, grav, bc, pad, cfl=0.5):
    """count steps of a domain: (result, the padded state whose ghosts the
    buffer of the result holds, dt of the next step, its speed)."""
    n = [V.shape[-1 - d] for d in range(3)]
    ghosts = [None, None]
    for k in range(count):
        U = pad(V)
        ghosts[k % 2] = U
        V = _core(_advance(U, cfl / _speed(V, h, g), h, g, grav, _walls(bc, n))[0]).clone()
    s = _speed(V, h, g)
    return V, ghosts[count % 2], cfl / s, s


def _exact_amr(case, seed, dev, g=1.4, cfl=0.5):
    cl, fl, Vc, Vf, h, lo, fe = _hierarchy(case, seed, dev)
    hf = tuple(v / 2 for v in h)
    dt = cfl / max(_speed(Vc, h, g), 0.5 * _speed(Vf, hf, g))
    wrap = (PERIODIC,) * 6
    old = _pad(Vc, wrap)
    V, F = _advance(old, dt, h, g)
    Vn = _core(V).clone()
    new = _pad(Vn, wrap)
    i = torch.arange(-NG, fe + NG, device=dev) + 2 * lo  # fine zone indices with ghosts
    par, off = torch.div(i, 2, rounding_mode="floor") + NG, torch.where(i % 2 == 0, -0.25, 0.25).double()

    def at(A, d=None, o=0):
        for a in range(3):
            A = A.index_select(A.dim() - 1 - a, par + (o if a == d else 0))
        return A
    rg, first, reg = range(3), None, {}
    for k in range(2):
        C = (1.0 - 0.5 * k) * old + 0.5 * k * new
        fine = at(C)
        for d in rg:
            dl, dr = at(C) - at(C, d, -1), at(C, d, 1) - at(C)
            dc = 0.5 * (dl + dr)
            s = torch.where(dl * dr > 0, torch.sign(dc) * torch.minimum(torch.minimum(
                dc.abs(), 2 * dl.abs()), 2 * dr.abs()), torch.zeros_like(dc))
            fine = fine + s * off.view([-1 if a == 2 - d else 1 for a in rg])
        _core(fine).copy_(Vf)
        first = fine.clone() if first is None else first
        W, Ff = _advance(fine, 0.5 * dt, hf, g)
        Vf = _core(W).clone()
        for d in rg:
            for side in (0, 1):
                f = torch.stack(Ff[d]).select(3 - d, NG + side * fe)[:, NG:NG + fe, NG:NG + fe]
                reg[d, side] = reg.get((d, side), 0.0) + sum(f[:, a::2, b::2] for a in (0, 1) for b in (0, 1))
    m = fe // 2
    for d in rg:
        for side in (0, 1):
            face = lo + side * m
            fc = torch.stack(F[d]).select(3 - d, face + NG)[:, NG + lo:NG + lo + m, NG + lo:NG + lo + m]
            z = Vn.select(3 - d, face - 1 if side == 0 else face)[:, lo:lo + m, lo:lo + m]
            z += (-1.0 if side == 0 else 1.0) * dt / h[d] * (reg[d, side] / 8.0 - fc)
    Vn[:, lo:lo + m, lo:lo + m, lo:lo + m] = sum(Vf[:, a::2, b::2, c::2] for a in (0, 1) for b in (0, 1)
                                                 for c in (0, 1)) / 8.0
    return _pack(cl, Vn, new), _pack(fl, Vf, first), torch.tensor([dt, 0.5 * dt], dtype=torch.float64)


def exact(case, seed):
    dev = torch.device("cuda")
    kind = case["kind"]
    if kind == "amr":
        return _exact_amr(case, seed, dev)
    if kind == "jet":
        wl, face = _jet(case, seed)
        lay, bc = wl.layout, wl.layout.bc
        V = torch.from_numpy(_core(torch.from_numpy(wl.arena).view(lay.stored_shape(0))).numpy().copy()).to(dev)
        f = face.to(dev)[:, :, None, :]

        def pad(V):
            out = _pad(V, (OUTFLOW,) * 4 + (PERIODIC,) * 2)
            out[:, :, :NG] = _pad(f, (OUTFLOW,) * 4 + (PERIODIC,) * 2)[:, :, :1]
            return out
        return _pack(lay, *_steps(V, case["steps"], wl.dx, 1.4, (0.0,) * 3, bc, pad)[:2])
    lay, n, h = _layout(case)
    V = _flow(case["flow"], seed, n, h, dev)
    kw = _params(case)
    g, grav, bc = kw["gamma"], kw["grav"], lay.bc
    if kind in ("step", "graph"):
        W, ghosts, dt, s = _steps(V, case.get("steps", 1), h, g, grav, bc, lambda v: _pad(v, bc))
        A = _pack(lay, W, ghosts)
        return (A, torch.tensor([dt, s], dtype=torch.float64)) if kind == "step" else A
    if kind == "species":
        X = _pad(_fractions(seed, n, h, case["ns"], dev), bc, odd=False)
        W, _, RX = _advance(_pad(V, bc), 0.5 / _speed(V, h, g), h, g, X=X)
        return _pack(lay, _core(W)), _pack(lay, _core(RX))
    # differentiation: periodic levels, whose neighbours wrap without ghosts
    U = V.clone().requires_grad_()
    w, W = _cotangent(seed, V), [U]
    for _ in range(case.get("steps", 1)):
        W.append(_advance(W[-1], 0.5 / _speed(W[-1].detach(), h, g), h, g)[0])
    G = torch.autograd.grad(W[-1], U, w)[0]
    # a roll-out's result lies in the buffer whose ghosts were filled two states before
    ghosts = _pad(W[-3].detach(), bc) if len(W) > 2 else None
    return _pack(lay, W[-1].detach(), ghosts), _pack(lay, G)
