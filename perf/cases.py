"""Timing cases of the entropy-stable moving-mesh solver on one MI355X.

Each case is one call (or a short run of whole time steps) through the public
entry points of ``paper_2202_07989_amd.es``, with inputs made from a seed on
the GPU: shock-bubble, tri-point, Riemann and smooth flows of the paper's
materials on a deformed (moving) mesh, at the sizes of the repository's own
configurations and at odd ones.

  listed()             the named cases
  draw(rng)            one more case of the same ranges
  prepare(case, seed)  what a program holds before the call
  run(state)           one pass
  work(case)           bytes and operations a pass cannot do without
  exact(case, seed)    the outputs in plain torch float64, from the same inputs

The float64 evaluation below is written from the scheme's formulas with
tensor operations only and shares no code with the library.
"""
from __future__ import annotations

import math
import random

import torch

NG = 3
F64 = torch.float64
ALPHA = (3.0 / 2.0, -3.0 / 10.0, 1.0 / 30.0)          # sixth-order EC flux and metrics
CHI_SMOOTH = (1.0 / 111.0, 10.0 / 111.0, 100.0 / 111.0)
CHI_SHOCK = (0.95, 0.045, 0.005)
SIGN_TOL, SIGN_TOL32 = 1e-12, 1e-6
PERIODIC, REFLECT, OUTFLOW, INFLOW = 0, 1, 2, 3

# one ideal gas; water / air; the shock-helium and the stiffened shock-bubble
# of the walled examples; the tri-point problem
FLUIDS = {
    "ideal": dict(gamma=(1.4,), cv=(1.0,), pinf=(0.0,), box=(1.0, 1.0, 1.0), chi=CHI_SMOOTH),
    "water": dict(gamma=(4.4, 1.4), cv=(1.0, 1.0), pinf=(6.0e8, 0.0), box=(1.0, 1.0, 1.0), chi=CHI_SHOCK),
    "helium": dict(gamma=(1.4, 1.647), cv=(0.287 / 0.4, 1.578 / 0.647), pinf=(0.0, 0.0),
                   box=(445.0, 89.0, 89.0), chi=CHI_SHOCK),
    "stiff": dict(gamma=(3.0, 1.4), cv=(1.0, 1.0), pinf=(100.0, 0.0), box=(445.0, 89.0, 89.0), chi=CHI_SHOCK),
    "tripoint": dict(gamma=(1.5, 1.4), cv=(1.0, 1.0), pinf=(0.0, 0.0), box=(7.0, 3.0, 3.0), chi=CHI_SHOCK),
}

MONITORS = {
    # density, as in the shock-bubble runs
    "rho": dict(sigma=[0], alpha=[1200.0]),
    # schlieren function, speed, partial densities and pressure (Example 5.9)
    "five": dict(sigma=[5, 4, 1, 2, 3], alpha=[600.0, 500.0, 1200.0, 1200.0, 1200.0], psi=[120.0, 20.0]),
    # gradient and Laplacian of the density (isentropic vortex)
    "lap": dict(sigma=[1], alpha=[20.0], beta=[10.0], form=1),
}


def listed():
    return [
        # the 64^2 one-species accuracy configuration: two short launches
        dict(name="rhs-2d-64", kind="rhs", fluid="ideal", n0=64, n1=64, n2=0, moving=False, recon="mr",
             precision="fp64"),
        # the 512^2 water/air shock-bubble, one Runge-Kutta stage on its moving mesh
        dict(name="stage-2d-512", kind="stage", fluid="water", n0=512, n1=512, n2=0, moving=True, recon="mr",
             precision="fp64"),
        # the headline 256^3 water/air shock-bubble, one stage
        dict(name="stage-3d-256", kind="stage", fluid="water", n0=256, n1=256, n2=256, moving=True, recon="mr",
             precision="fp64"),
        # the walled 3D shock-helium example at its own size, mixed precision
        dict(name="stage-3d-400x80x80-mixed", kind="stage", fluid="helium", n0=400, n1=80, n2=80, moving=True,
             recon="mr", precision="mixed"),
        # the classical-WENO comparison variant on an odd one-species box
        dict(name="rhs-3d-97x61x45-js", kind="rhs", fluid="ideal", n0=97, n1=61, n2=45, moving=True, recon="js",
             precision="fp64"),
        # GCL metrics of a stage mesh, needed twice in every moving-mesh step
        dict(name="metrics-3d-256", kind="metrics", fluid="water", n0=256, n1=256, n2=256),
        # mesh step of the walled stiffened shock-bubble with its five-variable monitor
        dict(name="mesh-2d-800x160", kind="mesh", fluid="stiff", n0=800, n1=160, n2=0, monitor="five", sweeps=10,
             smooth=3),
        # mesh step of the headline run
        dict(name="mesh-3d-256", kind="mesh", fluid="water", n0=256, n1=256, n2=256, monitor="rho", sweeps=5,
             smooth=3),
        # time-step bound and entropy total, taken once a step
        dict(name="diagnostics-3d-256", kind="diag", fluid="water", n0=256, n1=256, n2=256),
        # four whole steps of the walled tri-point problem from a kept state
        dict(name="step-2d-350x150", kind="step", fluid="tripoint", n0=350, n1=150, n2=0, monitor="rho", sweeps=10,
             smooth=10, steps=4, precision="fp64"),
        # two whole steps of the headline run from a kept state
        dict(name="step-3d-256", kind="step", fluid="water", n0=256, n1=256, n2=256, monitor="rho", sweeps=5,
             smooth=3, steps=2, precision="fp64"),
        # 64 independent instances of uneven size, two batched steps from a kept state
        dict(name="batch-64", kind="batch", fluid="water", count=64, lo=128, hi=1024, steps=2, precision="fp64"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _size(rng, dim):
    if dim == 2:
        return _log_int(rng, 24, 1400), _log_int(rng, 24, 1400), 0
    return _log_int(rng, 17, 224), _log_int(rng, 17, 224), _log_int(rng, 17, 224)


def draw(rng):
    kind = rng.choice(["rhs", "stage", "stage", "metrics", "mesh", "diag", "step", "batch"])
    if kind == "batch":
        lo = _log_int(rng, 32, 200)
        return dict(kind=kind, fluid="water", count=_log_int(rng, 1, 48), lo=lo, hi=lo + _log_int(rng, 16, 600),
                    steps=rng.choice([1, 2]), precision=rng.choice(["fp64", "fp64", "mixed"]))
    fluid = rng.choice(["ideal", "water", "water", "helium", "stiff", "tripoint"])
    n0, n1, n2 = _size(rng, rng.choice([2, 3]))
    case = dict(kind=kind, fluid=fluid, n0=n0, n1=n1, n2=n2)
    if kind in ("rhs", "stage"):
        recon = rng.choice(["mr", "mr", "mr", "js"])
        prec = "fp64" if recon == "js" else rng.choice(["fp64", "fp64", "mixed"])
        case.update(moving=rng.choice([True, True, False]), recon=recon, precision=prec)
    if kind in ("mesh", "step"):
        mon = rng.choice(["rho", "lap"] if fluid == "ideal" else ["rho", "rho", "five"])
        case.update(monitor=mon, sweeps=rng.choice([5, 10]), smooth=10 if mon == "lap" else rng.choice([3, 10]))
    if kind == "step":
        case.update(steps=rng.choice([1, 2]), precision=rng.choice(["fp64", "fp64", "mixed"]))
    return case


# --------------------------------------------------------------------------
# grids and fields: (components, z, y, x) arrays padded by three ghost layers
# --------------------------------------------------------------------------
def _device():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


def _spec(case, n=None):
    fl = FLUIDS[case["fluid"]]
    n = n or (case["n0"], case["n1"], case["n2"])
    dim = 3 if n[2] > 0 else 2
    n = tuple(n[:dim]) + (1,) * (3 - dim)
    box = fl["box"]
    sp = dict(dim=dim, nspec=len(fl["gamma"]), n=n, ng=NG, len=tuple(box[k] if k < dim else 1.0 for k in range(3)),
              dxi=tuple(box[k] / n[k] if k < dim else 1.0 for k in range(3)), w=3, gamma=fl["gamma"], cv=fl["cv"],
              pinf=fl["pinf"], chi=fl["chi"], weno_eps=1e-10, dissipation=1,
              reconstruction=1 if case.get("recon") == "js" else 0, sign_tol=SIGN_TOL, sign_tol32=SIGN_TOL32)
    if case["fluid"] == "tripoint":
        sp["bc"] = [(REFLECT, REFLECT)] * dim
        sp["wall"] = [(0.0, box[k]) for k in range(dim)]
        sp["inflow"] = {}
    if case["fluid"] in ("helium", "stiff"):
        sp["bc"] = [(OUTFLOW, INFLOW)] + [(REFLECT, REFLECT)] * (dim - 1)
        sp["wall"] = [(0.0, 445.0)] + [(-44.5, 44.5)] * (dim - 1)
        _, _, post = _states(case["fluid"])
        U = _conserved(sp, [torch.tensor(post[l], dtype=F64) for l in range(2)],
                       [torch.tensor(post[2] if k == 0 else 0.0, dtype=F64) for k in range(dim)],
                       torch.tensor(post[3], dtype=F64))
        sp["inflow"] = {(0, 1): [float(u) for u in U]}
    return sp


def _pad(sp, a):
    """Interior values (C, n2, n1, n0) in a padded array of zeros."""
    z = NG if sp["dim"] == 3 else 0
    return torch.nn.functional.pad(a, (NG, NG, NG, NG, z, z))


def _at(sp, a, **off):
    """Interior of a padded array, shifted by off (k0, k1, k2 nodes)."""
    n, z = sp["n"], NG if sp["dim"] == 3 else 0
    o = [off.get("k%d" % k, 0) for k in range(3)]
    return a[..., z + o[2]:z + o[2] + n[2], NG + o[1]:NG + o[1] + n[1], NG + o[0]:NG + o[0] + n[0]]


def _xi(sp, dev):
    out = []
    for k in range(sp["dim"]):
        shape = [1, 1, 1]
        shape[2 - k] = sp["n"][k]
        out.append(((torch.arange(sp["n"][k], device=dev, dtype=F64) + 0.5) * sp["dxi"][k]).view(shape))
    return out


def _bc(sp, k, side):
    return sp["bc"][k][side] if "bc" in sp else PERIODIC


def _gather(sp, a, outflow=False):
    """Every ghost node takes the value of the interior node it images."""
    for k in range(sp["dim"]):
        n = sp["n"][k]
        i = torch.arange(-NG, n + NG, device=a.device)
        img = i.clone()
        for side, out in ((0, i < 0), (1, i >= n)):
            kind = _bc(sp, k, side)
            if kind == PERIODIC:
                m = i % n
            elif kind == OUTFLOW and outflow:
                m = torch.full_like(i, 0 if side == 0 else n - 1)
            else:
                m = -1 - i if side == 0 else 2 * n - 1 - i
            img = torch.where(out, m, img)
        a = a.index_select(a.dim() - 1 - k, img + NG)
    return a


def _ghost_slices(sp, a, k):
    """(side, view) of the ghost layers of direction k."""
    d = a.dim() - 1 - k
    return [(0, a.narrow(d, 0, NG)), (1, a.narrow(d, NG + sp["n"][k], NG))]


def _fill(sp, a, what="plain"):
    """Ghost layers by the face rules: plain, mesh, disp, jxx or jxt fields."""
    a = _gather(sp, a)
    d = sp["dim"]
    for c in range(a.shape[0]):
        for k in range(d):
            for side, g in _ghost_slices(sp, a[c], k):
                if _bc(sp, k, side) == PERIODIC:
                    if what == "mesh" and c == k:
                        g += (1 if side else -1) * sp["len"][k]
                elif what == "mesh" and c == k:
                    g.mul_(-1.0).add_(2.0 * sp["wall"][k][side])
                elif (what in ("disp", "jxt") and c == k) or (what == "jxx" and (c // d == k) != (c % d == k)):
                    g.mul_(-1.0)
    return a


def _fill_state(sp, JU, J):
    """Ghost layers of J and JU: wrapped, reflected, outflow or inflow."""
    Jg = _gather(sp, J)
    if "bc" not in sp:
        return _gather(sp, JU), Jg
    N, d = sp["nspec"], sp["dim"]
    inside = torch.where(J > 0, J, torch.ones_like(J))
    U = _gather(sp, JU / inside, outflow=True)
    for k in range(d):
        for side, g in _ghost_slices(sp, U[N + k], k):
            if _bc(sp, k, side) == REFLECT:
                g.mul_(-1.0)
    for (k, side), state in sp["inflow"].items():
        for c in range(U.shape[0]):
            _ghost_slices(sp, U[c], k)[side][1].fill_(state[c])
    return U * Jg, Jg


# --------------------------------------------------------------------------
# inputs
# --------------------------------------------------------------------------
def _states(fluid):
    """Primitive states (rho_1, rho_2, v_1, p): bubble, ahead of and behind the shock."""
    if fluid == "helium":
        e = 0.03
        return (e, 1.225 * 0.287 / 1.578 - e, 0.0, 101325.0), (1.225 - e, e, 0.0, 101325.0), \
            (1.6861 - e, e, -113.5243, 159060.0)
    e = 0.05
    return (e, 5.0 - e, 0.0, 100.0), (1.0 - e, e, 0.0, 100.0), (1.980198 - e, e, -121.2497, 29800.0)


def _conserved(sp, rho, v, p):
    N, d = sp["nspec"], sp["dim"]
    rR = sum(rho[l] * (sp["cv"][l] * (sp["gamma"][l] - 1.0)) for l in range(N))
    T = (p + sum(sp["pinf"])) / rR
    rt = sum(rho)
    E = sum(sp["cv"][l] * rho[l] * T + sp["pinf"][l] for l in range(N)) + 0.5 * rt * sum(q * q for q in v)
    return torch.stack(torch.broadcast_tensors(*rho, *[rt * q for q in v], E))


def _modes(sp, rnd, xi, count=3):
    """A displacement field of unit size per direction: smooth waves, zero on
    the faces of a walled direction."""
    d, out = sp["dim"], []
    for k in range(d):
        f = 0.0
        for _ in range(count):
            a, t = rnd.uniform(0.3, 1.0) * rnd.choice([-1, 1]) / count, 1.0
            arg, ph = 0.0, rnd.uniform(0.0, 2.0 * math.pi)
            for j in range(d):
                m = rnd.choice([1, 1, 2])
                if "bc" in sp:
                    w = math.pi * m * xi[j] / sp["len"][j]
                    t = t * (torch.sin(w) if j == k else torch.cos(w))
                else:
                    arg = arg + 2.0 * math.pi * m * xi[j] / sp["len"][j]
            f = f + a * (t if "bc" in sp else torch.sin(arg + ph))
        out.append(f.expand(sp["n"][2], sp["n"][1], sp["n"][0]))
    return out


def _flow(case, sp, rnd, x):
    """Primitive variables of the case's flow at the mesh nodes x."""
    d, h, fl = sp["dim"], max(sp["dxi"][:sp["dim"]]), case["fluid"]
    z = torch.zeros_like(x[0])
    if fl == "ideal":
        ph = [rnd.uniform(0.0, 2.0 * math.pi) for _ in range(3)]
        s = 2.0 * math.pi * sum(x)
        rho = 1.0 + 0.2 * torch.sin(s + ph[0])
        v = [1.0 + 0.1 * torch.sin(2.0 * math.pi * x[(k + 1) % d] + ph[1]) for k in range(d)]
        return [rho], v, 1.0 + 0.05 * torch.sin(2.0 * math.pi * x[0] + ph[2])
    if fl == "tripoint":
        e = 1e-5
        left = 0.5 * (1.0 + torch.tanh((rnd.uniform(0.9, 1.1) - x[0]) / h))
        ft = 0.5 * (1.0 + torch.tanh((x[1] - rnd.uniform(1.4, 1.6)) / h))
        w = [left, (1.0 - left) * ft, (1.0 - left) * (1.0 - ft)]
        st = [(1.0 - e, e, 1.0), (0.125 - e, e, 0.1), (e, 1.0 - e, 0.1)]
        mix = [sum(w[q] * st[q][c] for q in range(3)) for c in range(3)]
        return [mix[0], mix[1]], [z] * d, mix[2]
    if fl == "water":
        mach, t = rnd.uniform(1.4, 1.6), 1e-3
        G = (4.4 * (1000.0 - t) + 1.4 * t) / 1000.0
        ratio = (G + 1.0) * mach ** 2 / ((G - 1.0) * mach ** 2 + 2.0)
        p0, pi = 1.0e5, 6.0e8
        p1 = (p0 + pi) * (2.0 * G * mach ** 2 - G + 1.0) / (G + 1.0) - pi
        u1 = mach * math.sqrt(G * (p0 + pi) / 1000.0) * (1.0 - 1.0 / ratio)
        b, a, q = (t, 1.0 - t, 0.0, p0), (1000.0 - t, t, 0.0, p0), ((1000.0 - t) * ratio, t * ratio, u1, p1)
        centre = [rnd.uniform(0.45, 0.55) for _ in range(d)]
        radius, width = rnd.uniform(0.18, 0.22), 2.0 * h
        shock = torch.tanh((x[0] - rnd.uniform(0.16, 0.22)) / width)
    else:
        b, a, q = _states(fl)
        centre = [rnd.uniform(220.0, 230.0)] + [rnd.uniform(-2.0, 2.0) for _ in range(d - 1)]
        radius, width = rnd.uniform(23.0, 27.0), h
        shock = torch.tanh((rnd.uniform(270.0, 280.0) - x[0]) / width)
    r = torch.sqrt(sum((x[k] - centre[k]) ** 2 for k in range(d)))
    fb = 0.5 * (1.0 + torch.tanh((radius - r) / width))
    fs = 0.5 * (1.0 - shock)
    w = [fb, (1.0 - fb) * (1.0 - fs), (1.0 - fb) * fs]
    mix = [w[0] * b[c] + w[1] * a[c] + w[2] * q[c] for c in range(4)]
    return [mix[0], mix[1]], [mix[2]] + [z] * (d - 1), mix[3]


def _inputs(case, seed, dev):
    """State, mesh, displacement and metrics of one grid."""
    sp = _spec(case)
    d, rnd = sp["dim"], random.Random(seed)
    xi = _xi(sp, dev)
    modes, more = _modes(sp, rnd, xi), _modes(sp, rnd, xi)
    low = [sp["wall"][k][0] if "wall" in sp else 0.0 for k in range(d)]
    # whole steps and mesh steps start from the uniform mesh; the others see
    # the deformed mesh of a run under way
    amp = 0.0 if case["kind"] in ("mesh", "step") else 0.02
    x = torch.stack([low[k] + xi[k] + amp * sp["len"][k] * modes[k] for k in range(d)])
    rho, v, p = _flow(case, sp, rnd, list(x))
    U = _conserved(sp, rho, v, p)
    x = _fill(sp, _pad(sp, x), "mesh")
    disp = _fill(sp, _pad(sp, torch.stack([0.15 * sp["dxi"][k] * more[k] for k in range(d)])), "disp")
    jxx = _metrics(sp, x)
    J = _pad(sp, _jacobian(sp, x, jxx))
    JU = _pad(sp, U * _at(sp, J))
    JU, J = _fill_state(sp, JU, J)
    lam = _wavespeed(sp, JU, J, jxx)
    dt = 0.3 / lam
    return dict(sp=sp, x=x, disp=disp, jxx=jxx, J=J, JU=JU, dt=dt.reshape(1), bump=more[0])


def _batch_sizes(case):
    rng = random.Random("sizes %d %d %d" % (case["count"], case["lo"], case["hi"]))
    return [max(8, int(case["lo"] * (case["hi"] / case["lo"]) ** rng.random())) for _ in range(case["count"])]


def _riemann(sp, rnd, dev):
    """Four-quadrant Riemann data on a uniform n x n mesh, layers two cells wide."""
    h = sp["dxi"][0]
    q = []
    for _ in range(4):
        r, y = rnd.uniform(0.5, 2.0), rnd.uniform(0.05, 0.95)
        th, s = rnd.uniform(0.0, 2.0 * math.pi), rnd.uniform(0.0, 1.0)
        q.append((r * y, r * (1.0 - y), s * math.cos(th), s * math.sin(th), rnd.uniform(5.0, 9.0)))

    def layer(s):
        f = 0.5 * (torch.tanh((s - 0.5) / (2 * h)) - torch.tanh((s - 1.0) / (2 * h)) - torch.tanh(s / (2 * h)) + 1.0)
        return f.clamp(0.0, 1.0)

    xi = _xi(sp, dev)
    a, b = layer(xi[0]), layer(xi[1])
    w = [(1 - a) * (1 - b), a * (1 - b), (1 - a) * b, a * b]
    m = [sum(w[k] * q[k][c] for k in range(4)) for c in range(5)]
    JU = _pad(sp, _conserved(sp, [m[0], m[1]], [m[2], m[3]], 10.0 ** m[4]))
    J = _pad(sp, torch.ones((1,) + tuple(JU.shape[1:]), dtype=F64, device=dev)[:, :, NG:-NG, NG:-NG])
    x = torch.stack(torch.broadcast_tensors(*[t + torch.zeros(1, sp["n"][1], sp["n"][0], dtype=F64, device=dev)
                                              for t in xi]))
    x = _fill(sp, _pad(sp, x), "mesh")
    JU, J = _fill_state(sp, JU, J)
    return JU, J, _metrics(sp, x)


def _batch_inputs(case, seed, dev):
    out = []
    for b, n in enumerate(_batch_sizes(case)):
        sp = _spec(case, (n, n, 0))
        out.append((sp,) + _riemann(sp, random.Random("%d %d" % (seed, b)), dev))
    return out


def _monitor(case):
    return dict(MONITORS[case["monitor"]], n_sweeps=case["sweeps"], n_smooth=case["smooth"])


CFL = 0.3


# --------------------------------------------------------------------------
# the cases through the library
# --------------------------------------------------------------------------
def prepare(case, seed):
    from paper_2202_07989_amd import es

    prec = es.ES_MIXED if case.get("precision") == "mixed" else es.ES_FP64
    dev = torch.device("cuda")
    if case["kind"] == "batch":
        insts = _batch_inputs(case, seed, dev)
        s = dict(case=case, batch=es.Batch([i[0] for i in insts], precision=prec))
        kept = torch.cat([t.reshape(-1) for _, JU, J, _ in insts for t in (JU, J)])
        work, parts, at = torch.empty_like(kept), [], 0
        for _, JU, J, _ in insts:
            for t in (JU, J):
                parts.append(work[at:at + t.numel()].view(t.shape))
                at += t.numel()
        s.update(kept=kept, work=work, JU=es.PtrTable(parts[0::2]), J=es.PtrTable(parts[1::2]),
                 jxx=es.PtrTable([i[3] for i in insts]), dt=torch.zeros(len(insts), dtype=F64, device=dev))
        work.copy_(kept)
        s["batch"].max_wavespeed_batched(s["JU"], s["J"], s["jxx"], CFL, None, s["dt"])
        s["batch"].es_batch_autotune(s["JU"], s["J"], s["jxx"], None, s["dt"], reps=2)
        return s
    f = _inputs(case, seed, dev)
    s = dict(case=case, ctx=es.Context(f["sp"], precision=prec), x=f["x"], JU=f["JU"], J=f["J"], jxx=f["jxx"],
             dt=f["dt"])
    kind, d = case["kind"], f["sp"]["dim"]
    if kind in ("rhs", "stage"):
        s["jxt"] = _time_metrics(f) if case["moving"] else None
        s["oU"], s["oJ"] = torch.zeros_like(f["JU"]), torch.zeros_like(f["J"])
        if kind == "stage":
            s["JUn"], s["Jn"] = _earlier(f)
    elif kind == "metrics":
        s["disp"] = f["disp"]
        s["ojx"], s["ojt"] = torch.zeros_like(f["jxx"]), torch.zeros_like(f["jxx"][:d])
    elif kind == "mesh":
        s.update(mon=_monitor(case), disp=torch.zeros_like(f["x"]), dtau=torch.zeros(1, dtype=F64, device=dev))
    elif kind == "diag":
        s.update(lam=torch.zeros(1, dtype=F64, device=dev), odt=torch.zeros(1, dtype=F64, device=dev),
                 total=torch.zeros(1, dtype=F64, device=dev))
    elif kind == "step":
        parts = [f["JU"], f["J"], f["x"]]
        kept = torch.cat([t.reshape(-1) for t in parts])
        work, views, at = torch.empty_like(kept), [], 0
        for t in parts:
            views.append(work[at:at + t.numel()].view(t.shape))
            at += t.numel()
        s.update(kept=kept, work=work, JU=views[0], J=views[1], x=views[2], jxx=None, mon=_monitor(case),
                 odt=torch.zeros(1, dtype=F64, device=dev), dtau=torch.zeros(1, dtype=F64, device=dev))
    return s


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "batch":
        s["work"].copy_(s["kept"])
        for _ in range(case["steps"]):
            s["batch"].es_step_batched(CFL, s["JU"], s["J"], s["jxx"], None, s["dt"])
        return s["work"], s["dt"]
    ctx = s["ctx"]
    if kind == "rhs":
        ctx.es_rhs(s["JU"], s["J"], s["jxx"], s["jxt"], s["oU"], s["oJ"])
        return s["oU"], s["oJ"]
    if kind == "stage":
        ctx.es_rk_stage(1, s["dt"], s["JUn"], s["Jn"], s["JU"], s["J"], s["jxx"], s["jxt"], s["oU"], s["oJ"])
        return s["oU"], s["oJ"]
    if kind == "metrics":
        ctx.es_metrics(s["x"], s["disp"], 0.5, s["dt"], s["ojx"], s["ojt"])
        return s["ojx"], s["ojt"]
    if kind == "mesh":
        ctx.mesh_redistribute(s["mon"], s["JU"], s["J"], s["x"], s["disp"], s["dtau"])
        return s["disp"], s["dtau"]
    if kind == "diag":
        ctx.max_wavespeed(s["JU"], s["J"], s["jxx"], CFL, s["lam"], s["odt"])
        ctx.es_entropy(s["JU"], s["J"], s["total"])
        return s["lam"], s["odt"], s["total"]
    s["work"].copy_(s["kept"])
    for _ in range(case["steps"]):
        ctx.es_step(s["JU"], s["J"], s["x"], mon=s["mon"], cfl=CFL, move_mesh=True, dt_dev=s["odt"],
                    dtau_dev=s["dtau"])
    return s["JU"], s["J"], s["x"], s["odt"], s["dtau"]


def work(case):
    """Each input read once and each output written once; operations of the
    flux per cell and stage (primitives, two-point fluxes, dissipation)."""
    if case["kind"] == "batch":
        cells = sum(n * n for n in _batch_sizes(case))
        return dict(bytes=8.0 * cells * case["steps"] * (2 * 6 + 4), flops=4040.0 * 3 * cells * case["steps"])
    d = 3 if case["n2"] else 2
    N = 1 if case["fluid"] == "ideal" else 2
    cells = float(case["n0"] * case["n1"] * (case["n2"] or 1))
    nc, dd = N + d + 1, d * d
    stage_flops = {(2, 1): 3029.0, (2, 2): 4040.0, (3, 1): 5804.0, (3, 2): 7337.0}[(d, N)]
    kind = case["kind"]
    if kind in ("rhs", "stage"):
        fields = 2 * (nc + 1) + dd + (d if case["moving"] else 0) + (nc + 1 if kind == "stage" else 0)
        return dict(bytes=8.0 * cells * fields, flops=stage_flops * cells)
    if kind == "metrics":
        return dict(bytes=8.0 * cells * (2 * d + dd + d), flops=cells * (90.0 * d if d == 3 else 40.0))
    mon = MONITORS[case.get("monitor", "rho")]
    reads = nc + 1 if len(mon["sigma"]) > 1 else N + 1
    mesh_flops = cells * (27.0 * case.get("smooth", 0) + 40.0 * case.get("sweeps", 0) + 40.0 * len(mon["sigma"]))
    if kind == "mesh":
        return dict(bytes=8.0 * cells * (reads + 2 * d), flops=mesh_flops)
    if kind == "diag":
        return dict(bytes=8.0 * cells * (2 * (nc + 1) + dd), flops=cells * 150.0)
    return dict(bytes=case["steps"] * 8.0 * cells * 2 * (nc + 1 + d),
                flops=case["steps"] * (3 * stage_flops * cells + 2 * cells * (90.0 * d if d == 3 else 40.0) + mesh_flops))


# --------------------------------------------------------------------------
# the same in plain torch float64
# --------------------------------------------------------------------------
def exact(case, seed):
    dev = _device()
    if dev.type == "cpu" and case["kind"] != "batch" and case["n0"] * case["n1"] * max(1, case["n2"]) > 300000:
        return None
    if case["kind"] == "batch":
        parts, dts = [], []
        for sp, JU, J, jxx in _batch_inputs(case, seed, dev):
            for _ in range(case["steps"]):
                dt = CFL / _wavespeed(sp, JU, J, jxx)
                JU, J = _rk3(sp, JU, J, dt, lambda st: (jxx, None))
            parts += [JU.reshape(-1), J.reshape(-1)]
            dts.append(dt)
        return torch.cat(parts), torch.stack(dts)
    f = _inputs(case, seed, dev)
    sp, kind = f["sp"], case["kind"]
    if kind in ("rhs", "stage"):
        jxt = _time_metrics(f) if case["moving"] else None
        dU, dJ = _rhs(sp, f["JU"], f["J"], f["jxx"], jxt)
        if kind == "rhs":
            return _pad(sp, dU), _pad(sp, dJ)
        JUn, Jn = _earlier(f)
        return tuple(_pad(sp, 0.75 * _at(sp, qn) + 0.25 * (_at(sp, q) + f["dt"] * L))
                     for qn, q, L in ((JUn, f["JU"], dU), (Jn, f["J"], dJ)))
    if kind == "metrics":
        jxx = _metrics(sp, f["x"] + 0.5 * f["disp"])
        return jxx, _time_metrics(dict(f, jxx=jxx))
    if kind == "mesh":
        return _redistribute(sp, _monitor(case), f["JU"], f["J"], f["x"])
    if kind == "diag":
        lam = _wavespeed(sp, f["JU"], f["J"], f["jxx"])
        return lam.reshape(1), (CFL / lam).reshape(1), _entropy(sp, f["JU"], f["J"]).reshape(1)
    JU, J, x = f["JU"], f["J"], f["x"]
    mon = _monitor(case)
    for _ in range(case["steps"]):
        disp, dtau = _redistribute(sp, mon, JU, J, x)
        dt = CFL / _wavespeed(sp, JU, J, _metrics(sp, x))

        def at_stage(st):
            jxx = _metrics(sp, x + (0.0, 1.0, 0.5)[st] * disp)
            return jxx, _time_metrics(dict(sp=sp, disp=disp, dt=dt, jxx=jxx))

        JU, J = _rk3(sp, JU, J, dt, at_stage)
        x = _fill(sp, x + disp, "mesh")
    return JU, J, x, dt.reshape(1), dtau


def _rk3(sp, JU, J, dt, metrics_of):
    sU, sJ = JU, J
    for st, (a, b) in enumerate(((0.0, 1.0), (0.75, 0.25), (1.0 / 3.0, 2.0 / 3.0))):
        dU, dJ = _rhs(sp, sU, sJ, *metrics_of(st))
        oU = a * _at(sp, JU) + b * (_at(sp, sU) + dt * dU)
        oJ = a * _at(sp, J) + b * (_at(sp, sJ) + dt * dJ)
        sU, sJ = _fill_state(sp, _pad(sp, oU), _pad(sp, oJ))
    return sU, sJ


def _earlier(f):
    """A Q_n a little off Q_s."""
    sp = f["sp"]
    g = 1.0 + 1e-3 * f["bump"]
    return _pad(sp, _at(sp, f["JU"]) * g), _pad(sp, _at(sp, f["J"]) * (2.0 - g))


def _delta(a, k):
    d = a.dim() - 1 - k
    n = a.shape[d] - 2 * NG
    return 0.5 * sum(ALPHA[m - 1] * (a.narrow(d, NG + m, n) - a.narrow(d, NG - m, n)) for m in (1, 2, 3))


def _cut(a, k):
    d = a.dim() - 1 - k
    return a.narrow(d, NG, a.shape[d] - 2 * NG)


def _metrics(sp, x):
    d, h = sp["dim"], sp["dxi"]
    if d == 2:
        e0, e1 = _cut(_delta(x, 0), 1) / h[0], _cut(_delta(x, 1), 0) / h[1]
        m = torch.stack([e1[1], -e1[0], -e0[1], e0[0]])
    else:
        out = []
        for k in range(3):
            a, b = (k + 1) % 3, (k + 2) % 3
            for j in range(3):
                p, q = x[(j + 1) % 3], x[(j + 2) % 3]
                t = _delta(_delta(p, a) * _cut(q, a), b) - _delta(_delta(p, b) * _cut(q, b), a)
                out.append(_cut(t, k) / (h[a] * h[b]))
        m = torch.stack(out)
    return _fill(sp, _pad(sp, m), "jxx")


def _jacobian(sp, x, jxx):
    d, J = sp["dim"], 0.0
    for k in range(d):
        g = _delta(x, k)
        for q in range(d):
            if q != k:
                g = _cut(g, q)
        for j in range(d):
            J = J + g[j] / sp["dxi"][k] * _at(sp, jxx[k * d + j])
    return (J / d).unsqueeze(0)


def _time_metrics(f):
    sp, jxx = f["sp"], f["jxx"]
    d = sp["dim"]
    v = _at(sp, f["disp"]) / f["dt"]
    m = torch.stack([-sum(v[j] * _at(sp, jxx[k * d + j]) for j in range(d)) for k in range(d)])
    return _fill(sp, _pad(sp, m), "jxt")


def _prims(sp, JU, J):
    N, d = sp["nspec"], sp["dim"]
    U = JU / J
    rho = [U[l] for l in range(N)]
    rt = sum(rho)
    v = [U[N + j] / rt for j in range(d)]
    e = U[N + d] - 0.5 * sum(U[N + j] * v[j] for j in range(d)) - sum(sp["pinf"])
    T = e / sum(sp["cv"][l] * rho[l] for l in range(N))
    return rho, v, T


def _gas(sp):
    return [sp["cv"][l] * (sp["gamma"][l] - 1.0) for l in range(sp["nspec"])]


def _wavespeed(sp, JU, J, jxx):
    d, N, Rg = sp["dim"], sp["nspec"], _gas(sp)
    Ji = _at(sp, J)[0]
    rho, v, T = _prims(sp, _at(sp, JU), Ji)
    cvr = sum(sp["cv"][l] * rho[l] for l in range(N))
    G = sum(sp["cv"][l] * sp["gamma"][l] * rho[l] for l in range(N)) / cvr
    c = torch.sqrt(G * T * sum(Rg[l] * rho[l] for l in range(N)) / sum(rho))
    lam = 0.0
    for k in range(d):
        n = [_at(sp, jxx[k * d + j]) for j in range(d)]
        lam = lam + ((sum(v[j] * n[j] for j in range(d))).abs() + c * torch.sqrt(sum(q * q for q in n))) \
            / (Ji * sp["dxi"][k])
    return lam.max()


def _entropy(sp, JU, J):
    Ji, Rg = _at(sp, J)[0], _gas(sp)
    rho, _, T = _prims(sp, _at(sp, JU), Ji)
    eta = -sum(rho[l] * (sp["cv"][l] * torch.log(T) - Rg[l] * torch.log(rho[l])) for l in range(sp["nspec"]))
    return (Ji * eta).sum() * math.prod(sp["dxi"][:sp["dim"]])


def _logmean(a, b):
    s, f = a + b, (a - b) / (a + b)
    g = f.abs() > 1e-7
    safe = torch.where(g, f, torch.full_like(f, 0.5))
    return 0.5 * s * torch.where(g, safe / torch.atanh(safe), 1.0 - f * f / 3.0)


def _rhs(sp, JU, J, jxx, jxt):
    """d(JU)/dt and dJ/dt at the interior nodes."""
    d = sp["dim"]
    dU, dJ = 0.0, 0.0
    for k in range(d):
        def slab(a):
            for j in range(d):
                if j != k:
                    a = _cut(a, j)
            return a

        F, G = _interface(sp, k, slab(JU), slab(J), slab(jxx[k * d:(k + 1) * d]),
                          slab(jxt[k:k + 1]) if jxt is not None else None)
        ax, n = 3 - k, sp["n"][k]
        dU = dU - (F.narrow(ax, 1, n) - F.narrow(ax, 0, n)) / sp["dxi"][k]
        dJ = dJ - (G.narrow(ax, 1, n) - G.narrow(ax, 0, n)) / sp["dxi"][k]
        del F, G
    return dU, dJ


def _interface(sp, k, JU, J, jx, jt):
    """Numerical flux and GCL flux at the n + 1 interfaces along k."""
    N, d, Rg = sp["nspec"], sp["dim"], _gas(sp)
    cv, gam, pin = sp["cv"], sp["gamma"], sum(sp["pinf"])
    rho, v, T = _prims(sp, JU, J[0])
    beta = 1.0 / T
    nt = jt[0] if jt is not None else torch.zeros_like(T)
    ax, n1 = 2 - k, sp["n"][k] + 1

    def nd(a, t):                       # node i + t of the interfaces i + 1/2
        return a.narrow(ax, 2 + t, n1)

    def pair(a, b):
        mean = lambda q: 0.5 * (nd(q, a) + nd(q, b))
        vm = [mean(q) for q in v]
        v2 = sum(mean(q * q) for q in v)
        nx, ntm = [mean(jx[j]) for j in range(d)], mean(nt)
        vdn = sum(vm[j] * nx[j] for j in range(d))
        rl = [_logmean(nd(q, a), nd(q, b)) for q in rho]
        ib = 1.0 / _logmean(nd(beta, a), nd(beta, b))
        Pi = sum(Rg[l] * mean(rho[l]) for l in range(N)) / mean(beta)
        M = [q * (vdn + ntm) for q in rl]
        Mt = sum(M)
        mom = [vm[j] * Mt + (Pi - pin) * nx[j] for j in range(d)]
        E = sum(M[l] * (cv[l] * ib - 0.5 * v2) for l in range(N)) + Mt * sum(q * q for q in vm) + Pi * vdn + pin * ntm
        return torch.stack(M + mom + [E]), ntm

    F, G = 0.0, 0.0
    for m in (1, 2, 3):
        for s in range(m):
            f, g = pair(-s, m - s)
            F = F + ALPHA[m - 1] * f
            G = G + ALPHA[m - 1] * g
    return F - _dissipation(sp, nd, rho, v, T, beta, jx, nt), G.unsqueeze(0)


def _dissipation(sp, nd, rho, v, T, beta, jx, nt):
    N, d, Rg = sp["nspec"], sp["dim"], _gas(sp)
    cv, gam = sp["cv"], sp["gamma"]
    mean = lambda q: 0.5 * (nd(q, 0) + nd(q, 1))
    nx, ntm = [mean(jx[j]) for j in range(d)], mean(nt)
    nn = torch.sqrt(sum(q * q for q in nx))
    # rotation onto the interface normal
    if d == 2:
        rows = [[nx[0] / nn, nx[1] / nn], [-nx[1] / nn, nx[0] / nn]]
    else:
        r = torch.sqrt(nx[0] ** 2 + nx[1] ** 2)
        some = r > 0
        rs = torch.where(some, r, torch.ones_like(r))
        ct = torch.where(some, nx[0] / rs, torch.ones_like(r))
        st = torch.where(some, nx[1] / rs, torch.zeros_like(r))
        cp, sp_ = r / nn, nx[2] / nn
        rows = [[cp * ct, cp * st, sp_], [-st, ct, None], [-sp_ * ct, -sp_ * st, cp]]

    def turn(a):
        return [sum(rows[i][j] * a[j] for j in range(d) if rows[i][j] is not None) for i in range(d)]

    vb = [mean(q) for q in v]
    vh = turn(vb)
    K = 0.5 * sum(q * q for q in vh)
    Tb = 1.0 / _logmean(nd(beta, 0), nd(beta, 1))
    rl = [_logmean(nd(q, 0), nd(q, 1)) for q in rho]
    if N == 1:
        c = torch.sqrt(gam[0] * Rg[0] * Tb)
        H = gam[0] * cv[0] * Tb + K
        sa, se = torch.sqrt(rl[0] / (2.0 * gam[0] * Rg[0])), torch.sqrt(rl[0] / (cv[0] * gam[0]))
        tang = torch.sqrt(rl[0] * Tb)
    else:
        rt = rho[0] + rho[1]
        cvr = sum(cv[l] * rho[l] for l in range(2))
        rR = sum(Rg[l] * rho[l] for l in range(2))
        Gb, Rb = mean(sum(cv[l] * gam[l] * rho[l] for l in range(2)) / cvr), mean(rR / rt)
        p = mean(rR * T - sum(sp["pinf"]))
        rb = _logmean(nd(rt, 0), nd(rt, 1))
        H = (p + sum(cv[l] * rl[l] * Tb + sp["pinf"][l] for l in range(2))) / rb + K
        Y = [q / rb for q in rl]
        e2 = [K - (cv[l] + Rg[l] - Gb * cv[l]) * Tb / (Gb - 1.0) for l in range(2)]
        c, sq = torch.sqrt(Gb * Rb * Tb), torch.sqrt(rb / (Gb * Rb))
        sa = sq / math.sqrt(2.0)
        yy = sq * torch.sqrt(Y[0] * Y[1] * Gb)
        d11, d21 = -yy * math.sqrt(Rg[1] / Rg[0]), yy * math.sqrt(Rg[0] / Rg[1])
        d12, d22 = sq * Y[0] * torch.sqrt(Gb - 1.0), sq * Y[1] * torch.sqrt(Gb - 1.0)
        tang = sq * c
    s = (ntm + sum(vb[j] * nx[j] for j in range(d))).abs() + nn * c
    # columns of R in rows (species, momenta, energy), acoustic pair first
    one = torch.ones_like(c)

    def column(sps, un, scale):
        return [q * scale for q in sps] + [(vh[0] + un) * scale] + [vh[t] * scale for t in range(1, d)]

    ya = [one] if N == 1 else Y
    cols = [column(ya, -c, sa) + [(H - c * vh[0]) * sa], column(ya, c, sa) + [(H + c * vh[0]) * sa]]
    if N == 1:
        cols.append(column([one], 0.0, se) + [K * se])
    else:
        for a, b in ((d11, d21), (d12, d22)):
            cols.append([a, b] + [q * (a + b) for q in vh] + [a * e2[0] + b * e2[1]])
    zero = torch.zeros_like(c)
    for t in range(1, d):
        cols.append([zero] * N + [tang if q == t else zero for q in range(d)] + [tang * vh[t]])
    # entropy variables of the stencil nodes, rotated
    v2 = sum(q * q for q in v)
    Vs = [cv[l] * torch.log(beta) + Rg[l] * torch.log(rho[l]) + cv[l] * gam[l] - 0.5 * beta * v2 for l in range(N)]
    Vm = [beta * q for q in v]
    st = []
    for t in range(-2, 4):
        st.append([nd(q, t) for q in Vs] + turn([nd(q, t) for q in Vm]) + [-nd(beta, t)])
    ay = sum(nd(q.abs(), 0) + nd(q.abs(), 1) for q in Vs)
    av = sum(nd(q.abs(), 0) + nd(q.abs(), 1) for q in Vm)
    ae = nd(beta, 0) + nd(beta, 1)
    RZ = [0.0] * (N + d + 1)
    for col in cols:
        W = [sum(col[e] * y[e] for e in range(N + d + 1) if col[e] is not zero) for y in st]
        B = torch.stack([q.abs() for q in col[:N]]).amax(0) * ay + sum(q.abs() for q in col[N:N + d]) * av \
            + col[N + d].abs() * ae
        jump = W[3] - W[2]
        weno = _weno_js if sp["reconstruction"] else _weno_mr
        # the mirrored stencil's differences change sign, and an odd function with them
        jw = jump - weno(sp, *[W[5 - q] - W[4 - q] for q in range(4)]) - weno(
            sp, *[W[q + 1] - W[q] for q in range(4)])
        Z = torch.where((jw * jump > 0) & (jump.abs() > sp["sign_tol"] * B), jw, zero)
        for e in range(N + d + 1):
            if col[e] is not zero:
                RZ[e] = RZ[e] + col[e] * Z
    mom = [sum(rows[i][j] * RZ[N + i] for i in range(d) if rows[i][j] is not None) for j in range(d)]
    return 0.5 * s * torch.stack(RZ[:N] + mom + [RZ[N + d]])


def _weno_mr(sp, D0, D1, D2, D3):
    """Reconstruction minus the centre value, from the stencil's differences."""
    chi, eps = sp["chi"], sp["weno_eps"]
    a2, a3 = 0.5 * (D1 + D2), 0.5 * (D2 - D1)
    t1 = (7.0 * (D1 + D2) - (D0 + D3)) / 12.0
    t2 = (11.0 * (D0 - D3) + 163.0 * (D2 - D1)) / 260.0
    b4, b5 = (D0 + D3 - D1 - D2) / 12.0, -(D0 - D3 + 3.0 * (D2 - D1)) / 24.0
    be1 = torch.minimum(D1 * D1, D2 * D2)
    be2 = a2 * a2 + 13.0 / 3.0 * a3 * a3
    be3 = t1 * t1 + 13.0 / 3.0 * t2 * t2 + 781.0 / 20.0 * b4 * b4 + 1421461.0 / 2275.0 * b5 * b5
    tau = (0.5 * ((be3 - be1).abs() + (be3 - be2).abs())) ** 2
    w = [chi[m] * (1.0 + tau / (eps + b)) for m, b in enumerate((be1, be2, be3))]
    h2 = (D1 + 2.0 * D2) / 6.0
    h3 = (-2.0 * D0 + 11.0 * D1 + 24.0 * D2 - 3.0 * D3) / 60.0
    return (w[1] * h2 + w[2] * (h3 - chi[1] * h2) / chi[2]) / (w[0] + w[1] + w[2])


def _weno_js(sp, D0, D1, D2, D3):
    eps = sp["weno_eps"]
    b0 = 13.0 / 12.0 * (D1 - D0) ** 2 + 0.25 * (3.0 * D1 - D0) ** 2
    b1 = 13.0 / 12.0 * (D2 - D1) ** 2 + 0.25 * (D1 + D2) ** 2
    b2 = 13.0 / 12.0 * (D3 - D2) ** 2 + 0.25 * (3.0 * D2 - D3) ** 2
    w = [0.1 / (eps + b0) ** 2, 0.6 / (eps + b1) ** 2, 0.3 / (eps + b2) ** 2]
    c = [(5.0 * D1 - 2.0 * D0) / 6.0, (D1 + 2.0 * D2) / 6.0, (4.0 * D2 - D3) / 6.0]
    return (w[0] * c[0] + w[1] * c[1] + w[2] * c[2]) / (w[0] + w[1] + w[2])


def _redistribute(sp, mon, JU, J, x):
    """Displacement (with ghost layers) and Delta_tau of one mesh step."""
    d, h, N = sp["dim"], sp["dxi"], sp["nspec"]
    Js = torch.where(J[0] > 0, J[0], torch.ones_like(J[0]))
    rho, v, T = _prims(sp, JU, Js)
    rt = sum(rho)

    def central(s):
        ks = ["k%d" % k for k in range(d)]
        g = torch.sqrt(sum(((_at(sp, s, **{q: 1}) - _at(sp, s, **{q: -1})) / (2.0 * h[k])) ** 2
                           for k, q in enumerate(ks)))
        lap = sum((_at(sp, s, **{q: 1}) - 2.0 * _at(sp, s) + _at(sp, s, **{q: -1})) / h[k] ** 2
                  for k, q in enumerate(ks)).abs()
        return g, lap

    def variable(sig):
        if sig == 0:
            return rt
        if sig == 1:
            return rho[0]
        if sig == 2:
            return rho[N - 1]
        if sig == 3:
            return sum(_gas(sp)[l] * rho[l] for l in range(N)) * T - sum(sp["pinf"])
        if sig == 4:
            return torch.sqrt(sum(q * q for q in v))
        g, _ = central(rt)
        psi = (mon["psi"][0] * rho[0] + mon["psi"][1] * (rt - rho[0])) / rt if N == 2 else mon["psi"][0] + 0.0 * rt
        phi = torch.exp(-_at(sp, psi) * g / g.max()) if float(g.max()) > 0 else torch.ones_like(g)
        return _fill(sp, _pad(sp, phi.unsqueeze(0)))[0]

    th = 1.0
    for s, sig in enumerate(mon["sigma"]):
        g, lap = central(variable(sig))
        if float(g.max()) > 0:
            r = g / g.max()
            th = th + mon["alpha"][s] * (r if mon.get("form") else r * r)
        if mon.get("form") and float(lap.max()) > 0:
            th = th + mon["beta"][s] * lap / lap.max()
    th = _fill(sp, _pad(sp, torch.sqrt(th + torch.zeros_like(_at(sp, rt))).unsqueeze(0)))
    for _ in range(mon["n_smooth"]):
        f = th
        for k in range(d):
            ax = f.dim() - 1 - k
            n = f.shape[ax] - 2
            f = 0.25 * f.narrow(ax, 0, n) + 0.5 * f.narrow(ax, 1, n) + 0.25 * f.narrow(ax, 2, n)
        for k in range(d):
            f = f.narrow(f.dim() - 1 - k, NG - 1, sp["n"][k])
        th = _fill(sp, _pad(sp, f))
    xm = x
    for _ in range(mon["n_sweeps"]):
        num, den = 0.0, 0.0
        for k in range(d):
            for o in (1, -1):
                off = {"k%d" % k: o}
                t = 0.5 * (_at(sp, th) + _at(sp, th, **off)) / h[k] ** 2
                num, den = num + t * _at(sp, xm, **off), den + t
        xm = _fill(sp, _pad(sp, num / den), "mesh")
    dtau = torch.ones((), dtype=F64, device=x.device)
    for k in range(d):
        dx = _at(sp, xm[k]) - _at(sp, x[k])
        up = _at(sp, x[k], **{"k%d" % k: 1}) - _at(sp, x[k])
        dn = _at(sp, x[k]) - _at(sp, x[k], **{"k%d" % k: -1})
        b = torch.where(dx < 0, -dn / (2.0 * dx), torch.where(dx > 0, up / (2.0 * dx), torch.ones_like(dx)))
        dtau = torch.minimum(dtau, torch.where(dx == 0, torch.ones_like(b), b).min())
    disp = _fill(sp, _pad(sp, dtau * (_at(sp, xm) - _at(sp, x))), "disp")
    return disp, dtau.reshape(1)
