"""The framework's work, as cases that can be timed and compared.

A case is one pass through the public entry points of paper_2211_15716_amd on
a grid of (nx, ny, nz) points:

  step      igg.diffusion_step: one step of the time loop with its halo update
  run       nt steps: diffusion.forward ("driver": "forward") or
            igg.diffusion_run ("driver": "run", a captured graph)
  adjoint   one reverse step, Laplacian or staggered flux form
  flux      igg.diffusion_flux_step: cells, three face fields, their halo
  gradient  diffusion.loss_and_grad: forward sweep, loss, reverse sweep with
            time-loop checkpointing
  setup     what a program does before its loop: halo update of both fields,
            the stable time step, the conserved heat content

Overlaps are 2 (the default).  "periods" is written "xyz" as 0/1 digits, and
"split" is the boundary split (16, 2, 2) of the time loop or none.
"""
import math
import types

import torch

from paper_2211_15716_amd import diffusion, igg

DTYPE = {"f64": torch.float64, "f32": torch.float32, "f16": torch.float16}
SIZE = {"f64": 8, "f32": 4, "f16": 2}
LAM = 1.0
SPLIT = (16, 2, 2)
SR_SEED = 17


def _case(name, kind, n, dtype, periods="111", split=True, **more):
    return dict(name=name, kind=kind, nx=n[0], ny=n[1], nz=n[2], dtype=dtype, periods=periods, split=split, **more)


def listed():
    return [
        # the parity grid and smallest call: an interactive or test-sized
        # step, where the launches and the call itself are the cost
        _case("step_32_f64", "step", (32, 32, 32), "f64"),
        # a small study in the listing's default topology (no periods): the
        # whole time loop handed to the library as a graph
        _case("run_96_f64", "run", (96, 80, 64), "f64", periods="000", nt=50, driver="run"),
        # an ordinary grid whose sizes nobody rounded, periods mixed
        _case("step_odd_f32", "step", (301, 257, 203), "f32", periods="101"),
        # an ordinary time loop: the Python driver over 20 steps
        _case("run_256_f64", "run", (256, 256, 256), "f64", nt=20, driver="forward"),
        # the benchmark's grid in its three precisions
        _case("step_512_f64", "step", (512, 512, 512), "f64"),
        _case("step_512_f32", "step", (512, 512, 512), "f32"),
        _case("step_512_f16", "step", (512, 512, 512), "f16", stochastic=True),
        # one reverse step of the inverse problem
        _case("adjoint_256_f64", "adjoint", (256, 256, 256), "f64", form="laplacian"),
        # the same for the flux form, ragged sizes, no split
        _case("adjoint_flux_odd_f32", "adjoint", (255, 190, 131), "f32", form="flux", split=False),
        # the largest grid: staggered form, four output fields
        _case("flux_768_f32", "flux", (768, 768, 768), "f32", split=False),
        # the inverse problem as a whole: 200 steps, snapshot every 16
        _case("gradient_256_f64", "gradient", (256, 256, 256), "f64", nt=200, schedule="periodic", arg=16),
        # before the loop: halos, time step, conserved sum
        _case("setup_256_f64", "setup", (256, 250, 241), "f64"),
    ]


def _edge(rng, lo, hi):
    """An edge spread over the logarithm of its range; half of them rounded
    to a multiple of 8, the others as they fall."""
    e = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    if rng.random() < 0.5:
        e = max(lo, e // 8 * 8)
    return e


def draw(rng):
    kind = rng.choice(["step", "step", "step", "run", "run", "adjoint", "adjoint", "flux", "gradient", "setup"])
    lo, hi, most = {"step": (32, 512, 1 << 27), "run": (32, 320, 1 << 24), "adjoint": (48, 400, 1 << 26),
                    "flux": (48, 640, 1 << 27), "gradient": (32, 200, 1 << 23), "setup": (48, 400, 1 << 26)}[kind]
    while True:
        n = tuple(_edge(rng, lo, hi) for _ in range(3))
        if n[0] * n[1] * n[2] <= most:
            break
    dtype = rng.choice(["f64", "f32", "f16"] if kind in ("step", "run") else ["f64", "f32"])
    periods = "111" if rng.random() < 0.6 else rng.choice(["000", "100", "011", "101"])
    c = dict(kind=kind, nx=n[0], ny=n[1], nz=n[2], dtype=dtype, periods=periods, split=rng.random() < 0.7)
    if kind in ("step", "run") and dtype == "f16":
        c["stochastic"] = rng.random() < 0.8
    if kind == "run":
        c["nt"] = rng.randint(8, 64)
        # graph replays would repeat the stochastic-rounding counter
        c["driver"] = "forward" if c.get("stochastic") else rng.choice(["forward", "run"])
    if kind == "adjoint":
        c["form"] = rng.choice(["laplacian", "flux"])
    if kind == "gradient":
        c["nt"] = rng.randint(10, 100)
        c["schedule"], c["arg"] = rng.choice([("periodic", 16), ("periodic", 8), ("sqrt", 0), ("binomial", 8)])
    return c


# ------------------------------------------------------------------ inputs
def _spacings(case):
    return tuple(1.0 / (case[k] - 1) for k in ("nx", "ny", "nz"))


def _periods(case):
    return tuple(int(c) for c in case["periods"])


def _split(case):
    if not case["split"]:
        return None
    # the flux form's faces need one more plane than the cells
    flux = case["kind"] == "flux" or case.get("form") == "flux"
    return tuple(max(w, 3) for w in SPLIT) if flux else SPLIT


def _raw(case, seed):
    """The seed's fields in the case's type, halo planes not yet updated: a
    noisy bump T, Ci = U(0.5, 1.5)/2, and for the reverse step an adjoint
    state."""
    dev = "cuda"
    g = torch.Generator(device=dev)
    g.manual_seed(1000003 * seed + 11)
    shape = (case["nz"], case["ny"], case["nx"])
    work = torch.float32 if case["dtype"] == "f32" else torch.float64
    ax = [torch.linspace(0, 1, m, dtype=work, device=dev) - 0.5 for m in shape]
    e = [torch.exp(-a * a / 0.01) for a in ax]
    t = DTYPE[case["dtype"]]
    T = torch.randn(shape, dtype=work, device=dev, generator=g).mul_(1e-3).add_(1.7)
    T += e[0][:, None, None] * e[1][None, :, None] * e[2][None, None, :]
    Ci = torch.rand(shape, dtype=work, device=dev, generator=g).add_(0.5).mul_(0.5)
    out = [T.to(t), Ci.to(t)]
    if case["kind"] in ("adjoint", "gradient"):
        # a residual for the adjoint state, an observed state for the loss
        X = torch.randn(shape, dtype=work, device=dev, generator=g).mul_(1e-2)
        out.append((X if case["kind"] == "adjoint" else X + 1.7).to(t))
    return out


def _zero_fixed(A, periods):
    """Zero on the halo planes of the dimensions without a period."""
    for d, p in zip((2, 1, 0), periods):
        if not p:
            A.select(d, 0).zero_()
            A.select(d, A.shape[d] - 1).zero_()


def _grid(case):
    """The process's global grid for this case (kept where it fits)."""
    n, periods = (case["nx"], case["ny"], case["nz"]), _periods(case)
    try:
        topo = igg.topology()
    except igg.IggError:
        topo = None
    if topo is not None and topo["n"] == n and topo["periods"] == periods:
        return
    if topo is not None:
        torch.cuda.synchronize()
        igg.finalize_global_grid()
    igg.init_global_grid(*n, periods=periods)


def prepare(case, seed):
    _grid(case)
    s = types.SimpleNamespace(case=case, d=_spacings(case), split=_split(case), T2=None, rnd=None)
    fields = _raw(case, seed)
    s.T, s.Ci = fields[0], fields[1]
    if case["kind"] == "setup":
        return s
    igg.update_halo(s.T, s.Ci)
    s.dt = igg.diffusion_dt(s.Ci, LAM, *s.d)
    if case["kind"] in ("step", "run", "flux"):
        s.T2 = s.T.clone()
    if case.get("stochastic"):
        s.rnd = igg.rounding("stochastic", SR_SEED, 5)
    if case["kind"] == "flux":
        s.q = diffusion.FluxProblem.face_arrays(s.T)
    if case["kind"] == "adjoint":
        s.lp = fields[2]
        _zero_fixed(s.lp, _periods(case))
        igg.update_halo(s.lp)
        s.ln, s.gCi = torch.zeros_like(s.lp), torch.zeros_like(s.lp)
    if case["kind"] == "gradient":
        s.T_obs = fields[2]
        s.prob = diffusion.Problem(LAM, s.dt, *s.d, split=s.split)
        s.schedule = (case["schedule"], case["arg"]) if case["arg"] else (case["schedule"],)
    return s


def run(s):
    c = s.case
    kind = c["kind"]
    if kind == "step":
        igg.diffusion_step(s.T2, s.T, s.Ci, LAM, s.dt, *s.d, split=s.split, rnd=s.rnd)
        return s.T2
    if kind == "run":
        if c["driver"] == "forward":
            out = diffusion.forward(s.T, s.Ci, c["nt"], LAM, s.dt, *s.d, split=s.split, work=s.T2,
                                    sr_seed=SR_SEED if c.get("stochastic") else None)
        else:
            out = igg.diffusion_run(s.T, s.T2, s.Ci, LAM, s.dt, *s.d, c["nt"], split=s.split, rnd=s.rnd)
        if out is s.T2:  # the next pass goes on from here
            s.T, s.T2 = s.T2, s.T
        return out
    if kind == "adjoint":
        step = igg.diffusion_flux_step_adjoint if c["form"] == "flux" else igg.diffusion_step_adjoint
        step(s.ln, s.lp, s.T, s.Ci, s.gCi, LAM, s.dt, *s.d, split=s.split)
        return s.ln, s.gCi
    if kind == "flux":
        igg.diffusion_flux_step(s.T2, s.T, s.Ci, *s.q, LAM, s.dt, *s.d, split=s.split)
        return [s.T2] + list(s.q)
    if kind == "gradient":
        L, gT0, gCi, _ = diffusion.loss_and_grad(s.T, s.Ci, s.T_obs, s.prob, c["nt"], s.schedule)
        return L, gT0, gCi
    igg.update_halo(s.T, s.Ci)
    dt = igg.diffusion_dt(s.Ci, LAM, *s.d)
    heat = igg.reduce(igg.RED_SUM_RATIO, s.T, s.Ci)
    return s.T, s.Ci, dt, heat


def work(case):
    nx, ny, nz = case["nx"], case["ny"], case["nz"]
    e, pts = SIZE[case["dtype"]], nx * ny * nz
    kind = case["kind"]
    if kind == "step":
        return {"bytes": 3 * e * pts, "flops": 17 * pts}
    if kind == "run":
        return {"bytes": 3 * e * pts, "flops": 17 * pts * case["nt"]}
    if kind == "adjoint":
        return {"bytes": 6 * e * pts, "flops": 34 * pts}
    if kind == "flux":
        return {"bytes": 6 * e * pts, "flops": 21 * pts}
    if kind == "gradient":
        return {"bytes": 5 * e * pts, "flops": (17 + 34) * pts * case["nt"]}
    faces = 2 * (nx * ny + ny * nz + nx * nz)
    return {"bytes": 2 * e * pts + 2 * 2 * e * faces, "flops": 3 * pts}


# ------------------------------------------------------- 64-bit reference
def _halo(A, case):
    """Halo update of a field of the case's grid (n or n+1 points)."""
    n = (case["nx"], case["ny"], case["nz"])
    for d, p in enumerate(_periods(case)):
        if not p:
            continue
        t = 2 - d
        m = A.shape[t]
        ol = 2 + m - n[d]
        lo, hi = A.select(t, ol - 1).clone(), A.select(t, m - ol).clone()
        A.select(t, m - 1).copy_(lo)
        A.select(t, 0).copy_(hi)
    return A


def _lap(A, d):
    c = A[1:-1, 1:-1, 1:-1]
    out = (A[1:-1, 1:-1, 2:] - c - (c - A[1:-1, 1:-1, :-2])) / d[0] ** 2
    out += (A[1:-1, 2:, 1:-1] - c - (c - A[1:-1, :-2, 1:-1])) / d[1] ** 2
    out += (A[2:, 1:-1, 1:-1] - c - (c - A[:-2, 1:-1, 1:-1])) / d[2] ** 2
    return out


def _inner(A):
    return A[1:-1, 1:-1, 1:-1]


def _step(T, Ci, dt, case):
    out = T.clone()
    _inner(out).add_(_lap(T, _spacings(case)).mul_(_inner(Ci)).mul_(dt * LAM))
    return _halo(out, case)


def _reverse(lp, T, Ci, g, dt, case):
    d = _spacings(case)
    ln = torch.zeros_like(lp)
    _inner(ln).copy_(_inner(lp) + dt * LAM * _lap(Ci * lp, d))
    _inner(g).add_(_lap(T, d).mul_(_inner(lp)).mul_(dt * LAM))
    return _halo(ln, case)


def exact(case, seed):
    f = [x.double() for x in _raw(case, seed)]
    kind = case["kind"]
    T, Ci = _halo(f[0], case), _halo(f[1], case)
    d = _spacings(case)
    m = float(Ci.max())
    dt = min(v * v for v in d) / LAM / m / 6.1
    if kind == "setup":
        return T, Ci, dt, float((_inner(T) / _inner(Ci)).sum())
    if kind == "step":
        return _step(T, Ci, dt, case)
    if kind == "run":
        for _ in range(case["nt"]):
            T = _step(T, Ci, dt, case)
        return T
    if kind == "adjoint":
        lp = f[2]
        _zero_fixed(lp, _periods(case))
        _halo(lp, case)
        g = torch.zeros_like(lp)
        # the flux form's adjoint is the Laplacian form's on this grid
        return _reverse(lp, T, Ci, g, dt, case), g
    if kind == "flux":
        q = _faces(T, d)
        out = T.clone()
        div = (q[0][1:-1, 1:-1, 2:-1] - q[0][1:-1, 1:-1, 1:-2]) / d[0]
        div += (q[1][1:-1, 2:-1, 1:-1] - q[1][1:-1, 1:-2, 1:-1]) / d[1]
        div += (q[2][2:-1, 1:-1, 1:-1] - q[2][1:-2, 1:-1, 1:-1]) / d[2]
        _inner(out).sub_(div.mul_(_inner(Ci)).mul_(dt))
        return [_halo(a, case) for a in [out] + q]
    states = [T]
    for _ in range(case["nt"]):
        states.append(_step(states[-1], Ci, dt, case))
    lam = torch.zeros_like(T)
    _inner(lam).copy_(_inner(states.pop()) - _inner(f[2]))
    L = float(0.5 * (lam * lam).sum())
    _halo(lam, case)
    g = torch.zeros_like(T)
    while states:
        lam = _reverse(lam, states.pop(), Ci, g, dt, case)
    grads = torch.zeros_like(T), torch.zeros_like(T)
    _inner(grads[0]).copy_(_inner(lam))
    _inner(grads[1]).copy_(_inner(g))
    return (L,) + grads


def _faces(T, d):
    """Face fluxes -lam*grad(T) on the faces 1..n-1 of the inner rows, zero
    elsewhere."""
    nz, ny, nx = T.shape
    q = [torch.zeros(s, dtype=T.dtype, device=T.device) for s in ((nz, ny, nx + 1), (nz, ny + 1, nx), (nz + 1, ny, nx))]
    q[0][1:-1, 1:-1, 1:-1] = -LAM * (T[1:-1, 1:-1, 1:] - T[1:-1, 1:-1, :-1]) / d[0]
    q[1][1:-1, 1:-1, 1:-1] = -LAM * (T[1:-1, 1:, 1:-1] - T[1:-1, :-1, 1:-1]) / d[1]
    q[2][1:-1, 1:-1, 1:-1] = -LAM * (T[1:, 1:-1, 1:-1] - T[:-1, 1:-1, 1:-1]) / d[2]
    return q
