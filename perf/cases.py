"""Timing cases of the anisotropic diffusion library: what its users run,
through the public entry points (paper_1008_0861_amd.binding and .autograd).

A case is a dict of plain values.  Kinds of case:
  si        semi-implicit steps of one grid (2-D or 3-D; 2-step or 4-step)
  explicit  steps of the explicit limited scheme
  batch     independent uneven 2-D problems advanced together
  adjoint   forward and backward of the differentiable step map
"tune": the launch-shape autotuner runs once in prepare, as a long run of one
grid does; without it the default launch shapes run.
"stream": the grid lives on the program's side stream (calls of 64 steps or
more then replay a captured graph); else on torch's current stream.
"""
import math
import random

import torch

from paper_1008_0861_amd import autograd
from paper_1008_0861_amd import binding as asd

DTYPES = {"f32": torch.float32, "f64": torch.float64}
BATCH_SIDES = range(64, 513, 32)
MOST_CELLS = 8192 * 8192 * 2  # cell updates of the largest listed case (2 steps of 8192^2)


def _si(name, nx, ny, nz=0, **kw):
    c = dict(name=name, kind="si", nx=nx, ny=ny, nz=nz, dtype="f32", bc="periodic", limiter="vanleer", field="random",
             chi="const", chi_perp=0.0, ncfl=20.0, four_step=False, source=False, nsteps=1, energy=True, tune=False,
             stream=True)
    c.update(kw)
    return c


def listed():
    return [
        # one small step per call, as a program does that couples diffusion to
        # other physics step by step: launches and host work are what counts
        _si("ring-64-f64-one-step", 64, 64, dtype="f64", bc="insulating", field="ring", ncfl=10.0, energy=False,
            stream=False),
        # the ring test's whole run: 200 steps with the energy of each
        _si("ring-64-f64-200-steps", 64, 64, dtype="f64", bc="insulating", field="ring", ncfl=10.0, nsteps=200),
        # the smooth test with T = 0 walls and a source, odd side, towards its steady state
        _si("smooth-129-f64-walls-source", 129, 129, dtype="f64", bc="dirichlet", field="cosine", ncfl=1000.0,
            source=True, nsteps=100),
        # the headline workload of bench.py: 1024^2 random field, 20 steps, tuned
        _si("random-1024-f32-tuned", 1024, 1024, nsteps=20, tune=True),
        # the same grid in FP64 with a small chi_perp and default launch shapes
        _si("random-1024-f64", 1024, 1024, dtype="f64", chi_perp=1e-3, nsteps=10),
        # a ragged grid: no side a multiple of the wave, per-cell chi, another limiter, walls
        _si("ragged-1403x937-f32-chi-mc", 1403, 937, bc="insulating", limiter="mc", chi="cell", nsteps=10),
        # the large grids of bench.py
        _si("random-4096-f32", 4096, 4096, nsteps=4),
        _si("random-8192-f32-tuned", 8192, 8192, nsteps=2, tune=True),
        # 3-D, the 4-step scheme (the 2-step one's sweeps and a second solve in each direction)
        _si("curl-256cubed-f32-four-step", 256, 256, 256, ncfl=40.0, four_step=True, nsteps=4),
        # the explicit limited scheme in 3-D, the baseline of the method
        dict(name="explicit-256cubed-f32", kind="explicit", nx=256, ny=256, nz=256, dtype="f32", bc="periodic",
             limiter="vanleer", chi="const", chi_perp=0.0, ncfl=1.0, nsteps=8, energy=True),
        # 60 uneven problems advanced together, energies of every step
        dict(name="batch-60-f32", kind="batch", nprob=60, sides=40, dtype="f32", limiter="vanleer", ncfl=20.0,
             nsteps=10, energy=True),
        # gradient of a loss after 20 steps with respect to T0 and a per-cell chi (FP64: in FP32 a rounding
        # difference moves a few cells across a kink of the limiter, and their gradients with them)
        dict(name="adjoint-1024-f64", kind="adjoint", nx=1024, ny=1024, dtype="f64", ncfl=20.0, nsteps=20, every=10),
    ]


def _log_side(rng, lo, hi):
    n = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    return n | 1 if rng.random() < 0.3 else n


def draw(rng):
    kind = rng.choice(["si", "si", "si", "si3", "explicit", "batch", "adjoint"])
    dtype = rng.choice(["f32", "f32", "f64"])
    if kind == "si":
        hi = 8192 if dtype == "f32" else 4096
        nx = _log_side(rng, 16, hi)
        ny = nx if rng.random() < 0.4 else _log_side(rng, max(16, nx // 8), min(hi, 8 * nx))
        steps = max(1, min(rng.choice([1, 4, 20, 100]), MOST_CELLS // (2 * nx * ny)))
        bc = rng.choice(["periodic", "periodic", "insulating", "dirichlet"])
        c = _si("", nx, ny, dtype=dtype, bc=bc, field="cosine" if bc == "dirichlet" else "random",
                limiter=rng.choice(["vanleer", "vanleer", "minmod", "mc"]), chi=rng.choice(["const", "const", "cell"]),
                chi_perp=rng.choice([0.0, 1e-3]), ncfl=rng.choice([10.0, 20.0, 100.0]), source=bc == "dirichlet",
                nsteps=steps, energy=rng.random() < 0.6, tune=rng.random() < 0.3, stream=rng.random() < 0.7)
    elif kind == "si3":
        nx, ny, nz = (_log_side(rng, 24, 300) for _ in range(3))
        four = rng.random() < 0.5
        c = _si("", nx, ny, nz, dtype=dtype, bc=rng.choice(["periodic", "insulating"]), four_step=four,
                ncfl=40.0 if four else 10.0, nsteps=rng.choice([1, 3]), energy=rng.random() < 0.6,
                tune=rng.random() < 0.3)
    elif kind == "explicit":
        nz = _log_side(rng, 24, 256) if rng.random() < 0.5 else 0
        hi = 256 if nz else 4096
        nx, ny = _log_side(rng, 24, hi), _log_side(rng, 24, hi)
        c = dict(kind="explicit", nx=nx, ny=ny, nz=nz, dtype=dtype, bc=rng.choice(["periodic", "insulating"]),
                 limiter="vanleer", chi=rng.choice(["const", "cell"]), chi_perp=0.0, ncfl=1.0,
                 nsteps=rng.choice([4, 10]), energy=rng.random() < 0.6)
    elif kind == "batch":
        c = dict(kind="batch", nprob=rng.randint(8, 96), sides=rng.randrange(1000), dtype=dtype, limiter="vanleer",
                 ncfl=20.0, nsteps=rng.choice([4, 10, 20]), energy=rng.random() < 0.6)
    else:
        c = dict(kind="adjoint", nx=_log_side(rng, 64, 1400), ny=_log_side(rng, 64, 1400), dtype="f64", ncfl=20.0,
                 nsteps=rng.choice([6, 12]), every=rng.choice([3, 6, 10]))
    c.pop("name", None)
    return c


_side = []


def _side_stream():
    """The program's one side stream."""
    if not _side:
        _side.append(torch.cuda.Stream())
    return _side[0]


# ------------------------------------------------------------------ inputs
def _dev():
    return "cuda" if torch.cuda.is_available() else "cpu"


def _gen(seed, salt):
    return torch.Generator().manual_seed(1_000_003 * int(seed) + salt)


def _centres(n):
    return (torch.arange(n, dtype=torch.float64, device=_dev()) + 0.5) / n


def _potential_gradient(shape, k2, gen):
    """Gradient (x, y[, z] order) at the cell centres of a random potential
    with Gaussian amplitudes on the integer modes 1 <= |m|^2 <= k2."""
    nd, k = len(shape), int(math.isqrt(k2))
    m = torch.arange(-k, k + 1, dtype=torch.float64)
    grids = torch.meshgrid(*([m] * nd), indexing="ij")
    m2 = sum(g * g for g in grids)
    amp = torch.randn(m2.shape + (2,), generator=gen, dtype=torch.float64)
    amp = torch.view_as_complex(amp) * ((m2 >= 1) & (m2 <= k2))
    out = []
    for axis in range(nd):  # axis of the arrays: the last is x
        a = (amp * 2j * math.pi * grids[axis]).to(_dev())
        for q in range(nd):
            e = torch.exp(2j * math.pi * _centres(shape[q])[:, None] * m.to(_dev())[None, :])
            a = torch.movedim(torch.movedim(a, q, -1) @ e.T, -1, q)
        out.append(a.real.contiguous())
    return out[::-1]


def _unit(comps):
    mag = torch.sqrt(sum(c * c for c in comps))
    ok = mag > 1e-12 * mag.max()
    return [torch.where(ok, c / torch.where(ok, mag, torch.ones_like(mag)), torch.zeros_like(c)) for c in comps]


def _smoothed(shape, gen, sigma=4.0):
    """Unit-variance noise smoothed over sigma cells (periodic)."""
    spec = torch.fft.fftn(torch.randn(shape, generator=gen, dtype=torch.float64).to(_dev()))
    for q, n in enumerate(shape):
        f = torch.fft.fftfreq(n, dtype=torch.float64, device=_dev())
        spec *= torch.exp(-2.0 * math.pi ** 2 * sigma ** 2 * f * f).reshape([-1 if a == q else 1 for a in range(len(shape))])
    g = torch.fft.ifftn(spec).real
    g = g - g.mean()
    return g / g.std()


def _blobs(ny, nx, gen):
    """1 + 0.5 * eight tanh-edged blobs on the periodic unit square."""
    T = torch.ones(ny, nx, dtype=torch.float64, device=_dev())
    x, y = _centres(nx)[None, :], _centres(ny)[:, None]
    for cx, cy, u in torch.rand(8, 3, generator=gen, dtype=torch.float64).tolist():
        dx, dy = (x - cx).abs(), (y - cy).abs()
        d = torch.hypot(torch.minimum(dx, 1 - dx), torch.minimum(dy, 1 - dy))
        T += 0.25 * (1.0 - torch.tanh((d - (0.05 + 0.15 * u)) / 0.01))
    return T


def _ring(n, gen):
    """Circular b on [-1, 1]^2 (b = 0 outside r = 1), a hot patch of 12 on 10."""
    x, y = 2 * _centres(n)[None, :] - 1, 2 * _centres(n)[:, None] - 1
    r = torch.hypot(x, y)
    inside = (r <= 1.0) & (r > 0)
    bx, by = (torch.where(inside, v / torch.where(inside, r, torch.ones_like(r)), torch.zeros_like(r)) for v in (-y + 0 * x, x + 0 * y))
    turn = 2 * math.pi * float(torch.rand(1, generator=gen, dtype=torch.float64))
    th = torch.remainder(torch.atan2(y, x) - turn, 2 * math.pi)
    hot = (r > 0.5) & (r < 0.7) & (th > 11 * math.pi / 12) & (th < 13 * math.pi / 12)
    return [bx, by], torch.where(hot, 12.0, 10.0).to(torch.float64)


def _cosine(ny, nx, gen):
    """T = 0 walls on [-0.5, 0.5]^2: b along the contours of psi = cos cos,
    source 2 pi^2 psi, and a start between zero and the steady state."""
    x, y = math.pi * (_centres(nx)[None, :] - 0.5), math.pi * (_centres(ny)[:, None] - 0.5)
    psi = torch.cos(x) * torch.cos(y)
    b = _unit([-torch.cos(x) * torch.sin(y), torch.sin(x) * torch.cos(y)])
    a = float(torch.rand(1, generator=gen, dtype=torch.float64))
    return b, a * psi * (1.0 + 0.2 * torch.sin(2 * x + 1.0)), 2 * math.pi ** 2 * psi


def _problem(case, seed):
    """Inputs of one grid in FP64: dict of b, T, chi, Q, h, dt and options."""
    nx, ny, nz = case["nx"], case["ny"], case.get("nz", 0)
    gen = _gen(seed, 17)
    shape = (nz, ny, nx) if nz else (ny, nx)
    kind = case.get("field", "random")
    h, Q = tuple(1.0 / n for n in reversed(shape)), None
    chi_par = 1.0
    if kind == "ring":
        b, T = _ring(nx, gen)
        h, chi_par = (2.0 / nx, 2.0 / ny), 0.01
    elif kind == "cosine":
        b, T, Q = _cosine(ny, nx, gen)
    elif nz:
        g = [_potential_gradient(shape, 36, gen) for _ in range(3)]
        b = _unit([g[2][1] - g[1][2], g[0][2] - g[2][0], g[1][0] - g[0][1]])
        T = torch.exp(0.3 * _smoothed(shape, gen))
    else:
        gx, gy = _potential_gradient(shape, 64, gen)
        b = _unit([gy, -gx])
        T = torch.exp(0.3 * _smoothed(shape, gen)) if case["kind"] == "adjoint" else _blobs(ny, nx, gen)
    chi = torch.exp(0.5 * _smoothed(shape, gen)) if case.get("chi") == "cell" or case["kind"] == "adjoint" else None
    dtype = DTYPES[case["dtype"]]
    if chi is not None:
        chi = chi.to(dtype)
        chi_par = float(chi.max())
    p = dict(shape=shape, h=h, dt=case["ncfl"] * min(h) ** 2 / (4.0 * chi_par), chi_par=chi_par, chi=chi,
             b=[c.to(dtype).contiguous() for c in b], T=T.to(dtype).contiguous(),
             Q=Q.to(dtype).contiguous() if case.get("source") and Q is not None else None)
    if case["kind"] == "explicit":  # inside the scheme's limits in 2-D and 3-D
        p["dt"] = case["ncfl"] * min(h) ** 2 / ((4.0 if not nz else 10.0) * chi_par)
    return p


def _batch_sides(case):
    r = random.Random(case["sides"])
    return [(r.choice(BATCH_SIDES), r.choice(BATCH_SIDES), r.uniform(0.1, 1.0)) for _ in range(case["nprob"])]


def _batch_problems(case, seed):
    """Problems of a batch; their T are views of one flat tensor (each starts
    on a multiple of 64 elements)."""
    dtype = DTYPES[case["dtype"]]
    sides = _batch_sides(case)
    starts, total = [], 0
    for nx, ny, _ in sides:
        starts.append(total)
        total += (nx * ny + 63) // 64 * 64
    flat = torch.zeros(total, dtype=dtype, device=_dev())
    out = []
    for i, (nx, ny, chi) in enumerate(sides):
        gen = _gen(seed, 1000 + i)
        gx, gy = _potential_gradient((ny, nx), 64, gen)
        b = [c.to(dtype).contiguous() for c in _unit([gy, -gx])]
        T = flat[starts[i]:starts[i] + nx * ny].view(ny, nx)
        T.copy_(_blobs(ny, nx, gen))
        h = (1.0 / nx, 1.0 / ny)
        out.append(dict(shape=(ny, nx), h=h, chi_par=chi, dt=case["ncfl"] * min(h) ** 2 / (4.0 * chi), T=T, bx=b[0],
                        by=b[1]))
    return out, flat


def prepare(case, seed):
    kind = case["kind"]
    own = _side_stream() if case.get("stream", True) else torch.cuda.current_stream()
    if kind == "batch":
        probs, flat = _batch_problems(case, seed)
        own.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(own):
            b = asd.Batch(probs, dtype=DTYPES[case["dtype"]], limiter=case["limiter"])
        # the schedule that advances all problems at once, one launch per sweep
        return dict(kind=kind, batch=b, flat=flat, nsteps=case["nsteps"], energy=case["energy"], stream=own)
    p = _problem(case, seed)
    own.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(own):
        g = asd.Grid(p["shape"], p["h"], bc=case.get("bc", "periodic"), dtype=DTYPES[case["dtype"]],
                     limiter=case.get("limiter", "vanleer"), chi_par=p["chi_par"], chi_perp=case.get("chi_perp", 0.0),
                     per_cell_chi=p["chi"] is not None, four_step=case.get("four_step", False))
        g.set_b(*p["b"])
        if p["Q"] is not None:
            g.set_field("Q", p["Q"])
        if kind == "adjoint":
            T0, chi = p["T"].requires_grad_(True), p["chi"].requires_grad_(True)
            lam = torch.exp(0.3 * _smoothed(p["shape"], _gen(seed, 29))).to(p["T"].dtype)
            return dict(kind=kind, grid=g, T0=T0, chi=chi, lam=lam, dt=p["dt"], nsteps=case["nsteps"],
                        every=case["every"], stream=own)
        if p["chi"] is not None:
            g.set_field("chi", p["chi"])
        g.set_field("T", p["T"])
        if case.get("tune"):
            g.tune(p["dt"])
        e = torch.empty(case["nsteps"] + 1, dtype=torch.float64, device="cuda") if case["energy"] else None
    return dict(kind=kind, grid=g, dt=p["dt"], nsteps=case["nsteps"], energy=e, stream=own)


def run(s):
    with torch.cuda.stream(s["stream"]):
        if s["kind"] == "si":
            s["grid"].step_semi_implicit(s["dt"], s["nsteps"], out=s["energy"])
            return s["grid"].T, s["energy"]
        if s["kind"] == "explicit":
            s["grid"].step_explicit(s["dt"], s["nsteps"], out=s["energy"])
            return s["grid"].T, s["energy"]
        if s["kind"] == "batch":
            e = s["batch"].step(s["nsteps"], mode=2, energy=s["energy"])
            return s["flat"], e
        TN = autograd.semi_implicit_steps(s["T0"], s["chi"], s["grid"], s["dt"], s["nsteps"], s["every"])
        gT, gchi = torch.autograd.grad(TN, (s["T0"], s["chi"]), s["lam"])
        return TN, gT, gchi


def work(case):
    """Every step reads the state and b (and chi, Q) once and writes the state
    once; a reverse step reads the two states, lambda, b and chi and updates
    lambda and the chi gradient.  Operations: about 50 per cell and sweep."""
    es = 4 if case["dtype"] == "f32" else 8
    if case["kind"] == "batch":
        cells, nd, vals = sum(nx * ny for nx, ny, _ in _batch_sides(case)), 2, 4
    else:
        nd = 3 if case.get("nz") else 2
        cells = case["nx"] * case["ny"] * max(1, case.get("nz", 0))
        vals = 2 + nd + (case.get("chi") == "cell") + bool(case.get("source"))
    per = cells * case["nsteps"]
    if case["kind"] == "adjoint":
        return {"bytes": per * es * (5 + 9), "flops": per * 2 * (50 + 150)}
    sweeps = nd * (2 if case.get("four_step") else 1)
    return {"bytes": per * es * vals, "flops": per * 50 * sweeps}


# ------------------------------------------------- the scheme in 64 bits
def _shift(U, dim, s, bc, odd=True):
    """U at the neighbour s cells along dim: wrap, mirror, or (T = 0 walls) the odd ghost."""
    if bc == "periodic":
        return torch.roll(U, -s, dim)
    edge = U.narrow(dim, U.shape[dim] - 1 if s > 0 else 0, 1)
    rest = U.narrow(dim, 1 if s > 0 else 0, U.shape[dim] - 1)
    ghost = -edge if bc == "dirichlet" and odd else edge
    return torch.cat([rest, ghost] if s > 0 else [ghost, rest], dim)


def _limit(kind, a, b):
    pos = a * b > 0
    zero = torch.zeros_like(a)
    if kind == "vanleer":
        return torch.where(pos, 2 * a * b / torch.where(pos, a + b, torch.ones_like(a)), zero)
    if kind == "minmod":
        return torch.where(pos, torch.where(a.abs() <= b.abs(), a, b), zero)
    m = torch.where((2 * a).abs() <= (2 * b).abs(), 2 * a, 2 * b)
    mean = 0.5 * (a + b)
    return torch.where(pos, torch.where(m.abs() <= mean.abs(), m, mean), zero)


def _solve_rows(lo, di, up, rhs):
    """Tridiagonal systems along the last axis by cyclic reduction without pivoting (lo[0] = up[-1] = 0)."""
    n, s = di.shape[-1], 1
    while s < n:
        am, bm, cm = (torch.nn.functional.pad(v[..., :-s], (s, 0), value=f) for v, f in ((lo, 0.0), (di, 1.0), (up, 0.0)))
        ap, bp, cp = (torch.nn.functional.pad(v[..., s:], (0, s), value=f) for v, f in ((lo, 0.0), (di, 1.0), (up, 0.0)))
        k1, k2 = lo / bm, up / bp
        rhs = [r - k1 * torch.nn.functional.pad(r[..., :-s], (s, 0)) - k2 * torch.nn.functional.pad(r[..., s:], (0, s)) for r in rhs]
        di, lo, up = di - k1 * cm - k2 * ap, -k1 * am, -k2 * cp
        s *= 2
    return [r / di for r in rhs]


def _solve_line(alpha, wall, r):
    """x of (I + sum_f alpha_f (e_c - e_c')(e_c - e_c')^T + wall) x = r along the
    last axis; alpha_f sits at its left cell, the last one couples to cell 0."""
    am = torch.roll(alpha, 1, -1)
    lo, up, di = -am, -alpha, 1 + alpha + am + wall
    wrap = alpha[..., -1:]
    # the wrap coupling as a rank-one term: A = B + wrap (e_0 - e_n)(e_0 - e_n)^T
    lo, up = torch.cat([torch.zeros_like(wrap), lo[..., 1:]], -1), torch.cat([up[..., :-1], torch.zeros_like(wrap)], -1)
    di = torch.cat([di[..., :1] - wrap, di[..., 1:-1], di[..., -1:] - wrap], -1)
    v = torch.zeros_like(r)
    v[..., 0], v[..., -1] = 1.0, -1.0
    x, z = _solve_rows(lo, di, up, [r, v])
    num, den = x[..., :1] - x[..., -1:], 1 + wrap * (z[..., :1] - z[..., -1:])
    return x - z * (wrap * num / den)


class _Solve(torch.autograd.Function):
    """The line solve with its derivative (the matrix is symmetric)."""

    @staticmethod
    def forward(ctx, alpha, wall, r):
        x = _solve_line(alpha, wall, r)
        ctx.save_for_backward(alpha, wall, x)
        return x

    @staticmethod
    def backward(ctx, gx):
        alpha, wall, x = ctx.saved_tensors
        mu = _solve_line(alpha, wall, gx)
        return -(mu - torch.roll(mu, -1, -1)) * (x - torch.roll(x, -1, -1)), None, mu


def _faces(p, d, bc, chi_perp, dt_n, dt):
    """alpha and the transverse betas of the faces after each cell along axis
    d (0 = x), and the walls' addition to the diagonal."""
    nd = len(p["shape"])
    dim = nd - 1 - d
    b = [0.5 * (c + _shift(c, dim, 1, bc, odd=False)) for c in p["b"]]
    chi = p["chi"]
    if chi is None:
        chif = torch.full_like(b[0], p["chi_par"])
    else:
        other = _shift(chi, dim, 1, bc, odd=False)
        chif = 2 * chi * other / (chi + other)
    h = p["h"]
    inside = torch.ones_like(b[0])
    wall = torch.zeros_like(b[0])
    if bc != "periodic":
        inside.narrow(dim, p["shape"][dim] - 1, 1).zero_()
    if bc == "dirichlet":
        own = chi if chi is not None else torch.full_like(b[0], p["chi_par"])
        aw = 2 * dt_n * (chi_perp + (own - chi_perp) * p["b"][d] ** 2) / h[d] ** 2
        for at in (0, p["shape"][dim] - 1):
            wall.narrow(dim, at, 1).add_(aw.detach().narrow(dim, at, 1))
    alpha = inside * dt_n * (chi_perp + (chif - chi_perp) * b[d] * b[d]) / h[d] ** 2
    beta = {t: inside * dt * (chif - chi_perp) * b[d] * b[t] / (h[d] * h[t]) for t in range(nd) if t != d}
    return alpha, beta, wall


def _flux(U, beta, d, bc, limiter):
    """Limited transverse fluxes through the faces after each cell along d."""
    nd = U.dim()
    F = 0.0
    for t, bt in beta.items():
        dim = nd - 1 - t
        s = _limit(limiter, _shift(U, dim, 1, bc) - U, U - _shift(U, dim, -1, bc))
        F = F + bt * _limit(limiter, _shift(s, nd - 1 - d, 1, bc), s)
    return F


def _implicit_steps(case, p, T, nsteps):
    bc, lim, nd = case.get("bc", "periodic"), case.get("limiter", "vanleer"), T.dim()
    four = case.get("four_step", False)
    dt = p["dt"]
    coef = [_faces(p, d, bc, case.get("chi_perp", 0.0), dt * (0.5 if four else 1.0), dt) for d in range(nd)]
    dv = math.prod(p["h"])
    energy = [T.detach().sum() * dv]
    for _ in range(nsteps):
        for d in range(nd):
            dim = nd - 1 - d
            alpha, beta, wall = coef[d]
            F = _flux(T, beta, d, bc, lim)
            r = T + F - torch.roll(F, 1, dim)
            if d == 0 and p.get("Q") is not None:
                r = r + dt * p["Q"]
            a, w, r = (torch.movedim(v, dim, -1) for v in (alpha, wall, r))
            x = _Solve.apply(a, w, r)
            if four:
                x = _Solve.apply(a, w, x)
            T = torch.movedim(x, -1, dim)
        energy.append(T.detach().sum() * dv)
    return T, torch.stack(energy)


def _explicit_steps(case, p, T, nsteps):
    bc, lim, nd, dt = case["bc"], case["limiter"], T.dim(), p["dt"]
    coef = [_faces(p, d, bc, case["chi_perp"], dt, dt) for d in range(nd)]
    dv = math.prod(p["h"])
    energy = [T.sum() * dv]
    for _ in range(nsteps):
        out = T.clone()
        for d in range(nd):
            dim = nd - 1 - d
            alpha, beta, _ = coef[d]
            F = _flux(T, beta, d, bc, lim) + alpha * (_shift(T, dim, 1, bc) - T)
            out += F - torch.roll(F, 1, dim)
        T = out
        energy.append(T.sum() * dv)
    return T, torch.stack(energy)


def exact(case, seed):
    """What run returns, the scheme stated in FP64 torch on the same inputs."""
    up = lambda v: None if v is None else v.double()  # noqa: E731
    if case["kind"] == "batch":
        probs, flat = _batch_problems(case, seed)
        out, energy = torch.zeros(flat.numel(), dtype=torch.float64, device=flat.device), []
        for q in probs:
            p = dict(shape=q["shape"], h=q["h"], dt=q["dt"], chi_par=q["chi_par"], chi=None, b=[up(q["bx"]), up(q["by"])])
            T, e = _implicit_steps(dict(case, bc="periodic"), p, up(q["T"]), case["nsteps"])
            at = q["T"].storage_offset()
            out[at:at + T.numel()] = T.reshape(-1)
            energy.append(e)
        return out, torch.stack(energy) if case["energy"] else None
    p = _problem(case, seed)
    p.update(b=[up(c) for c in p["b"]], chi=up(p["chi"]), Q=up(p["Q"]))
    if case["kind"] == "adjoint":
        T0, chi = up(p["T"]).requires_grad_(True), p["chi"].requires_grad_(True)
        p["chi"] = chi
        lam = torch.exp(0.3 * _smoothed(p["shape"], _gen(seed, 29))).to(p["T"].dtype).double()
        TN, _ = _implicit_steps(case, p, T0, case["nsteps"])
        gT, gchi = torch.autograd.grad(TN, (T0, chi), lam)
        return TN.detach(), gT, gchi
    step = _explicit_steps if case["kind"] == "explicit" else _implicit_steps
    T, e = step(case, p, up(p["T"]), case["nsteps"])
    return T, e if case["energy"] else None
