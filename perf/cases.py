"""The work that users of this library have it do, as cases that can be timed and checked.

A case is a plain dict: an operation (``op``), its sizes, its precision and its options.
``prepare`` makes what a program holds before the call (device arrays, a step state, a captured
graph), ``run`` makes one call through the public binding, ``work`` counts the bytes and
operations that the call cannot do without and ``exact`` evaluates the same quantity in plain
float64 torch.  The configurations are the sheets of ``paper_1612_00474_amd.workloads`` (uniform
heights above the wall, projected area fraction 0.4, reduced units) with sizes from 256 to
262,144 spheres.

Operations:
  matvec    U = M F + M_C T (``torque``: with the second term; ``box``: pseudo-periodic in x, y)
  lanczos   M^{1/2} W to a relative tolerance
  multi     M^{1/2} W for several noise vectors of one configuration
  step      one stochastic Adams-Bashforth step of one suspension, noise drawn on the device
  batch     one graph-captured step of many independent suspensions of uneven size
"""
import math

import numpy as np
import torch

from paper_1612_00474_amd import Context, StepState
from paper_1612_00474_amd import workloads as wl

Z_LO, Z_HI = 1.1, 2.5
DT, DELTA = 0.01, 1e-4
F_GRAV, TORQUE, U0, B = -1.0, (0.0, 1.0, 0.0), 1.0, 0.1
STEP = dict(dt=DT, delta=DELTA, f_grav_z=F_GRAV, torque=TORQUE, steric_u0=U0, steric_b=B)
GRAPH_BUDGET = 16          # Lanczos iterations that a captured step enqueues

_contexts = {}


def _context(box=None):
    """The program's context (one for the unbounded wall, one per periodic box)."""
    if box is not None:
        return Context(0, box=box)
    if None not in _contexts:
        _contexts[None] = Context(0)
    return _contexts[None]


def listed():
    return [
        # One product of a small, dense-checkable sheet: the smallest call, where launches count.
        dict(name="matvec_fp64_256", op="matvec", n=256, precision="fp64", torque=True, box=False),
        # A product of an ordinary suspension of no round size, in float64.
        dict(name="matvec_fp64_4099", op="matvec", n=4099, precision="fp64", torque=True,
             box=False),
        # Forces alone in a pseudo-periodic box (nine images per pair), ragged size.
        dict(name="matvec_box_mixed_8191", op="matvec", n=8191, precision="mixed", torque=False,
             box=True),
        # A product of the largest sheet that the benchmark names.
        dict(name="matvec_mixed_262144", op="matvec", n=262144, precision="mixed", torque=True,
             box=False),
        # The Brownian increment of the small sheet to a tight tolerance: many cheap iterations.
        dict(name="lanczos_fp64_256", op="lanczos", n=256, precision="fp64", tol=1e-6),
        # The Brownian increment of a sheet of 2^15 rollers, the size of the paper's runs.
        dict(name="lanczos_mixed_32768", op="lanczos", n=32768, precision="mixed", tol=1e-3),
        # Four independent increments of one configuration.
        dict(name="multi_fp64_1100x4", op="multi", n=1100, nvec=4, precision="fp64", tol=1e-3),
        # Time stepping of the small sheet (noise, forces, products, Lanczos, drift, update).
        dict(name="step_fp64_256", op="step", n=256, precision="fp64", tol=1e-6),
        # Time stepping of a ragged suspension of a few thousand spheres.
        dict(name="step_fp64_2100", op="step", n=2100, precision="fp64", tol=1e-3),
        # Time stepping in float64 at the size of the long float64 runs.
        dict(name="step_fp64_16384", op="step", n=16384, precision="fp64", tol=1e-3),
        # Time stepping in mixed precision at the benchmark's size.
        dict(name="step_mixed_65536", op="step", n=65536, precision="mixed", tol=1e-3),
        # 64 independent suspensions of 1,024 to 8,192 spheres, one graph launch per step.
        dict(name="batch_mixed_64", op="batch", nsys=64, n_lo=1024, n_hi=8192, precision="mixed",
             tol=1e-3),
    ]


def _size(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["matvec", "matvec", "matvec", "lanczos", "lanczos", "multi", "step", "step",
                     "step", "batch"])
    precision = rng.choice(["fp64", "mixed"])
    if op == "matvec":
        box = rng.random() < 0.25
        top = 16384 if box else (131072 if precision == "mixed" else 65536)
        return dict(op=op, n=_size(rng, 256, top), precision=precision,
                    torque=rng.random() < 0.6, box=box)
    if op == "lanczos":
        return dict(op=op, n=_size(rng, 256, 32768), precision=precision,
                    tol=rng.choice([1e-3, 1e-4]))
    if op == "multi":
        return dict(op=op, n=_size(rng, 256, 8192), nvec=rng.randint(2, 6), precision=precision,
                    tol=1e-3)
    if op == "step":
        return dict(op=op, n=_size(rng, 256, 32768), precision=precision, tol=1e-3)
    lo = _size(rng, 64, 1024)
    return dict(op=op, nsys=_size(rng, 4, 64), n_lo=lo, n_hi=_size(rng, 2 * lo, 4096),
                precision=precision, tol=1e-3)


# ---- inputs -----------------------------------------------------------------------------------


def _positions(n, seed):
    if n == 256:   # the small dense sheet: no two centres closer than 2.05
        return wl.sample_positions(n, 32.0, Z_LO, 3.0, 2.05, seed=seed)
    return wl.sheet(n, Z_LO, Z_HI, seed=seed)


def _sizes(case):
    """The systems' sizes: those of the case, whatever the seed."""
    return [int(k) for k in wl.batch_sizes(
        wl.Workload("batch", 0, 0.0, Z_LO, Z_HI, nsys=case["nsys"], n_lo=case["n_lo"],
                    n_hi=case["n_hi"]))]


def _batch(case, seed):
    """Concatenated positions of the batch's sheets and their offsets."""
    sizes = _sizes(case)
    pos = np.vstack([wl.sheet(n, Z_LO, Z_HI, seed=seed * len(sizes) + s)
                     for s, n in enumerate(sizes)])
    return pos, np.concatenate([[0], np.cumsum(sizes)])


def _inputs(case, seed):
    """Positions and vectors of a single-system case on the GPU."""
    n = case["n"]
    pos = torch.from_numpy(_positions(n, seed)).cuda()
    gen = torch.Generator(device="cuda").manual_seed(seed + 1)
    k = case.get("nvec", 2)
    vec = torch.randn((k, n, 3), generator=gen, dtype=torch.float64, device="cuda")
    return pos, vec


def _box(case):
    side = wl.side_for_area_fraction(case["n"], wl.PHI)
    return (side, side)


def prepare(case, seed):
    op = case["op"]
    if op == "batch":
        pos, offs = _batch(case, seed)
        pos = torch.from_numpy(pos).cuda()
        u = torch.zeros_like(pos)
        graph = _context().step_graph(pos, u, offs, lanczos_tol=case["tol"], seed=seed,
                                      lanczos_max_iter=GRAPH_BUDGET, precision=case["precision"],
                                      **STEP)
        return dict(case=case, graph=graph, pos=pos, u=u)
    pos, vec = _inputs(case, seed)
    s = dict(case=case, ctx=_context(_box(case) if case.get("box") else None), seed=seed)
    if op == "step":
        s["state"] = StepState(pos)
    else:
        s.update(pos=pos, vec=vec)
    return s


def run(s):
    case = s["case"]
    op = case["op"]
    if op == "batch":
        s["graph"].launch()
        return s["pos"], s["u"]
    ctx, precision = s["ctx"], case["precision"]
    if op == "matvec":
        return ctx.matvec(s["pos"], s["vec"][0], s["vec"][1] if case["torque"] else None,
                          precision)
    if op == "lanczos":
        g, m, eps, _ = ctx.lanczos(s["pos"], s["vec"][0], case["tol"], precision=precision)
        return g, m, eps
    if op == "multi":
        g, m, eps, _ = ctx.lanczos_multi(s["pos"], s["vec"], case["tol"], precision=precision)
        return g, m, eps
    st = s["state"]
    m, eps, _ = ctx.sab_step(st, lanczos_tol=case["tol"], seed=s["seed"], precision=precision,
                             **STEP)
    return st.pos, st.u_prev, m, eps


# ---- what a call cannot do without ------------------------------------------------------------

# Operations per unordered pair (fused multiply-add = 2): the coefficients once (77) and a force
# applied in both directions (40); both torque couplings 77 more.
COEF, APPLY, COUPLE = 77, 40, 77


def _iterations(tol):
    """Krylov iterations that the sheets need (measured: 11-12 at 1e-3, 25 at 1e-6)."""
    return {1e-3: 12, 1e-4: 22, 1e-6: 25}[tol]


def _pairs(n):
    return n * (n + 1) / 2


def _step_flops(n, m):
    joint = COEF + 2 * APPLY + COUPLE            # M F + M_C T and M W
    return _pairs(n) * (joint + (m - 1 + 2) * (COEF + APPLY))


def work(case):
    op = case["op"]
    if op == "batch":
        sizes = _sizes(case)
        return {"bytes": 4 * 24 * sum(sizes),
                "flops": sum(_step_flops(n, _iterations(case["tol"])) for n in sizes)}
    n = case["n"]
    if op == "matvec":
        per = COEF + APPLY + (COUPLE if case["torque"] else 0)
        return {"bytes": 24 * n * (4 if case["torque"] else 3),
                "flops": _pairs(n) * per * (9 if case["box"] else 1)}
    m = _iterations(case["tol"])
    if op == "lanczos":
        return {"bytes": 24 * n * 3, "flops": _pairs(n) * m * (COEF + APPLY)}
    if op == "multi":
        k = case["nvec"]
        return {"bytes": 24 * n * (1 + 2 * k), "flops": _pairs(n) * m * (COEF + k * APPLY)}
    return {"bytes": 24 * n * 4, "flops": _step_flops(n, m)}


# ---- the same quantities in plain float64 torch -----------------------------------------------


def _rows(pos, force, torque, i0, i1, shift=(0.0, 0.0), box=None):
    """Rows i0..i1 of 8 pi eta (M F + M_C T) for the image of the sources shifted by `shift`
    (units a = 1): the unbounded Rotne-Prager tensors and the image part of the no-slip wall."""
    h = pos[:, 2].clamp(0.0, 1.0)
    z = pos[:, 2].clamp(min=1.0)
    dx = pos[i0:i1, 0, None] - pos[None, :, 0]
    dy = pos[i0:i1, 1, None] - pos[None, :, 1]
    if box is not None:
        dx = dx - box[0] * torch.round(dx / box[0]) + shift[0]
        dy = dy - box[1] * torch.round(dy / box[1]) + shift[1]
    zj = z[None, :]
    dz = z[i0:i1, None] - zj
    rz = z[i0:i1, None] + zj
    rho2 = dx * dx + dy * dy
    r = (rho2 + dz * dz).sqrt()
    far = r >= 2.0
    rs = r.clamp(min=2.0)
    near = (1.0 / r).masked_fill(r == 0.0, 0.0)
    ci = torch.where(far, (1.0 + 2.0 / (3.0 * rs * rs)) / rs, 4.0 / 3.0 - 0.375 * r)
    crr = torch.where(far, (1.0 - 2.0 / (rs * rs)) / rs ** 3, near / 8.0)
    inv = 1.0 / (rho2 + rz * rz).sqrt()
    e, x, q = rz * inv, inv * inv, zj * inv
    y, e2 = x * x, e * e
    c1 = -1 + x * (2 * e2 - 2 / 3) + y * (2 / 3 - 10 / 3 * e2) - 2 * e * q + 2 * q * q
    c2 = -1 + x * (2 - 10 * e2) + y * (70 / 3 * e2 - 10 / 3) + 6 * e * q - 6 * q * q
    c3 = (q * (2 - 12 * e2) + 12 * e * q * q + x * (20 * e2 * e - 4 * e) +
          y * (40 / 3 * e - 140 / 3 * e2 * e))
    c4 = 2 * q - 20 / 3 * y * e
    c5 = -4 * q * q - 4 * x * e2 + y * (20 * e2 - 8 / 3)
    ux = uy = uz = 0.0
    if force is not None:
        f = force * h[:, None]
        fx, fy, fz = f[None, :, 0], f[None, :, 1], f[None, :, 2]
        s = dx * fx + dy * fy
        rf = crr * (s + dz * fz)
        ef = (s + rz * fz) * inv
        along = inv * (c2 * ef + c3 * fz)            # times e
        up = inv * (c4 * ef + c5 * fz)               # times z
        a = ci + inv * c1
        ux = (a * fx + (rf + along * inv) * dx).sum(1)
        uy = (a * fy + (rf + along * inv) * dy).sum(1)
        uz = (a * fz + rf * dz + along * e + up).sum(1)
    if torque is not None:
        t = torque * h[:, None]
        tx, ty, tz = t[None, :, 0], t[None, :, 1], t[None, :, 2]
        ct = torch.where(far, 1.0 / rs ** 3, 0.5 - 3.0 / 16.0 * r)
        ex, ey = dx * inv, dy * inv
        d2 = 2 * x * e + 2 * q
        d3 = 10 * x * e - 6 * e + 6 * q
        w = ey * tx - ex * ty                        # (e x z) . T
        ux = ux + (ct * (ty * dz - tz * dy) + x * (ey * tz - e * ty + d2 * ty + d3 * ex * w)).sum(1)
        uy = uy + (ct * (tz * dx - tx * dz) + x * (e * tx - ex * tz - d2 * tx + d3 * ey * w)).sum(1)
        uz = uz + (ct * (tx * dy - ty * dx) +
                   x * (ex * ty - ey * tx + (d3 * e - 2 * x) * w)).sum(1)
    return torch.stack([ux, uy, uz], 1) * h[i0:i1, None]


def _product(pos, force, torque=None, box=None):
    n = pos.shape[0]
    out = torch.zeros_like(pos)
    step = max(1, (1 << 24) // n)
    images = [(0.0, 0.0)] if box is None else [(i * box[0], j * box[1]) for i in (-1, 0, 1)
                                               for j in (-1, 0, 1)]
    for i0 in range(0, n, step):
        i1 = min(n, i0 + step)
        for shift in images:
            out[i0:i1] += _rows(pos, force, torque, i0, i1, shift, box)
    return out / (8.0 * math.pi)


def _sqrt_apply(pos, w, tol, max_iter=64):
    """The Krylov iterate of M^{1/2} w at the first m >= 2 whose relative change is below tol."""
    norm = w.norm()
    basis, alpha, beta = [w / norm], [], []
    last = None
    for m in range(1, max_iter + 1):
        u = _product(pos, basis[-1])
        alpha.append(float((u * basis[-1]).sum()))
        for _ in range(2):
            for v in basis:
                u = u - (u * v).sum() * v
        beta.append(float(u.norm()))
        tri = np.diag(alpha) + np.diag(beta[:-1], 1) + np.diag(beta[:-1], -1)
        lam, vec = np.linalg.eigh(tri)
        y = float(norm) * (vec * np.sqrt(np.maximum(lam, 0.0))) @ vec[0]
        eps = 0.0
        if last is not None:
            eps = float(np.linalg.norm(y - np.append(last, 0.0)) / np.linalg.norm(last))
            if eps < tol:
                break
        last = y
        basis.append(u / beta[-1])
    return sum(float(c) * v for c, v in zip(y, basis)), m, eps


def _forces(pos):
    """Gravity, the soft repulsion between spheres and that of the wall."""
    out = torch.zeros_like(pos)
    out[:, 2] = F_GRAV + U0 / B * torch.exp(-(pos[:, 2] - 1.0).clamp(min=0.0) / B)
    n = pos.shape[0]
    step = max(1, (1 << 24) // n)
    for i0 in range(0, n, step):
        d = pos[i0:i0 + step, None, :] - pos[None, :, :]
        r = d.square().sum(-1).sqrt()
        f = U0 / B * torch.exp(-(r - 2.0).clamp(min=0.0) / B) / r
        f = f.masked_fill(r == 0.0, 0.0)
        out[i0:i0 + step] += (f[:, :, None] * d).sum(1)
    return out


def _normals(count, seed, stream):
    """The library's normals of step 0: Philox4x64-10 by (seed, stream) and block, Box-Muller."""
    bits = np.random.Philox(key=[seed, stream], counter=[2 ** 64 - 1] * 4)
    raw = bits.random_raw(4 * ((count + 3) // 4)).reshape(-1, 2)
    u = ((raw >> np.uint64(12)).astype(np.float64) + 0.5) * 2.0 ** -52
    rad, ang = np.sqrt(-2.0 * np.log(u[:, 0])), 2.0 * np.pi * u[:, 1]
    return np.stack([rad * np.cos(ang), rad * np.sin(ang)], 1).ravel()[:count]


def _step(pos, noise, noise_drift, tol, max_iter=64):
    """The first step (an Euler-Maruyama one): new positions, velocity, iterations, change."""
    torque = torch.tensor(TORQUE, dtype=torch.float64, device=pos.device).expand_as(pos)
    u = _product(pos, _forces(pos), torque)
    g, m, eps = _sqrt_apply(pos, noise, tol, max_iter)
    half = 0.5 * DELTA * noise_drift
    drift = (_product(pos + half, noise_drift) - _product(pos - half, noise_drift)) / DELTA
    return pos + DT * u + math.sqrt(2.0 * DT) * g + DT * drift, u, m, eps


def exact(case, seed):
    op = case["op"]
    if op == "batch":
        pos, offs = _batch(case, seed)
        if sum(float(k) ** 2 for k in np.diff(offs)) > 5e8:
            return None
        pos = torch.from_numpy(pos).cuda()
        w, wt = (torch.from_numpy(_normals(pos.numel(), seed, k).reshape(-1, 3)).cuda()
                 for k in (0, 1))
        new, vel = torch.empty_like(pos), torch.empty_like(pos)
        for a, b in zip(offs[:-1], offs[1:]):
            new[a:b], vel[a:b], _, _ = _step(pos[a:b], w[a:b], wt[a:b], case["tol"], GRAPH_BUDGET)
        return new, vel
    n = case["n"]
    if op == "matvec":
        if n > 70000:
            return None
        pos, vec = _inputs(case, seed)
        return _product(pos, vec[0], vec[1] if case["torque"] else None,
                        _box(case) if case["box"] else None)
    if n > 20000:
        return None
    if op == "step":
        pos = torch.from_numpy(_positions(n, seed)).cuda()
        w, wt = (torch.from_numpy(_normals(3 * n, seed, k).reshape(n, 3)).cuda() for k in (0, 1))
        return _step(pos, w, wt, case["tol"])
    pos, vec = _inputs(case, seed)
    if op == "lanczos":
        return _sqrt_apply(pos, vec[0], case["tol"])
    got = [_sqrt_apply(pos, v, case["tol"]) for v in vec]
    return (torch.stack([g for g, _, _ in got]), np.array([m for _, m, _ in got], np.int32),
            np.array([e for _, _, e in got]))
