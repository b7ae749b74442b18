"""Workloads that stand for what a program does with this framework.

Each case is a dict of plain values.  ``prepare`` builds what a program holds
before the call (levels, hierarchies, target fields), ``run`` is one pass
through the public entry points, ``work`` counts the bytes and operations a
pass cannot do without and ``exact`` evaluates the same pass in FP64 with
plain torch (the definition: pull, central moments about the local velocity,
relaxation per order, back-transform).

Kinds:
  box         fully periodic level: decaying turbulence, Taylor-Green start,
              buoyant smoke under a body force; `steps` steps in one call
  channel     one level with walls, inlet disk, sphere and outflow (the
              plume's reference scale before its finer scales are placed)
  gradient    periodic level whose adaptive factor takes the finite-difference
              gradient, normalised by its running maximum
  readback    density, velocity and vorticity of a state
  rollout     forward and gradient through a checkpointed rollout
  plume       reference steps of a three-scale hierarchy (boxes or bricks)
  plume_grad  forward and adjoint of reference steps of that hierarchy
"""
import math

import numpy as np
import torch
import torch.utils.checkpoint

from paper_1807_02284_amd import hierarchy, inputs, rollout
from paper_1807_02284_amd.level import F16S, F32, Level, Params

NU_HI = (0.005, 0.007, 0.009, 0.01)


def listed():
    return [
        # the Taylor-Green parity configuration: a level so small that a step
        # is one short launch; 100 steps in one call
        {"name": "tgv_32_100_steps", "kind": "box", "nx": 32, "ny": 32, "nz": 32, "half": False,
         "scalar": False, "force": False, "steps": 100, "macro": False},
        # an interactive loop: one step of a small smoke box, then its fields
        {"name": "smoke_frame_48", "kind": "box", "nx": 48, "ny": 48, "nz": 40, "half": False,
         "scalar": True, "force": False, "steps": 1, "macro": True},
        # the benchmark's workload: 256^3 decaying turbulence, FP32
        {"name": "turbulence_256_f32", "kind": "box", "nx": 256, "ny": 256, "nz": 256,
         "half": False, "scalar": False, "force": False, "steps": 20, "macro": False},
        # the same with binary16 storage
        {"name": "turbulence_256_f16", "kind": "box", "nx": 256, "ny": 256, "nz": 256,
         "half": True, "scalar": False, "force": False, "steps": 20, "macro": False},
        # a forced buoyant-smoke run on a box of odd sizes (the target run of
        # the optimisation examples), 10 steps between two outputs
        {"name": "smoke_force_ragged", "kind": "box", "nx": 181, "ny": 118, "nz": 77,
         "half": False, "scalar": True, "force": True, "steps": 10, "macro": False},
        # spin-up of a plume's reference scale: walls, inlet, sphere, outflow
        {"name": "channel_320x160x160", "kind": "channel", "nx": 320, "ny": 160, "nz": 160,
         "half": False, "scalar": True, "steps": 10},
        # turbulence with the literal |grad u| in the adaptive factor
        {"name": "gradient_160", "kind": "gradient", "n": 160, "steps": 10},
        # output of a frame: density, velocity, vorticity and speed
        {"name": "readback_256", "kind": "readback", "n": 256, "half": False},
        # one optimisation step of the buoyant-smoke problem: forward with
        # checkpoints, then the gradient of the final smoke's misfit
        {"name": "rollout_128", "kind": "rollout", "nx": 128, "ny": 128, "nz": 128, "steps": 12,
         "every": 6},
        # reference steps of a three-scale plume, finer scales as boxes
        {"name": "plume_boxes_256", "kind": "plume", "nx": 256, "bricks": False, "steps": 2},
        # the same scene with the finer scales stored in bricks
        {"name": "plume_bricks_256", "kind": "plume", "nx": 256, "bricks": True, "steps": 2},
        # gradient through two reference steps of a smaller plume
        {"name": "plume_gradient_160", "kind": "plume_grad", "nx": 160, "steps": 2, "every": 2},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["box", "box", "box", "channel", "channel", "gradient", "readback", "rollout",
                       "plume", "plume", "plume_grad"])
    if kind in ("box", "channel"):
        lo = 20 if kind == "box" else 48
        n = [_log(rng, lo, 288) for _ in range(3)]
        steps = _log(rng, 1, 100)
        steps = max(1, min(steps, int(2.0e8 / (n[0] * n[1] * n[2]))))
        c = {"kind": kind, "nx": n[0], "ny": n[1], "nz": n[2], "half": rng.random() < 0.3,
             "scalar": rng.random() < 0.5, "steps": steps}
        if kind == "box":
            c["force"] = rng.random() < 0.3
            c["macro"] = rng.random() < 0.3
        return c
    if kind == "gradient":
        return {"kind": kind, "n": _log(rng, 32, 224), "steps": rng.randint(1, 12)}
    if kind == "readback":
        return {"kind": kind, "n": _log(rng, 32, 256), "half": rng.random() < 0.5}
    if kind == "rollout":
        return {"kind": kind, "nx": _log(rng, 24, 128), "ny": _log(rng, 24, 128),
                "nz": _log(rng, 24, 128), "steps": rng.randint(2, 12), "every": rng.randint(1, 8)}
    if kind == "plume":
        return {"kind": kind, "nx": 2 * _log(rng, 48, 128), "bricks": rng.random() < 0.4,
                "steps": rng.randint(1, 2)}
    return {"kind": kind, "nx": 2 * _log(rng, 48, 80), "steps": rng.randint(1, 2), "every": 2}


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _velocity(nx, ny, nz, seed, rms):
    """Solenoidal random field [3][nz][ny][nx] on the GPU, E(k) ~ k^-5/3 over
    integer wavevectors 2 <= |k| <= 32 (at most a third of the shortest
    side), rms per component `rms`."""
    gen = torch.Generator(device="cuda").manual_seed(int(seed))
    kz, ky, kx = (torch.fft.fftfreq(m, d=1.0 / m, device="cuda") for m in (nz, ny, nx))
    kx = torch.fft.rfftfreq(nx, d=1.0 / nx, device="cuda")
    k = torch.stack(torch.meshgrid(kz, ky, kx, indexing="ij"))
    kk = k.square().sum(0).sqrt()
    top = max(2.0, min(32.0, min(nx, ny, nz) / 3.0))
    amp = torch.where((kk >= 2) & (kk <= top), kk.clamp(min=1.0) ** (-11.0 / 6.0),
                      torch.zeros_like(kk))
    c = torch.complex(*(torch.randn(3, *kk.shape, device="cuda", generator=gen) for _ in range(2)))
    c = c * amp
    kappa = k / torch.tensor([nz, ny, nx], device="cuda").reshape(3, 1, 1, 1)   # physical direction
    norm = kappa.square().sum(0).clamp(min=1e-12)
    c = c - kappa * ((kappa * c).sum(0) / norm)
    u = torch.fft.irfftn(c, s=(nz, ny, nx), dim=(1, 2, 3)).flip(0)              # (x, y, z)
    u = u - u.mean(dim=(1, 2, 3), keepdim=True)
    return (u * (rms / u.square().mean(dim=(1, 2, 3), keepdim=True).sqrt())).contiguous()


def _smoke(nx, ny, nz, seed):
    r = np.random.RandomState(seed % (1 << 31))
    centre = [m * r.uniform(0.35, 0.65) for m in (nx, ny, nz)]
    d = []
    for m, c in zip((nz, ny, nx), reversed(centre)):
        a = (torch.arange(m, device="cuda") - c).abs()
        d.append(torch.minimum(a, m - a).square())
    sigma = min(nx, ny, nz) / 8.0
    r2 = d[0][:, None, None] + d[1][None, :, None] + d[2][None, None, :]
    return torch.exp(-r2 / (2 * sigma * sigma)).reshape(-1)


def _box_params(c):
    if c["kind"] == "rollout":
        return Params(nu=1e-3, g_max=0.1, tau_s=0.51, beta=1e-4, s_ref=0.02)
    if c["kind"] == "gradient":
        return Params(nu=1e-4, g_max=0.1, grad_mode=1, gmax_running=True)
    if c["kind"] == "channel":
        return Params(nu=1e-4, g_max=0.1, tau_s=0.51, u_in=(0.05, 0.0, 0.0), s_in=1.0)
    buoyant = c.get("scalar", False)
    return Params(nu=1e-3 if buoyant else 1e-4, g_max=0.1, tau_s=0.51,
                  beta=1e-4 if buoyant else 0.0, s_ref=0.02 if buoyant else 0.0)


def _start(c, seed):
    """Start fields of a single-level case: u [3][N], s [N] or None, force or
    None, flags or None."""
    if c["kind"] in ("gradient", "readback"):
        nx = ny = nz = c["n"]
    else:
        nx, ny, nz = c["nx"], c["ny"], c["nz"]
    scalar = c["kind"] == "rollout" or bool(c.get("scalar", False))
    flags = None
    if c["kind"] == "channel":
        # wall, inlet disk, sphere and outflow, in proportion to the box
        s = min(ny, nz) / 256.0
        flags = inputs.plume_flags(nx, ny, nz, inlet_radius=32.0 * s,
                                   sphere_center=(0.3 * nx, ny / 2.0, nz / 2.0),
                                   sphere_radius=24.0 * s)
        u = _velocity(nx, ny, nz, seed, 0.01)
        y = torch.arange(ny, device="cuda") + 0.5 - ny / 2
        z = torch.arange(nz, device="cuda") + 0.5 - nz / 2
        jet = (y[None, :].square() + z[:, None].square() <= (32.0 * s) ** 2).float()
        u[0] += 0.05 * jet[:, :, None]
        u = u * torch.as_tensor(flags == 0, device="cuda").reshape(1, nz, ny, nx)
    else:
        u = _velocity(nx, ny, nz, seed, 0.02 if scalar else 0.04)
    sm = _smoke(nx, ny, nz, seed) if scalar else None
    force = None
    if c["kind"] == "rollout" or c.get("force"):
        force = _velocity(nx, ny, nz, seed + 1, 1e-5).reshape(3, -1)
    return (nx, ny, nz), u.reshape(3, -1), sm, force, flags


def _level(c, seed):
    shape, u, s, force, flags = _start(c, seed)
    lev = Level(*shape, _box_params(c), storage=F16S if c.get("half") else F32,
                scalar=s is not None, periodic=7 if flags is None else 0, flags=flags, force=force)
    lev.init_equilibrium(None, u.cpu(), None if s is None else s.cpu())
    return lev, force


def _tube_radius(nx, k):
    """Radius of the brick-stored tube of finer scale k (0, 1)."""
    return min(0.14 * nx, nx / 4 - 13) - (0, 16)[k]


def _plume_hierarchy(nx, bricks, seed):
    """Reference box nx * nx/2 * nx/2 with walls, inlet, sphere and outflow and
    two finer scales (spacing ratios 1.5 and 2) around the jet."""
    ny = nz = nx // 2
    sc = nx / 512.0
    flags = inputs.plume_flags(nx, ny, nz)
    p0 = Params(nu=1e-4, g_max=0.1, tau_s=0.51, u_in=(0.05, 0.0, 0.0), s_in=1.0)
    lev0 = Level(nx, ny, nz, p0, scalar=True, periodic=0, flags=flags)
    u = _velocity(nx, ny, nz, seed, 0.005)
    y = torch.arange(ny, device="cuda") + 0.5 - ny / 2
    z = torch.arange(nz, device="cuda") + 0.5 - nz / 2
    jet = (y[None, :].square() + z[:, None].square() <= (32.0 * sc) ** 2).float()
    u[0] += 0.05 * jet[:, :, None]
    u = u * torch.as_tensor(flags == 0, device="cuda").reshape(1, nz, ny, nx)
    s = (jet[:, :, None] * (torch.arange(nx, device="cuda") < 64 * sc)).reshape(-1)
    lev0.init_equilibrium(None, u.reshape(3, -1).cpu(), s.cpu())
    centre = (160.0 * sc, ny / 2.0, nz / 2.0)
    r = 24.0 * sc

    def sphere(px, py, pz):
        return ((px + 0.5 - centre[0]) ** 2 + (py + 0.5 - centre[1]) ** 2
                + (pz + 0.5 - centre[2]) ** 2) <= r * r

    h = int(0.15 * ny) + 3
    levels, kinds = [lev0], [flags]
    for k, alpha in enumerate((1.5, 2.0)):
        lo = [3 + 2 * k, ny // 2 - h + 2 * k, nz // 2 - h + 2 * k]
        hi = [nx - 4 - 2 * k, ny // 2 + h - 1 - 2 * k, nz // 2 + h - 1 - 2 * k]
        if bricks:
            # a tube around the jet and the sphere, thinner and shorter on the
            # finer scale (left out where it would cut the sphere)
            rr = _tube_radius(nx, k)
            if rr <= r + 5:
                break
            x0, x1 = (12, 0.8 * nx) if k == 0 else (26, 0.6 * nx)
            region = lambda px, py, pz, x0=x0, x1=x1, rr=rr: (  # noqa: E731
                (px >= x0) & (px <= x1) & ((py - ny / 2) ** 2 + (pz - nz / 2) ** 2 <= rr * rr))
            lev, kd = hierarchy.brick_scale([3 + 2 * k] * 3, [nx - 13, ny - 13, nz - 13], alpha, p0,
                                            region, sphere, scalar=True, storage=F32)
        else:
            lev, kd = hierarchy.fine_scale(lo, hi, alpha, p0, sphere, scalar=True, storage=F32)
        hierarchy.fill_from_parent(levels[-1], lev)
        levels.append(lev)
        kinds.append(kd)
    return hierarchy.Hierarchy(levels, kinds)


# ---------------------------------------------------------------------------
# prepare and run
# ---------------------------------------------------------------------------
def prepare(case, seed):
    c = case
    if c["kind"] in ("box", "channel", "gradient", "readback"):
        lev, _ = _level(c, seed)
        if c["kind"] == "readback":
            lev.step(2)     # a state whose density varies
        return {"c": c, "lev": lev}
    if c["kind"] == "rollout":
        lev, theta = _level(c, seed)
        h0, g0 = lev.get_populations(shifted=True)
        target = _smoke(c["nx"], c["ny"], c["nz"], seed + 7)
        return {"c": c, "lev": lev, "theta": theta, "h0": h0, "g0": g0, "target": target}
    H = _plume_hierarchy(c["nx"], bool(c.get("bricks", False)), seed)
    st = {"c": c, "H": H}
    if c["kind"] == "plume_grad":
        gen = torch.Generator(device="cuda").manual_seed(int(seed))
        st["M"] = rollout.MultiscaleRollout(H, c["every"])
        st["lam"] = [1e-3 * torch.randn(27, lv.n, device="cuda", generator=gen) for lv in H.levels]
        st["mu"] = [1e-3 * torch.randn(7, lv.n, device="cuda", generator=gen) for lv in H.levels]
    return st


def _state(lev):
    out = {"f": lev.f.reshape(27, lev.plane)[:, : lev.n]}
    if lev.g is not None:
        out["g"] = lev.g.reshape(7, lev.plane)[:, : lev.n]
    return out


def run(st):
    c = st["c"]
    if c["kind"] in ("box", "channel", "gradient"):
        lev = st["lev"]
        lev.step(c["steps"])
        out = _state(lev)
        if c["kind"] == "gradient":
            out["vel"] = lev.vel
        if c.get("macro"):
            out["rho"], out["u"], s = lev.read_macro()
            if s is not None:
                out["s"] = s
        return out
    if c["kind"] == "readback":
        rho, u, _ = st["lev"].read_macro()
        omega, speed = st["lev"].vorticity()
        return {"rho": rho, "u": u, "omega": omega, "speed": speed}
    if c["kind"] == "rollout":
        leaves = [st[k].detach().requires_grad_(True) for k in ("theta", "h0", "g0")]
        s = rollout.rollout(st["lev"], *leaves, c["steps"], c["every"])
        loss = 0.5 * (s - st["target"]).square().sum()
        d = torch.autograd.grad(loss, leaves)
        return {"s": s.detach(), "dtheta": d[0], "dh0": d[1], "dg0": d[2]}
    if c["kind"] == "plume":
        st["H"].step(c["steps"])
        return [_state(lv) for lv in st["H"].levels]
    st["M"].forward(c["steps"])
    lam, mu = st["M"].backward(st["lam"], st["mu"])
    return {"state": [_state(lv) for lv in st["H"].levels], "lam": lam, "mu": mu}


# ---------------------------------------------------------------------------
# the work a pass cannot do without
# ---------------------------------------------------------------------------
def _plume_cells(c):
    nx, ny = c["nx"], c["nx"] // 2
    if c.get("bricks", False):
        r0, r1 = _tube_radius(nx, 0), _tube_radius(nx, 1)
        return (nx * ny * ny, math.pi * r0 * r0 * (0.8 * nx - 12) * 1.5 ** 3,
                math.pi * r1 * r1 * (0.6 * nx - 26) * 8 if r1 > 24 * nx / 512 + 5 else 0)
    h = int(0.15 * ny) + 3
    return (nx * ny * ny, (nx - 7) * (2 * h) ** 2 * 1.5 ** 3, (nx - 11) * (2 * h - 4) ** 2 * 8)


def work(case):
    """Bytes: each input state, force and flag read once, each output written
    once.  Operations: about 650 FP32 operations per lattice update of the
    central-moment collision and its transforms, 30 for the scalar, three
    times that for an update's adjoint."""
    c = case
    k = c["kind"]
    if k in ("box", "channel"):
        n = c["nx"] * c["ny"] * c["nz"]
        b = 2 * 27 * (2 if c["half"] else 4) + (56 if c["scalar"] else 0)
        b += (12 if c.get("force") else 0) + (1 if k == "channel" else 0)
        b += (16 + (4 if c["scalar"] else 0)) if c.get("macro") else 0
        return {"bytes": n * b, "flops": n * c["steps"] * (680 if c["scalar"] else 650)}
    if k == "gradient":
        n = c["n"] ** 3
        return {"bytes": n * (216 + 24), "flops": n * c["steps"] * 670}
    if k == "readback":
        n = c["n"] ** 3
        return {"bytes": n * (27 * (2 if c["half"] else 4) + 16 + 8), "flops": n * 120}
    if k == "rollout":
        n = c["nx"] * c["ny"] * c["nz"]
        return {"bytes": n * (2 * 12 + 2 * 136 + 8), "flops": n * c["steps"] * (680 + 3 * 680)}
    cells = _plume_cells(c)
    ups = c["steps"] * (cells[0] + 2 * cells[1] + 2 * cells[2])
    if k == "plume":
        return {"bytes": sum(cells) * (2 * 136 + 1), "flops": ups * 680}
    return {"bytes": sum(cells) * (4 * 136 + 1), "flops": ups * 4 * 680}


# ---------------------------------------------------------------------------
# the same passes in FP64
# ---------------------------------------------------------------------------
# velocities in the order of the populations
CX = (0, 1, -1, 0, 0, 0, 0, 1, -1, 1, -1, 1, -1, 1, -1, 0, 0, 0, 0, 1, -1, 1, -1, 1, -1, 1, -1)
CY = (0, 0, 0, 1, -1, 0, 0, 1, 1, -1, -1, 0, 0, 0, 0, 1, -1, 1, -1, 1, 1, -1, -1, 1, 1, -1, -1)
CZ = (0, 0, 0, 0, 0, 1, -1, 0, 0, 0, 0, 1, 1, -1, -1, 1, 1, -1, -1, 1, 1, 1, 1, -1, -1, -1, -1)
W1 = {0: 2.0 / 3.0, 1: 1.0 / 6.0, -1: 1.0 / 6.0}
W = [W1[a] * W1[b] * W1[c] for a, b, c in zip(CX, CY, CZ)]
OPP = [next(j for j in range(27) if (CX[j], CY[j], CZ[j]) == (-CX[i], -CY[i], -CZ[i]))
       for i in range(27)]
SLOT = [(CZ[i] + 1) * 9 + (CY[i] + 1) * 3 + CX[i] + 1 for i in range(27)]
SW = (0.25,) + (0.125,) * 6


def _f32(x):
    return float(np.float32(x))


def _equilibrium(i, rho, u):
    cu = CX[i] * u[0] + CY[i] * u[1] + CZ[i] * u[2]
    uu = u[0] * u[0] + u[1] * u[1] + u[2] * u[2]
    return W[i] * rho * (1.0 + 3.0 * cu + 4.5 * cu * cu - 1.5 * uu)


def _to_central(t, u):
    """27 populations (list, slot order) -> raw central moments, by axis."""
    t = list(t)
    for stride, v in ((1, u[0]), (3, u[1]), (9, u[2])):
        for b in range(27):
            if (b // stride) % 3:
                continue
            am, a0, ap = t[b], t[b + stride], t[b + 2 * stride]
            s0, s1, s2 = am + a0 + ap, ap - am, ap + am
            t[b], t[b + stride], t[b + 2 * stride] = s0, s1 - v * s0, s2 - 2 * v * s1 + v * v * s0
    return t


def _from_central(t, u):
    t = list(t)
    for stride, v in ((9, u[2]), (3, u[1]), (1, u[0])):
        for b in range(27):
            if (b // stride) % 3:
                continue
            k0, k1, k2 = t[b], t[b + stride], t[b + 2 * stride]
            s1 = k1 + v * k0
            s2 = k2 + 2 * v * k1 + v * v * k0
            t[b], t[b + stride], t[b + 2 * stride] = 0.5 * (s2 - s1), k0 - s2, 0.5 * (s2 + s1)
    return t


def _collide(f, p, force, grad=None):
    """f: 27 tensors in population order.  Returns the post-collision tensors
    and the velocity."""
    rho = sum(f)
    u = [(sum(cc[i] * f[i] for i in range(27) if cc[i]) + 0.5 * F) / rho
         for cc, F in zip((CX, CY, CZ), force)]
    t = [None] * 27
    q = [None] * 27
    for i in range(27):
        t[SLOT[i]] = f[i]
        q[SLOT[i]] = _equilibrium(i, rho, u)
    k, e = _to_central(t, u), _to_central(q, u)
    del t, q
    S = 1.0 / (3.0 * p.nu + 0.5)
    xx, yy, zz = (k[a] - e[a] for a in (2, 6, 18))
    xy, xz, yz = (k[a] - e[a] for a in (4, 10, 12))
    tr = (xx + yy + zz) / 3.0
    dev = [xx - tr, yy - tr, zz - tr]
    if grad is None:
        pp = sum(d * d for d in dev) + 2.0 * (xy * xy + xz * xz + yz * yz)
        # the square root's slope at 0 is not needed anywhere but there
        grad = 1.5 * S / rho * torch.sqrt(2.0 * pp + 1e-300)
        gm = p.g_max
    else:
        grad, gm = grad
    phi = p.a * torch.clamp(grad / gm, max=1.0) + p.b
    om = [1.0 - 1.0 / (phi * 3.0 * v + 0.5) for v in NU_HI]
    out = [None] * 27
    for s in range(27):
        order = s % 3 + (s // 3) % 3 + s // 9
        if order == 0:
            out[s] = k[s]
        elif order == 1:
            out[s] = k[s] + force[{1: 0, 3: 1, 9: 2}[s]]
        elif order == 2:
            n = k[s] - e[s]
            if s in (2, 6, 18):
                out[s] = e[s] + (1.0 - S) * dev[{2: 0, 6: 1, 18: 2}[s]] + om[0] * tr
            else:
                out[s] = e[s] + (1.0 - S) * n
        else:
            out[s] = e[s] + om[order - 3] * (k[s] - e[s])
    del k, e
    out = _from_central(out, u)
    return [out[SLOT[i]] for i in range(27)], u


def _pull(a, c):
    """x - c of a [nz][ny][nx] tensor, periodic."""
    return torch.roll(a, (c[2], c[1], c[0]), (0, 1, 2)) if any(c) else a


def _step64(f, g, p, kinds=None, solid=None, theta=None, vel=None, running=False):
    """One step of lists of [nz][ny][nx] FP64 tensors (physical f)."""
    zero = torch.zeros((), dtype=torch.float64, device=f[0].device)
    old, oldg = f, g
    f = [_pull(old[i], (CX[i], CY[i], CZ[i])) for i in range(27)]
    if g is not None:
        g = [_pull(oldg[i], (CX[i], CY[i], CZ[i])) for i in range(7)]
    if kinds is not None:
        for i in range(1, 27):
            f[i] = torch.where(solid[i], old[OPP[i]], f[i])
            if g is not None and i < 7:
                g[i] = torch.where(solid[i], oldg[OPP[i]], g[i])
    force = [zero, zero, zero] if theta is None else [theta[a] for a in range(3)]
    s = None
    if g is not None:
        s = sum(g)
        force[2] = force[2] + p.beta * (s - p.s_ref)
    grad = None
    if vel is not None:
        tot = 0.0
        for v in vel:
            for axis in range(3):
                tot = tot + ((torch.roll(v, -1, axis) - torch.roll(v, 1, axis)) / 2).square()
        G = tot.sqrt()
        grad = (G, G.max() if running else p.g_max)
    f, u = _collide(f, p, force, grad)
    if g is not None:
        g = [g[i] - (g[i] - SW[i] * s * (1.0 + 4.0 * (CX[i] * u[0] + CY[i] * u[1] + CZ[i] * u[2])))
             / p.tau_s for i in range(7)]
    if kinds is not None:
        rho1 = torch.ones((), dtype=torch.float64, device=f[0].device)
        uin = [_f32(v) * rho1 for v in p.u_in]
        for i in range(27):
            f[i] = torch.where(kinds == 1, W[i] * rho1, f[i])
            f[i] = torch.where(kinds == 2, _equilibrium(i, rho1, uin), f[i])
            f[i] = torch.where(kinds == 3, torch.roll(old[i], 1, 2), f[i])
        if g is not None:
            for i in range(7):
                cu = CX[i] * uin[0] + CY[i] * uin[1] + CZ[i] * uin[2]
                g[i] = torch.where(kinds == 1, zero, g[i])
                g[i] = torch.where(kinds == 2, SW[i] * p.s_in * (1.0 + 4.0 * cu), g[i])
                g[i] = torch.where(kinds == 3, torch.roll(oldg[i], 1, 2), g[i])
    return f, g, u


def _blocked(kinds):
    """Per velocity: the pull source is solid or outside the box."""
    nz, ny, nx = kinds.shape
    pad = torch.ones(nz + 2, ny + 2, nx + 2, dtype=torch.bool, device=kinds.device)
    pad[1:-1, 1:-1, 1:-1] = kinds == 1
    fluid = kinds == 0
    return [fluid & pad[1 - CZ[i]:1 - CZ[i] + nz, 1 - CY[i]:1 - CY[i] + ny, 1 - CX[i]:1 - CX[i] + nx]
            for i in range(27)]


def _macro64(f, g, p, theta):
    rho = sum(f)
    F = [0.0, 0.0, 0.0] if theta is None else [theta[a] for a in range(3)]
    s = None if g is None else sum(g)
    if g is not None:
        F[2] = F[2] + p.beta * (s - p.s_ref)
    u = [(sum(cc[i] * f[i] for i in range(27) if cc[i]) - 0.5 * v) / rho
         for cc, v in zip((CX, CY, CZ), F)]
    return rho, u, s


def _start64(c, seed):
    """The start state in FP64 from the same FP32 fields (rounded once more
    for binary16 storage, as the stored start is)."""
    (nx, ny, nz), u, s, force, flags = _start(c, seed)
    shape = (nz, ny, nx)
    u = u.double().reshape(3, *shape)
    one = torch.ones(shape, dtype=torch.float64, device="cuda")
    f = [_equilibrium(i, one, u) for i in range(27)]
    if c.get("half"):
        f = [(f[i] - W[i]).to(torch.float16).double() + W[i] for i in range(27)]
    g = None
    if s is not None:
        s = s.double().reshape(shape)
        g = [SW[i] * s * (1.0 + 4.0 * (CX[i] * u[0] + CY[i] * u[1] + CZ[i] * u[2])) for i in range(7)]
    theta = None if force is None else force.double().reshape(3, *shape)
    kinds = None if flags is None else torch.as_tensor(flags, device="cuda").reshape(shape)
    return shape, f, g, theta, kinds


def exact(case, seed):
    c = case
    if c["kind"] in ("plume", "plume_grad"):
        return None     # several scales and their exchanges: no plain form of moderate size
    if c["kind"] == "rollout":
        return _exact_rollout(c, seed)
    with torch.no_grad():
        p = _box_params(c)
        shape, f, g, theta, kinds = _start64(c, seed)
        if c["kind"] == "readback":
            for _ in range(2):
                f, _, _ = _step64(f, None, p)
            rho, u, _ = _macro64(f, None, p, None)

            def d(a, axis):
                return (torch.roll(a, -1, axis) - torch.roll(a, 1, axis)) / 2

            w = (d(u[2], 1) - d(u[1], 0), d(u[0], 0) - d(u[2], 2), d(u[1], 2) - d(u[0], 1))
            mag = lambda v: sum(x * x for x in v).sqrt().reshape(-1)   # noqa: E731
            return {"rho": rho.reshape(-1), "u": torch.stack(u).reshape(3, -1), "omega": mag(w),
                    "speed": mag(u)}
        vel = _macro64(f, g, p, theta)[1] if c["kind"] == "gradient" else None
        solid = None if kinds is None else _blocked(kinds)
        for _ in range(c["steps"]):
            f, g, u = _step64(f, g, p, kinds, solid, theta, vel, c["kind"] == "gradient")
            vel = u if vel is not None else None
        out = {"f": torch.stack([(f[i] - W[i]).reshape(-1) for i in range(27)])}
        if g is not None:
            out["g"] = torch.stack([x.reshape(-1) for x in g])
        if c["kind"] == "gradient":
            out["vel"] = torch.stack(vel).reshape(-1)
        if c.get("macro"):
            rho, u, s = _macro64(f, g, p, theta)
            out["rho"], out["u"] = rho.reshape(-1), torch.stack(u).reshape(3, -1)
            if s is not None:
                out["s"] = s.reshape(-1)
        return out


def _exact_rollout(c, seed):
    p = _box_params(c)
    with torch.no_grad():
        shape, f, g, theta, _ = _start64(c, seed)
        h0 = torch.stack([f[i] - W[i] for i in range(27)])
        g0 = torch.stack(g)
        del f, g
    leaves = [x.detach().requires_grad_(True) for x in (theta, h0, g0)]
    target = _smoke(c["nx"], c["ny"], c["nz"], seed + 7).double().reshape(shape)

    def one(h, g, th):
        a, b, _ = _step64([h[i] + W[i] for i in range(27)], list(g), p, theta=th)
        return torch.stack([a[i] - W[i] for i in range(27)]), torch.stack(b)

    h, g = leaves[1], leaves[2]
    for _ in range(c["steps"]):
        h, g = torch.utils.checkpoint.checkpoint(one, h, g, leaves[0], use_reentrant=False)
    s = g.sum(0)
    d = torch.autograd.grad(0.5 * (s - target).square().sum(), leaves)
    return {"s": s.detach().reshape(-1), "dtheta": d[0].reshape(3, -1), "dh0": d[1].reshape(27, -1),
            "dg0": d[2].reshape(7, -1)}
