"""Performance cases of the free-surface LBM library: what a user's program has
it do, through the Python entry points, over the range of sizes it is used at.

Every case is a simulation or a gradient of one:

  step     n time steps, then the macroscopic fields of the result are read
           (device tensors), as a run that writes output every n steps does.
           Scenes: the open-channel film and its convergence sizes, the
           sloshing tank (plain and with a surface varying in z, odd sizes
           too), the tank with surface tension and height functions, the tank
           with a solid ramp, a droplet with surface tension.
  restart  a saved state is set, the health check and totals are read and
           every field is exported: a program that resumes and checkpoints.
  adjoint  forward and backward of a window of steps with frozen cell classes
           through the autograd function: one evaluation of a loss and its
           gradients with respect to the state, the gas pressure and gravity.

Inputs are synthetic and made on the GPU from the seed alone.  exact() computes
the same outputs in 64 bits with a plain torch implementation of the method that
shares no code with the library.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1409_5645_amd import fslbm, workloads

GAS, IFACE, LIQ, SOLID = 0, 1, 2, 3
BYTES = {"fp64": 8, "fp32": 4, "fp16s": 2}
MACRO = ("rho", "u", "phi", "flags")
COMPONENTS = {"rho": 1, "u": 3, "phi": 1, "f": 19, "mass": 1, "rho_c": 1, "u_c": 3}
EVERY = ("rho", "u", "phi", "flags", "f", "mass", "rho_c", "u_c")
PROBED = 1_000_000  # cells above which a step case reads only the macroscopic fields

# link order of the library's population buffers (odd q: its opposite is q + 1)
C = ((0, 0, 0), (1, 0, 0), (-1, 0, 0), (0, 1, 0), (0, -1, 0), (0, 0, 1), (0, 0, -1), (1, 1, 0), (-1, -1, 0),
     (1, -1, 0), (-1, 1, 0), (1, 0, 1), (-1, 0, -1), (1, 0, -1), (-1, 0, 1), (0, 1, 1), (0, -1, -1), (0, 1, -1),
     (0, -1, 1))
OPP = (0, 2, 1, 4, 3, 6, 5, 8, 7, 10, 9, 12, 11, 14, 13, 16, 15, 18, 17)
W = (1 / 3,) + (1 / 18,) * 6 + (1 / 36,) * 12


def _step(name, scene, size, form, steps, rule=1, sigma=0.0, plic=0, gy=-2e-5, tau=0.55, waves=0):
    nx, ny, nz = size
    return {"name": name, "kind": "step", "scene": scene, "nx": nx, "ny": ny, "nz": nz, "form": form, "steps": steps,
            "rule": rule, "sigma": sigma, "plic": plic, "gy": gy, "tau": tau, "waves": waves}


def listed():
    return [
        # the validation film (the smallest lattice a user steps thousands of times): latency
        _step("film_8x48x8_fp64", "film", (8, 48, 8), "fp64", 100, tau=0.8),
        # a convergence-study film with the FSK rule
        _step("film_4x80x4_fp32", "film", (4, 80, 4), "fp32", 100, rule=0, tau=0.8),
        # a small tank of odd sizes that sloshes hard (conversions every step), with the shear-rate boundary term
        _step("tank_61x45x37_fp64_stress", "tank", (61, 45, 37), "fp64", 50, rule=3, gy=-2e-4, tau=0.6, waves=1),
        # an ordinary tank, the default form of parameter studies
        _step("tank_128x96x128_fp32", "tank", (128, 96, 128), "fp32", 50),
        # an ordinary tank of odd row length in 16-bit storage, surface varying in z
        _step("tank_253x159x131_fp16s", "tank", (253, 159, 131), "fp16s", 20, waves=1),
        # the 256 tank in 16-bit storage
        _step("tank_256x160x256_fp16s", "tank", (256, 160, 256), "fp16s", 20),
        # the full tank, 16-bit storage and double: the largest calls
        _step("tank_512x320x512_fp16s", "tank", (512, 320, 512), "fp16s", 20),
        _step("tank_512x320x512_fp64", "tank", (512, 320, 512), "fp64", 10),
        # surface tension with height functions (capillary waves in a tank)
        _step("tension_256x160x256_fp32", "tank", (256, 160, 256), "fp32", 20, sigma=1e-4, plic=2, waves=1),
        # a solid ramp under the tank
        _step("ramp_192x96x64_fp64", "ramp", (192, 96, 64), "fp64", 30, tau=0.6),
        # resume from a saved state, check it, export every field
        {"name": "restart_256x160x256_fp32", "kind": "restart", "scene": "tank", "nx": 256, "ny": 160, "nz": 256,
         "form": "fp32", "steps": 0, "rule": 1, "sigma": 0.0, "plic": 0, "gy": -2e-5, "tau": 0.55, "waves": 1},
        # gradients through a window of steps (every step's record kept)
        {"name": "adjoint_128x96x128_fp32", "kind": "adjoint", "scene": "tank", "nx": 128, "ny": 96, "nz": 128,
         "form": "fp32", "steps": 100, "rule": 1, "sigma": 0.0, "plic": 0, "gy": -2e-5, "tau": 0.55, "waves": 0,
         "spacing": 0},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """A case of the ranges above: films of up to a few thousand cells, tanks
    from a few thousand cells to the full one, every form and the options."""
    kind = rng.choice(["film", "tank", "tank", "tank", "tension", "droplet", "ramp", "restart", "adjoint"])
    form = rng.choice(["fp64", "fp32", "fp16s"])
    if kind == "film":
        n = rng.choice([2, 3, 4, 5, 8])
        return _drawn("step", "film", (n, _log_int(rng, 20, 96), n), rng.choice(["fp64", "fp32"]),
                      rng.randint(20, 200), rule=rng.choice([0, 1]), tau=0.8)
    if kind == "droplet":
        n = rng.randint(24, 72)
        return _drawn("step", "droplet", (n, n, n), form, rng.randint(5, 40), sigma=1e-3, plic=rng.choice([0, 1]),
                      gy=0.0, tau=0.8)
    top = {"tank": 64e6, "tension": 8e6, "ramp": 2e6, "restart": 8e6, "adjoint": 1e6}[kind]
    cells = math.exp(rng.uniform(math.log(6e3), math.log(top)))
    if form == "fp64":
        cells = min(cells, 32e6)
    nx = max(8, min(640, int(round((cells * rng.uniform(0.6, 3.0)) ** (1 / 3)))))
    ny = max(16, int(round(nx * rng.uniform(0.55, 0.85))))
    nz = max(3, min(640, int(round(cells / (nx * ny)))))
    size = (nx, ny, nz)
    n = nx * ny * nz
    steps = max(2, min(60, int(4e8 / n)))
    rough = n < 1e6 and rng.random() < 0.5
    if kind == "tension":
        return _drawn("step", "tank", size, form, max(2, steps // 2), sigma=1e-4, plic=rng.choice([0, 1, 2]), waves=1)
    if kind == "ramp":
        return _drawn("step", "ramp", size, form, steps, rule=rng.choice([0, 1]), tau=0.6)
    if kind == "restart":
        return _drawn("restart", "tank", size, form, 0, waves=1)
    if kind == "adjoint":
        c = _drawn("adjoint", "tank", size, rng.choice(["fp64", "fp32"]), rng.randint(4, 40), rule=rng.choice([0, 1]),
                   waves=rng.choice([0, 1]))
        c["spacing"] = rng.choice([0, 0, 7])
        return c
    rule = rng.choice([0, 1, 1, 1, 2, 3])
    return _drawn("step", "tank", size, form, steps, rule=rule, gy=-2e-4 if rough else -2e-5, tau=0.6 if rough else 0.55,
                  waves=rng.choice([0, 1]))


def _drawn(kind, scene, size, form, steps, **more):
    c = _step("", scene, size, form, steps, **more)
    del c["name"]
    c["kind"] = kind
    return c


# ---------------------------------------------------------------- inputs
def _params(case):
    film, drop = case["scene"] == "film", case["scene"] == "droplet"
    g = (1e-6, 0.0, 0.0) if film else (0.0, 0.0, 0.0) if drop else (0.0, case["gy"], 0.0)
    per = (1, 0, 1) if film else (1, 1, 1) if drop else (0, 0, 0)
    return workloads.Params(nx=case["nx"], ny=case["ny"], nz=case["nz"], periodic=per, tau=case["tau"], g=g,
                            sigma=case["sigma"], plic=case["plic"])


def _shift(a, c, axes=(-1, -2, -3)):
    """a at x + c (wrapping; the caller masks what lies beyond a wall)."""
    moves = [(-d, ax) for d, ax in zip(c, axes) if d]
    return torch.roll(a, [m[0] for m in moves], [m[1] for m in moves]) if moves else a


def _beyond(c, shape, periodic, dev):
    """Whether x + c lies beyond a wall, broadcastable to [nz, ny, nx]; None where it never does."""
    out = None
    for d, n, per, dim in ((c[0], shape[2], periodic[0], 2), (c[1], shape[1], periodic[1], 1),
                           (c[2], shape[0], periodic[2], 0)):
        if d == 0 or per:
            continue
        m = torch.zeros(n, dtype=torch.bool, device=dev)
        m[n - 1 if d > 0 else 0] = True
        m = m.reshape([-1 if k == dim else 1 for k in range(3)])
        out = m if out is None else out | m
    return out


def _near(mask, periodic):
    """Cells with one of their 18 neighbours in mask (neighbours beyond a wall excluded)."""
    out = torch.zeros_like(mask)
    for c in C[1:]:
        b = _beyond(c, mask.shape, periodic, mask.device)
        s = _shift(mask, c)
        out |= s if b is None else s & ~b
    return out


def _scene(case, seed, dev="cuda"):
    """Classes [nz, ny, nx], fill, populations [19, ...] and mass of the
    initial state, and the wall table of the ramp."""
    nx, ny, nz = case["nx"], case["ny"], case["nz"]
    p = _params(case)
    r = np.random.default_rng(seed)
    th, thz, part, frac = (float(v) for v in r.random(4))
    f64 = dict(dtype=torch.float64, device=dev)
    x, y, z = (torch.arange(n, **f64) for n in (nx, ny, nz))
    if case["scene"] == "droplet":
        rad = 0.25 * nx
        at = [0.5 * nx + (v - 0.5) for v in (th, thz, part)]
        sub = (torch.arange(6, **f64) + 0.5) / 6
        d2 = [((a[:, None] + sub[None, :] - o) ** 2) for a, o in zip((x, y, z), at)]
        fill = torch.zeros(nz, ny, nx, **f64)
        for i in range(6):
            for j in range(6):
                for k in range(6):
                    fill += (d2[2][:, k][:, None, None] + d2[1][:, j][None, :, None] + d2[0][:, i][None, None, :]
                             <= rad * rad)
        fill /= 216.0
        rho = torch.full_like(fill, 1.0 + 6.0 * case["sigma"] / rad)
    else:
        if case["scene"] == "film":
            eta = torch.full((nz, nx), float(int(0.68 * ny)) + 0.2 + 0.6 * frac, **f64)
        else:
            amp = max(0.7, 0.0375 * ny) * (1.0 if not case["waves"] else 0.8)
            eta = (0.6 * ny + 0.3 * frac + amp * torch.cos(2 * math.pi * ((x + 0.5) / nx + th)))[None, :].repeat(nz, 1)
            if case["waves"]:
                eta = eta + 0.5 * amp * torch.cos(2 * math.pi * ((z + 0.5) / nz + thz))[:, None]
        fill = (eta[:, None, :] - y[None, :, None]).clamp_(0.0, 1.0)
        rho = 1.0 + 3.0 * abs(p.g[1]) * (eta[:, None, :] - (y + 0.5)[None, :, None])
    cls = torch.where(fill >= 1.0, LIQ, torch.where(fill <= 0.0, GAS, IFACE)).to(torch.uint8)
    cls[(cls == LIQ) & _near(cls == GAS, p.periodic)] = IFACE
    walls = None
    if case["scene"] == "ramp":  # cells whose centre lies below a plane rising with x are solid
        slope = 0.2 + 0.2 * part
        nrm = torch.tensor([-slope, 1.0, 0.0], **f64) / math.hypot(slope, 1.0)
        base = 0.1 * ny - slope * 0.35 * nx
        side = (nrm[0] * (x + 0.5)[None, None, :] + nrm[1] * ((y + 0.5)[None, :, None] - base)).expand(nz, ny, nx)
        cls[side < 0.0] = SOLID
        solid = cls == SOLID
        at = torch.nonzero((_near(solid, p.periodic) & ~solid).reshape(-1)).reshape(-1)
        delta = torch.full((19, at.numel()), 0.5, **f64)
        s0 = side.reshape(-1)[at]
        for q in range(1, 19):
            b = _beyond(C[q], cls.shape, p.periodic, dev)
            hit = _shift(solid, C[q]) if b is None else _shift(solid, C[q]) & ~b
            hit = hit.reshape(-1)[at]
            s1 = s0 + float(nrm[0] * C[q][0] + nrm[1] * C[q][1])
            delta[q] = torch.where(hit, s0 / (s0 - s1), delta[q])
        walls = {"cells": at.to(torch.int32), "delta": delta}
    fill = torch.where(cls == SOLID, 0.0, fill)
    act = (cls == IFACE) | (cls == LIQ)
    # velocity: the film's parabola at part of its strength, a weak sway else
    if case["scene"] == "film":
        nu = (p.tau - 0.5) / 3.0
        h = float(eta[0, 0])
        ux = (0.2 + 0.7 * part) * p.g[0] / nu * (h * (y + 0.5) - 0.5 * (y + 0.5) ** 2)[None, :, None]
    else:
        ux = (part - 0.5) * 2e-3 * torch.sin(math.pi * (x + 0.5) / nx)[None, None, :]
    ux = ux.expand(nz, ny, nx)
    f = torch.zeros(19, nz, ny, nx, **f64)
    usq = ux * ux
    for q in range(19):  # post-collision state of an equilibrium: e+(rho, u) + e-(u + g/2)
        cu = C[q][0] * ux
        cg = 0.5 * sum(C[q][a] * p.g[a] for a in range(3))
        f[q] = torch.where(act, W[q] * (rho + 4.5 * cu * cu - 1.5 * usq + 3.0 * (cu + cg)), 0.0)
    mass = torch.where(cls == IFACE, fill * rho, 0.0)
    return p, cls, fill, f, mass, walls


def prepare(case, seed):
    p, cls, fill, f, mass, walls = _scene(case, seed)
    n = p.n_cells
    sim = fslbm.Sim(p, cls.cpu().numpy().reshape(-1), precision=case["form"], freeze=case["kind"] == "adjoint")
    if walls is not None:
        sim.set_walls(walls["cells"].cpu().numpy(), walls["delta"].cpu().numpy())
    f, mass, fill = f.reshape(19, n), mass.reshape(n), fill.reshape(n)
    state = {"sim": sim, "case": case}
    if case["kind"] == "step":
        sim.set_state(f, mass, fill)
        state["names"] = MACRO if n > PROBED else EVERY[:6]
        return state
    state.update(f=f, mass=mass, fill=fill)
    if case["kind"] == "adjoint":
        gen = torch.Generator("cuda").manual_seed(seed)
        state["P_b"] = torch.tensor(p.rho_gas / 3.0, dtype=torch.float64, device="cuda")
        state["g"] = torch.tensor(p.g, dtype=torch.float64, device="cuda")
        state["iface"] = (cls == IFACE).reshape(n)
        state["u_goal"] = 1e-3 * torch.randn(3, n, dtype=torch.float64, device="cuda", generator=gen)
        state["c"] = torch.tensor(C, dtype=torch.float64, device="cuda").T.contiguous()
    return state


def _loss(state, f, phi, g):
    """Squared distance of the interface velocity from a goal and of the fill from one half."""
    u = state["c"] @ f - 0.5 * g[:, None]
    at = state["iface"]
    return ((u - state["u_goal"]) ** 2).sum(0)[at].sum() + ((phi - 0.5) ** 2)[at].sum()


def run(state):
    sim, case = state["sim"], state["case"]
    if case["kind"] == "step":
        sim.step(case["steps"], case["rule"])
        return sim.fields(state["names"], device=True)
    if case["kind"] == "restart":
        sim.set_state(state["f"], state["mass"], state["fill"])
        s = sim.stats()
        out = sim.fields(EVERY, device=True)
        out["total_mass"], out["interface"], out["liquid"] = s["total_mass"], s["interface"], s["liquid"]
        return out
    free = [state[k].detach().requires_grad_(True) for k in ("f", "mass", "fill", "P_b", "g")]
    f, _, phi = fslbm.window_apply(sim, case["steps"], case["rule"], *free, K=case["spacing"])
    loss = _loss(state, f, phi, free[4])
    grads = torch.autograd.grad(loss, free)
    return {"loss": loss.detach(), **dict(zip(("f0", "m0", "phi0", "P_b", "g"), grads))}


def work(case):
    n = case["nx"] * case["ny"] * case["nz"]
    share = {"film": 0.7, "tank": 0.61, "ramp": 0.5, "droplet": 4 / 3 * math.pi / 64}[case["scene"]]
    act, s = share * n, BYTES[case["form"]]
    step = act * 38 * s + n
    if case["kind"] == "adjoint":  # a forward and a reverse step each, the state in, the gradients out
        return {"bytes": case["steps"] * (step + act * 41 * s) + 8.0 * n * (3 * 19 + 4), "flops": case["steps"] * act * 900.0}
    names = EVERY if case["kind"] == "restart" or n <= PROBED else MACRO
    out = act * 19 * s + n * (1.0 + 8.0 * sum(COMPONENTS[k] for k in names if k != "flags"))
    back = act * 19 * (8 + s) + act * 19 * s if case["kind"] == "restart" else 0.0
    return {"bytes": case["steps"] * step + out + back, "flops": (case["steps"] * 400.0 + 60.0) * act}


# ------------------------------------------------- the same in 64 bits, plainly
class _Plain:
    """One step of the method on [nz, ny, nx] fields in float64: the bulk by
    shifted arrays, the interface cells by index lists.  Differentiable where
    the classes stay fixed."""

    def __init__(self, p, cls, walls):
        self.p, self.shape = p, tuple(cls.shape)
        self.dev = cls.device
        self.lp = -1.0 / p.tau
        self.lm = -1.0 / (p.Lambda / (p.tau - 0.5) + 0.5)
        self.slot = None
        if walls is not None:
            self.slot = torch.full((p.n_cells,), -1, dtype=torch.int64, device=self.dev)
            self.slot[walls["cells"].long()] = torch.arange(walls["cells"].numel(), device=self.dev)
            self.delta = walls["delta"]

    def at(self, idx, c):
        """Index of x + c (its wrap), and whether it lies beyond a wall."""
        n = (self.p.nx, self.p.ny, self.p.nz)
        xyz = (idx % n[0], (idx // n[0]) % n[1], idx // (n[0] * n[1]))
        out, bad = [], torch.zeros_like(idx, dtype=torch.bool)
        for a in range(3):
            v = xyz[a] + c[a]
            if not self.p.periodic[a]:
                bad = bad | (v < 0) | (v >= n[a])
            out.append(v % n[a])
        return out[0] + n[0] * (out[1] + n[1] * out[2]), bad

    def moments(self, rows):
        rho = sum(rows)
        j = [sum(C[q][a] * rows[q] for q in range(19) if C[q][a]) for a in range(3)]
        return rho, j

    @staticmethod
    def even(q, rho, u):
        cu = sum(C[q][a] * u[a] for a in range(3) if C[q][a])
        nl = -1.5 * (u[0] * u[0] + u[1] * u[1] + u[2] * u[2])
        return W[q] * (rho + (nl if q == 0 else 4.5 * cu * cu + nl))

    def collide(self, rows, g):
        rho, j = self.moments(rows)
        u = [j[a] + 0.5 * g[a] for a in range(3)]
        ue = [j[a] - g[a] / self.lm for a in range(3)]
        out = [None] * 19
        out[0] = rows[0] + self.lp * (rows[0] - self.even(0, rho, u))
        for q in range(1, 19, 2):
            odd = 3.0 * W[q] * sum(C[q][a] * ue[a] for a in range(3) if C[q][a])
            np_ = 0.5 * (rows[q] + rows[q + 1]) - self.even(q, rho, u)
            nm = 0.5 * (rows[q] - rows[q + 1]) - odd
            out[q] = rows[q] + self.lp * np_ + self.lm * nm
            out[q + 1] = rows[q + 1] + self.lp * np_ - self.lm * nm
        return out, rho, u

    def wall_links(self, rows, own, idx, solid, fluid):
        """Interpolated wall closure of the links that pull from a solid cell (walls at rest)."""
        s = self.slot[idx].clamp_min(0)
        out = list(rows)
        for q in range(1, 19):
            o = OPP[q]
            d = self.delta[o][s]
            kap = (1 - 2 * d) / (1 + 2 * d)
            v = torch.where(fluid[o], own[o] + kap * (rows[o] - own[q]), own[o])
            out[q] = torch.where(solid[q], v, rows[q])
        return out

    def columns(self, idx, cls, seen, n):
        """Heights of the 3 x 3 columns along the normal's largest axis, and where they are complete."""
        best = torch.zeros_like(idx)
        top = n[0].abs()
        for a in (1, 2):
            more = n[a].abs() > top
            best, top = torch.where(more, a, best), torch.where(more, n[a].abs(), top)
        h = torch.zeros(3, 3, idx.numel(), dtype=torch.float64, device=self.dev)
        good = torch.ones_like(idx, dtype=torch.bool)
        side = torch.where(torch.stack(n).gather(0, best[None])[0] > 0, 1, -1)
        for a in range(3):
            m = torch.nonzero(best == a).reshape(-1)
            if not m.numel():
                continue
            e1, e2 = (1, 2) if a == 0 else (2, 0) if a == 1 else (0, 1)
            for i in (-1, 0, 1):
                for k in (-1, 0, 1):
                    for t in range(-3, 4):
                        c = [0, 0, 0]
                        c[a], c[e1], c[e2] = t, i, k
                        s, bad = self.at(idx[m], c)
                        v = torch.where(cls[s] == LIQ, 1.0, torch.where(cls[s] == GAS, 0.0, seen[s]))
                        end = torch.where(t == -3 * side[m], v >= 1.0, torch.where(t == 3 * side[m], v <= 0.0, True))
                        good[m] &= ~bad & (cls[s] != SOLID) & end
                        h[i + 1, k + 1, m] += v
        return h, best, side, good

    @staticmethod
    def curvature_of(h):
        h1, h2 = 0.5 * (h[2, 1] - h[0, 1]), 0.5 * (h[1, 2] - h[1, 0])
        h11, h22 = h[2, 1] - 2 * h[1, 1] + h[0, 1], h[1, 2] - 2 * h[1, 1] + h[1, 0]
        h12 = 0.25 * (h[2, 2] - h[2, 0] - h[0, 2] + h[0, 0])
        return (h11 * (1 + h2 * h2) + h22 * (1 + h1 * h1) - 2 * h12 * h1 * h2) / (1 + h1 * h1 + h2 * h2) ** 1.5

    @staticmethod
    def plane_offset(phi, n):
        """Offset of the plane with normal n that cuts the fill phi, by bisection of the cut volume."""
        s = torch.stack([v.abs() for v in n]).sort(0).values
        tot = s.sum(0)
        s1, s2, s3 = s / tot
        v = phi.clamp(0.0, 1.0)
        t = torch.where(v > 0.5, 1.0 - v, v)

        def volume(al):
            cube = lambda d: d.clamp_min(0.0) ** 3  # noqa: E731
            tiny = s1 < 1e-5  # a plane that holds an axis: the two-dimensional cut
            q = lambda d: d.clamp_min(0.0) ** 2  # noqa: E731
            two = torch.where(s2 > 1e-12, (q(al) - q(al - s2) - q(al - s3)) / (2 * s2 * s3), al / s3)
            b = torch.where(tiny, 1.0, s1)
            return torch.where(tiny, two, (cube(al) - cube(al - s1) - cube(al - s2) - cube(al - s3)
                                           + cube(al - s1 - s2)) / (6 * b * s2 * s3))

        lo, hi = torch.zeros_like(t), torch.full_like(t, 0.5)
        for _ in range(54):
            mid = 0.5 * (lo + hi)
            low = volume(mid) < t
            lo, hi = torch.where(low, mid, lo), torch.where(low, hi, mid)
        al = 0.5 * (lo + hi)
        return tot * (torch.where(v > 0.5, 1.0 - al, al) - 0.5)

    def shear(self, f, idx, own, liquid, n, g):
        """Boundary shear rate from the liquid neighbour whose link points most directly into the liquid."""
        best = torch.full_like(idx, -1)
        top = torch.zeros_like(n[0])
        for k in range(1, 19):
            cn = -sum(C[k][a] * n[a] for a in range(3))
            v = cn.abs() * cn / (1.0 if k <= 6 else 2.0)
            take = liquid[OPP[k]] & ((best < 0) | (v > top))
            best, top = torch.where(take, k, best), torch.where(take, v, top)
        src = idx.clone()
        for k in range(1, 19):
            src = torch.where(best == k, self.at(idx, C[k])[0], src)
        fl = f.reshape(19, -1)
        rows = [torch.where(best < 0, own[q], fl[q][src]) for q in range(19)]
        rho, j = self.moments(rows)
        u = [j[a] - 0.5 * g[a] for a in range(3)]
        M = torch.zeros(3, 3, idx.numel(), dtype=torch.float64, device=self.dev)
        for q in range(1, 19, 2):
            ne = (0.5 * (rows[q] + rows[q + 1]) - self.even(q, rho, u)) / (1 + self.lp)
            for a in range(3):
                for b in range(3):
                    if C[q][a] * C[q][b]:
                        M[a, b] += 2 * C[q][a] * C[q][b] * ne
        tr = (M[0, 0] + M[1, 1] + M[2, 2]) / 5
        S = 1.5 * self.lp * (M - torch.eye(3, dtype=torch.float64, device=self.dev)[:, :, None] * tr)
        N = torch.stack(n)
        Sn = (S * N[None]).sum(1)
        nSn = (Sn * N).sum(0)
        return S - Sn[:, None] * N[None] - N[:, None] * Sn[None] + (nSn + nSn / 3) * N[:, None] * N[None]

    def step(self, s, rule, g, rho_b, convert=True):
        p, cls = self.p, s["cls"]
        f, phi, m = s["f"], s["phi"], s["m"]
        flat = cls.reshape(-1)
        gas3, solid3 = cls == GAS, cls == SOLID
        # bulk: pull with bounce-back, collide
        rows = []
        for q in range(19):
            back = tuple(-v for v in C[q])
            b = _beyond(back, self.shape, p.periodic, self.dev)
            v = _shift(f[q], back)
            rows.append(v if b is None else torch.where(b, f[OPP[q]], v))
        fl = f.reshape(19, -1)
        post, _, _ = self.collide(rows, g)
        del rows
        for q in range(19):
            post[q] = torch.where(gas3 | solid3, 0.0, post[q])
        new = torch.stack(post).reshape(19, -1)
        del post

        def gathered(idx):
            own = [fl[q][idx] for q in range(19)]
            pulled, kind, src = [own[0]], [None], [None]
            for q in range(1, 19):
                a, bad = self.at(idx, tuple(-v for v in C[q]))
                k = torch.where(bad, SOLID, flat[a].to(torch.int64))
                pulled.append(torch.where(bad, own[OPP[q]], fl[q][a]))
                kind.append(k)
                src.append((a, bad))
            if self.slot is not None:
                solid = [None] + [(kind[q] == SOLID) & ~src[q][1] for q in range(1, 19)]
                fluid = [None] + [(kind[q] == LIQ) | (kind[q] == IFACE) for q in range(1, 19)]
                pulled = self.wall_links(pulled, own, idx, solid, fluid)
            return own, pulled, kind, src

        if self.slot is not None:  # liquid cells next to the obstacle
            idx = torch.nonzero((self.slot >= 0) & (flat == LIQ)).reshape(-1)
            _, pulled, _, _ = gathered(idx)
            new = new.index_copy(1, idx, torch.stack(self.collide(pulled, g)[0]))
        idx = torch.nonzero(flat == IFACE).reshape(-1)
        own, pulled, kind, src = gathered(idx)
        me, mass = phi[idx], m[idx]
        near = [None] + [torch.where(kind[q] == IFACE, phi[src[q][0]], me) for q in range(1, 19)]
        seen = [None] + [torch.where(kind[q] == LIQ, 1.0, torch.where(kind[q] == GAS, 0.0, near[q]))
                         for q in range(1, 19)]
        dm = 0.0
        for q in range(1, 19):
            w = torch.where(kind[q] == LIQ, 1.0, torch.where(kind[q] == IFACE, 0.5 * (me + near[q]), 0.0))
            dm = dm + w * (pulled[q] - own[OPP[q]])
        mass = mass + dm
        grad = [0.5 * (seen[2 * a + 2] - seen[2 * a + 1]) for a in range(3)]
        sq = grad[0] ** 2 + grad[1] ** 2 + grad[2] ** 2
        has = sq > 0
        nrm = torch.sqrt(torch.where(has, sq, 1.0))
        n = [torch.where(has, -v / nrm, 0.0) for v in grad]
        press = torch.zeros_like(me)
        if p.sigma:
            press = 3.0 * p.sigma * self.kappa(idx, flat, phi, me, seen, sq, has, n)
        dist = me - 0.5
        if p.plic and rule & 1:
            if p.plic == 2:
                h, ax, side, good = self.columns(idx, flat, phi, n)
                h1, h2 = 0.5 * (h[2, 1] - h[0, 1]), 0.5 * (h[1, 2] - h[1, 0])
                r = 1.0 / torch.sqrt(1.0 + h1 * h1 + h2 * h2)
                hf = []
                for a in range(3):  # axis a is the columns' axis, its first or its second cross axis
                    v = torch.where(ax == a, side.double(), torch.where((ax + 1) % 3 == a, -h1, -h2))
                    hf.append(v * r)
                n = [torch.where(good & has, hf[a], n[a]) for a in range(3)]
            safe = [torch.where(has, n[a], 1.0 if a == 0 else 0.0) for a in range(3)]
            dist = torch.where(has, self.plane_offset(me, safe), dist)
        rho_t, j = self.moments(own)
        u_t = [j[a] - 0.5 * g[a] for a in range(3)]
        shear = self.shear(f, idx, own, [None] + [kind[q] == LIQ for q in range(1, 19)], n, g) if rule & 2 else None
        fresh = list(pulled)
        for q in range(1, 19):
            o = OPP[q]
            e_b = self.even(o, rho_b - press, u_t)
            fsk = 2 * e_b - own[o]
            v = fsk
            cSc = 0.0
            if shear is not None:
                cSc = sum(C[o][a] * C[o][b] * shear[a, b] for a in range(3) for b in range(3) if C[o][a] * C[o][b])
                D = -(p.tau - 0.5) * 3 * W[o] * torch.where(has, 1.0, 0.0)
                v = fsk = fsk + 2 * D * cSc
            if rule & 1:
                nc = sum(C[o][a] * n[a] for a in range(3) if C[o][a])
                use = has & (kind[o] != GAS) & (nc > 0)
                d = (dist / torch.where(use, nc, 1.0)).clamp(0.0, 1.0)
                ne = (0.5 * (own[o] + own[q]) - self.even(o, rho_t, u_t)) / (1 + self.lp)
                fsl = (0.5 - d) * own[o] + 0.5 * own[q] + (d - 1) * pulled[o] + self.lp * (d - 1.5) * ne + e_b
                v = torch.where(use, fsl if shear is None else fsl + D * cSc, fsk)
            fresh[q] = torch.where(kind[q] == GAS, v, pulled[q])
        out, rho, u = self.collide(fresh, g)
        new = new.index_copy(1, idx, torch.stack(out))
        t = {"f": new.reshape(f.shape), "phi": phi.index_copy(0, idx, mass / rho), "m": m.index_copy(0, idx, mass),
             "cls": cls, "reservoir": s["reservoir"], "rho_c": torch.zeros_like(phi).index_copy(0, idx, rho),
             "u_c": torch.zeros(3, phi.numel(), dtype=phi.dtype, device=self.dev).index_copy(1, idx, torch.stack(u))}
        if convert:
            self.convert(t, idx, mass, rho, g)
        return t

    def kappa(self, idx, flat, phi, me, seen, sq, has, n):
        def v(*c):
            return me if c == (0, 0, 0) else seen[C.index(tuple(-x for x in c))]

        e = [tuple(int(a == b) for b in range(3)) for a in range(3)]
        add = lambda a, b, s, t: tuple(s * i + t * j for i, j in zip(a, b))  # noqa: E731
        d = [0.5 * (v(*e[a]) - v(*add(e[a], e[a], -1, 0))) for a in range(3)]
        H = [[None] * 3 for _ in range(3)]
        for a in range(3):
            for b in range(3):
                if a == b:
                    H[a][a] = v(*e[a]) - 2 * me + v(*add(e[a], e[a], -1, 0))
                else:
                    H[a][b] = 0.25 * (v(*add(e[a], e[b], 1, 1)) - v(*add(e[a], e[b], 1, -1))
                                      - v(*add(e[a], e[b], -1, 1)) + v(*add(e[a], e[b], -1, -1)))
        gHg = sum(d[a] * H[a][b] * d[b] for a in range(3) for b in range(3))
        safe = torch.where(has, sq, 1.0)
        kap = torch.where(has, (sq * (H[0][0] + H[1][1] + H[2][2]) - gHg) / (safe * torch.sqrt(safe)), 0.0)
        if self.p.plic != 2:
            return kap
        h, _, _, good = self.columns(idx, flat, phi, n)
        good = good & has
        hf = torch.full((flat.numel(),), float("nan"), dtype=torch.float64, device=self.dev)
        hf[idx[good]] = self.curvature_of(h)[good]
        tot, cnt = torch.zeros_like(kap), torch.zeros_like(kap)
        for c in C[1:]:
            a, bad = self.at(idx, c)
            ok = ~bad & (flat[a] == IFACE) & ~torch.isnan(hf[a])
            tot, cnt = tot + torch.where(ok, hf[a], 0.0), cnt + ok
        return torch.where(good, hf[idx], torch.where(cnt > 0, tot / cnt.clamp_min(1), kap))

    def convert(self, t, idx, mass, rho, g):
        p, cls = self.p, t["cls"]
        eps = p.eps
        full = torch.zeros(p.n_cells, dtype=torch.bool, device=self.dev)
        empty = full.clone()
        full[idx[mass > (1 + eps) * rho]] = True
        empty[idx[mass < -eps * rho]] = True
        if not bool(full.any() | empty.any()):
            return
        full3, empty3 = full.reshape(self.shape), empty.reshape(self.shape)
        empty3 = empty3 & ~_near(full3, p.periodic)
        from_gas = ((cls == GAS) & _near(full3, p.periodic)).reshape(-1)
        from_liq = ((cls == LIQ) & _near(empty3, p.periodic)).reshape(-1)
        empty = empty3.reshape(-1)
        after = cls.clone().reshape(-1)
        after[full], after[empty], after[from_gas | from_liq] = LIQ, GAS, IFACE
        old, f = cls.reshape(-1), t["f"].reshape(19, -1)
        c = torch.nonzero(from_gas).reshape(-1)
        if c.numel():  # equilibrium of the mean density and velocity of the fluid neighbours
            r, u, k = 0.0, 0.0, 0.0
            for d in C[1:]:
                a, bad = self.at(c, d)
                ok = (~bad & (old[a] != GAS) & (old[a] != SOLID)).double()
                r, u, k = r + ok * t["rho_c"][a], u + ok * t["u_c"][:, a], k + ok
            r, u = r / k, u / k
            for q in range(19):
                f[q, c] = self.even(q, r, u) + 3 * W[q] * sum(C[q][a] * (u[a] + 0.5 * g[a]) for a in range(3))
            t["rho_c"][c], t["m"][c] = r, 0.0
        c = torch.nonzero(from_liq).reshape(-1)
        t["rho_c"][c] = t["m"][c] = f[:, c].sum(0)
        c = torch.nonzero(full | empty).reshape(-1)
        excess = torch.where(full[c], t["m"][c] - t["rho_c"][c], t["m"][c])
        takers = [(a, ~bad & (after[a] == IFACE)) for a, bad in (self.at(c, d) for d in C[1:])]
        k = sum(ok.double() for _, ok in takers)
        t["reservoir"] = t["reservoir"] + float(excess[k == 0].sum())
        for a, ok in takers:
            t["m"].index_add_(0, a[ok], (excess / k.clamp_min(1))[ok])
            t["phi"][a[ok]] = t["m"][a[ok]] / t["rho_c"][a[ok]]
        for a, ok in takers:  # again, now that every share has arrived
            t["phi"][a[ok]] = t["m"][a[ok]] / t["rho_c"][a[ok]]
        t["cls"] = after.reshape(self.shape)
        f[:, after == GAS] = 0.0


def exact(case, seed):
    p, cls, fill, f, mass, walls = _scene(case, seed)
    n = p.n_cells
    if case["kind"] == "adjoint" and n * case["steps"] > 2e8:
        return None
    plain = _Plain(p, cls, walls)
    s = {"cls": cls, "f": f, "phi": fill.reshape(n), "m": mass.reshape(n), "reservoir": 0.0}
    if case["kind"] == "adjoint":
        return _exact_adjoint(case, seed, p, plain, s)
    for _ in range(case["steps"]):
        s = plain.step(s, case["rule"], p.g, p.rho_gas)
    k = s["cls"].reshape(-1)
    f, act, itf = s["f"].reshape(19, n), (k == LIQ) | (k == IFACE), k == IFACE
    rho, j = plain.moments(list(f))
    out = {"rho": torch.where(act, rho, 0.0),
           "u": torch.stack([torch.where(act, j[a] - 0.5 * p.g[a], 0.0) for a in range(3)]),
           "phi": torch.where(k == LIQ, 1.0, torch.where(itf, s["phi"], 0.0)), "flags": k}
    if case["kind"] == "step":
        if n <= PROBED:
            out.update(f=torch.where(act, f, 0.0), mass=torch.where(itf, s["m"], 0.0))
        return out
    out.update(f=torch.where(act, f, 0.0), mass=torch.where(itf, s["m"], 0.0), rho_c=torch.where(itf, rho, 0.0),
               u_c=torch.where(itf, out["u"], 0.0), total_mass=float((rho * (k == LIQ)).sum() + s["m"][itf].sum()),
               interface=int(itf.sum()), liquid=int((k == LIQ).sum()))
    return out


def _exact_adjoint(case, seed, p, plain, s):
    from torch.utils.checkpoint import checkpoint
    n = p.n_cells
    gen = torch.Generator("cuda").manual_seed(seed)
    goal = {"iface": (s["cls"] == IFACE).reshape(n),
            "u_goal": 1e-3 * torch.randn(3, n, dtype=torch.float64, device="cuda", generator=gen),
            "c": torch.tensor(C, dtype=torch.float64, device="cuda").T.contiguous()}
    f, m, phi = (s[k].clone().requires_grad_(True) for k in ("f", "m", "phi"))
    P_b = torch.tensor(p.rho_gas / 3.0, dtype=torch.float64, device="cuda", requires_grad=True)
    g = torch.tensor(p.g, dtype=torch.float64, device="cuda", requires_grad=True)

    def one(f, m, phi, P_b, g):
        t = plain.step({**s, "f": f, "m": m, "phi": phi}, case["rule"], g, 3.0 * P_b, convert=False)
        return t["f"], t["m"], t["phi"]

    state = (f, m, phi)
    for _ in range(case["steps"]):
        state = checkpoint(one, *state, P_b, g, use_reentrant=False)
    loss = _loss(goal, state[0].reshape(19, n), state[2], g)
    grads = torch.autograd.grad(loss, (f, m, phi, P_b, g))
    act = (s["cls"] != GAS).reshape(n)
    itf = goal["iface"]
    return {"loss": loss.detach(), "f0": torch.where(act, grads[0].reshape(19, n), 0.0),
            "m0": torch.where(itf, grads[1], 0.0), "phi0": torch.where(itf, grads[2], 0.0), "P_b": grads[3],
            "g": grads[4]}
