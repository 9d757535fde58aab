"""What a user of this solver has it do, as cases that can be timed and checked.

Four kinds of pass, each through the public Python front-end:
  steps    sim.step(n): time stepping between two outputs;
  sample   sim.step(n), then the fields and the global sums -- a run that is
           watched or coupled to another code;
  fields   the fields and the global sums of a state, without a step;
  rollout  the differentiable rollout, forward and backward.
A case names the box (nz, ny, nx), the storage format, the geometry (periodic
box, 10% spheres of radius 4 to 12, channel with walls in y, lid-driven
cavity), the equilibrium and the schedule (1: the default single steps, 2:
fused pairs, "auto").  Everything random comes from the seed.
"""
import math

import torch

from paper_1112_0850_amd.lbm import LBM, rollout

SOLID, MOVING = 1, 4
LID = (0.05, 0.0, 0.0)
BYTES = {"f32": 4, "f32x": 4, "f16": 2, "bf16": 2, "f64": 8}
# velocities of the interface order (x, y, z) and their weights
E = [(0, 0, 0), (1, 0, 0), (-1, 0, 0), (0, 1, 0), (0, -1, 0), (0, 0, 1), (0, 0, -1),
     (1, 1, 0), (-1, -1, 0), (1, -1, 0), (-1, 1, 0), (1, 0, 1), (-1, 0, -1), (1, 0, -1),
     (-1, 0, 1), (0, 1, 1), (0, -1, -1), (0, 1, -1), (0, -1, 1)]
W = [1 / 3] + [1 / 18] * 6 + [1 / 36] * 12
OPP = [0] + [i + 1 if i % 2 else i - 1 for i in range(1, 19)]


def _case(name, kind, shape, **kw):
    nz, ny, nx = shape
    case = {"kind": kind, "nz": nz, "ny": ny, "nx": nx, "storage": "f32", "geometry": "box",
            "equilibrium": "qian", "tau": 0.6, "fx": 0.0, "steps": 0, "schedule": "1", "every": 0}
    case.update(kw)
    return dict(case, name=name) if name else case


def listed():
    return [
        # the smallest calls: one step of a small cavity, its fields and sums
        # read back each time, as a viewer or a coupled code does
        _case("sample_cavity24_f32", "sample", (24, 24, 24), geometry="cavity", steps=1),
        # a small box run for a while: the Taylor-Green decay on 32^3
        _case("steps_tg32_f32", "steps", (32, 32, 32), geometry="taylor_green", steps=100,
              schedule="auto"),
        # a small porous sample with body force
        _case("steps_porous64_f32", "steps", (64, 64, 64), geometry="porous", tau=0.55, fx=1e-6,
              steps=50, schedule="auto"),
        # the forced channel 256 x 128 x 128 between walls
        _case("steps_channel256_f32", "steps", (128, 128, 256), geometry="channel", fx=1e-6,
              steps=50, schedule="auto"),
        # the default schedule with the fields and sums of every 20th step
        _case("sample_porous128_f32", "sample", (128, 128, 128), geometry="porous", tau=0.55,
              fx=1e-6, steps=20),
        # a ragged lid-driven cavity in bfloat16 (moving walls)
        _case("steps_cavity200_bf16", "steps", (200, 200, 200), storage="bf16", geometry="cavity",
              steps=20, schedule="auto"),
        # an uneven all-fluid box in double precision, incompressible equilibrium
        _case("steps_box192_f64", "steps", (180, 200, 192), storage="f64",
              equilibrium="incompressible", steps=20, schedule="2"),
        # 16-bit storage on the default schedule, rows that are no multiple of 64
        _case("steps_porous300_f16", "steps", (300, 300, 300), storage="f16", geometry="porous",
              tau=0.55, fx=1e-6, steps=10),
        # the largest: the 512^3 porous box in fused pairs (the benchmark's workload)
        _case("steps_porous512_f32", "steps", (512, 512, 512), geometry="porous", tau=0.55,
              fx=1e-6, steps=10, schedule="2"),
        # post-processing: fields and sums of a 256^3 porous state
        _case("fields_porous256_f32", "fields", (256, 256, 256), geometry="porous", tau=0.55,
              fx=1e-6),
        # gradients of a periodic 128^3 rollout for the initial velocity and the force
        _case("rollout_box128", "rollout", (128, 128, 128), fx=1e-6, steps=60, every=20),
        # the same around obstacles, an uneven box, short segments
        _case("rollout_porous100", "rollout", (72, 80, 100), geometry="porous", fx=1e-6, steps=24,
              every=8),
    ]


# cell updates that a drawn case may ask for (the largest listed: 1.3e9 in FP32)
_MOST_UPDATES = 2.0e8


def draw(rng):
    kind = rng.choice(["steps", "steps", "steps", "steps", "sample", "fields", "rollout"])
    top = 160 if kind == "rollout" else 320
    edge = math.exp(rng.uniform(math.log(16), math.log(top)))
    shape = tuple(max(12, min(top, round(edge * math.exp(rng.uniform(-0.4, 0.4)))))
                  for _ in range(3))
    cells = shape[0] * shape[1] * shape[2]
    geometry = rng.choice(["box", "porous", "channel", "cavity"])
    kw = {"geometry": geometry, "tau": rng.choice([0.55, 0.6, 0.8]),
          "fx": rng.choice([0.0, 1e-6]),
          "equilibrium": rng.choice(["qian", "qian", "incompressible"])}
    if kind == "rollout":
        kw["steps"] = min(rng.randint(2, 60), max(2, int(_MOST_UPDATES / 4 / cells)))
        kw["every"] = rng.randint(1, 20)
        kw["schedule"] = rng.choice(["1", "2"])
    else:
        kw["storage"] = rng.choice(["f32", "f32", "f16", "bf16", "f64", "f32x"])
        kw["schedule"] = rng.choice(["1", "2", "auto"])
        if kind != "fields":
            kw["steps"] = min(rng.randint(1, 100), max(1, int(_MOST_UPDATES / cells)))
    return _case("", kind, shape, **kw)


def _generator(seed, salt):
    return torch.Generator().manual_seed(1_000_003 * (seed % (1 << 40)) + salt)


def _flags(case, seed):
    """uint8 flags on the GPU, or None for an all-fluid box."""
    nz, ny, nx = case["nz"], case["ny"], case["nx"]
    geometry = case["geometry"]
    if geometry in ("box", "taylor_green"):
        return None
    f = torch.zeros(nz, ny, nx, dtype=torch.uint8, device="cuda")
    if geometry == "channel":
        f[:, 0] = f[:, ny - 1] = SOLID
    elif geometry == "cavity":
        f[0] = f[:, 0] = f[:, ny - 1] = f[:, :, 0] = f[:, :, nx - 1] = SOLID
        f[nz - 1] = SOLID | MOVING
    else:
        # one sphere of radius 4..12 somewhere in every 30^3 block: 10% solid
        b = 30
        n = [-(-s // b) for s in (nz, ny, nx)]
        r = 4 + 8 * torch.rand(n, generator=_generator(seed, 1))
        centre = r + (b - 2 * r) * torch.rand([3] + n, generator=_generator(seed, 2))
        r, centre = r.cuda(), centre.cuda()
        blk = [torch.arange(s, device="cuda") // b for s in (nz, ny, nx)]
        pos = [(torch.arange(s, device="cuda") % b).float() for s in (nz, ny, nx)]
        for z0 in range(0, nz, b):  # a layer of blocks at a time
            z = slice(z0, min(z0 + b, nz))
            at = (z0 // b, blk[1][:, None], blk[2][None, :])
            d2 = (pos[0][z][:, None, None] - centre[0][at]) ** 2 + \
                (pos[1][:, None] - centre[1][at]) ** 2 + (pos[2][None, :] - centre[2][at]) ** 2
            f[z] = (d2 <= r[at] ** 2).to(torch.uint8) * SOLID
    return f


def _velocity(case, seed, salt, amplitude=0.02):
    """A smooth velocity [3, nz, ny, nx] (float32): two waves per component."""
    nz, ny, nx = case["nz"], case["ny"], case["nx"]
    ph = 2 * math.pi * torch.rand(3, 2, generator=_generator(seed, salt))
    k = torch.randint(1, 4, (3, 2), generator=_generator(seed, salt + 1))
    ax = [2 * math.pi / s * torch.arange(s, device="cuda", dtype=torch.float32) for s in (nz, ny, nx)]
    x, y, z = ax[2][None, None, :], ax[1][None, :, None], ax[0][:, None, None]
    if case["geometry"] == "taylor_green":
        a, b = x + float(ph[0, 0]), y + float(ph[0, 1])
        u = [-0.01 * torch.cos(a) * torch.sin(b) + 0 * z, 0.01 * torch.sin(a) * torch.cos(b) + 0 * z,
             0 * (x + y + z)]
        return torch.stack(u).contiguous()
    u = torch.empty(3, nz, ny, nx, device="cuda")
    for c, (p, q) in enumerate(((y, z), (z, x), (x, y))):
        u[c] = 0.5 * amplitude * (torch.sin(int(k[c, 0]) * p + float(ph[c, 0])) +
                                  torch.sin(int(k[c, 1]) * q + float(ph[c, 1])))
    return u


def _wall_u(case):
    return LID if case["geometry"] == "cavity" else (0.0, 0.0, 0.0)


def _f16_scale(case):
    return (10 if case["geometry"] == "cavity" else 12) if case["storage"] == "f16" else 0


def prepare(case, seed):
    shape = (case["nz"], case["ny"], case["nx"])
    flags = _flags(case, seed)
    u0 = _velocity(case, seed, 11)
    if case["kind"] == "rollout":
        return {"kind": "rollout", "u0": u0.requires_grad_(), "flags": flags,
                "g": torch.tensor([case["fx"], 0.0, 0.0], dtype=torch.float64, requires_grad=True),
                "target": _velocity(case, seed, 21), "steps": case["steps"], "tau": case["tau"],
                "every": case["every"], "wall_u": _wall_u(case),
                "equilibrium": case["equilibrium"],
                "steps_per_pass": 2 if case["schedule"] == "2" else 0}
    schedule = {"1": 0, "2": 2, "auto": "auto"}[case["schedule"]]
    sim = LBM(shape, case["tau"], (case["fx"], 0.0, 0.0), case["storage"], flags=flags, u0=u0,
              f16_scale_log2=_f16_scale(case), wall_u=_wall_u(case),
              equilibrium=case["equilibrium"], steps_per_pass=schedule)
    return {"kind": case["kind"], "sim": sim, "steps": case["steps"]}


def run(state):
    if state["kind"] == "rollout":
        rho, u = rollout(state["u0"], state["g"], steps=state["steps"], tau=state["tau"],
                         flags=state["flags"], checkpoint_every=state["every"],
                         wall_u=state["wall_u"], equilibrium=state["equilibrium"],
                         steps_per_pass=state["steps_per_pass"])
        loss = ((u - state["target"]) ** 2).mean() + ((rho - 1.0) ** 2).mean()
        du0, dg = torch.autograd.grad(loss, (state["u0"], state["g"]))
        return {"rho": rho.detach(), "u": u.detach(), "du0": du0, "dg": dg}
    sim = state["sim"]
    if state["kind"] != "fields":
        sim.step(state["steps"])
    if state["kind"] == "steps":
        return {"f": sim.populations()[..., :sim.shape[2]]}
    rho, u = sim.macroscopics()
    return {"rho": rho, "u": u, "sums": sim.reduce()}


def work(case):
    """The state read once and written once, however many steps lie between."""
    cells = case["nz"] * case["ny"] * case["nx"]
    state = 19 * BYTES[case["storage"]]
    flags = 0 if case["geometry"] in ("box", "taylor_green") else 1
    flops = 250 * case["steps"]  # moments, equilibrium, relaxation, force of one update
    if case["kind"] == "rollout":  # velocity, target and flags in; fields and gradient out
        return {"bytes": cells * (12 + 12 + flags + 16 + 12), "flops": cells * (flops + 350 * case["steps"])}
    moved = state + flags
    if case["kind"] in ("steps", "sample"):
        moved += state
    if case["kind"] in ("sample", "fields"):
        moved += 16
        flops += 80
    return {"bytes": cells * moved, "flops": cells * flops}


# ---------------------------------------------------------------------------
# The same in 64 bits, in plain torch.
# ---------------------------------------------------------------------------
def _equilibrium(i, rho, u, incompressible):
    eu = sum(c * u[d] for d, c in enumerate(E[i]) if c)
    uu = u[0] * u[0] + u[1] * u[1] + u[2] * u[2]
    poly = 3 * eu + 4.5 * eu * eu - 1.5 * uu
    return W[i] * (rho + poly) if incompressible else W[i] * rho * (1 + poly)


def _initial(u0, solid, incompressible):
    u = u0.double()
    if solid is not None:
        u = torch.where(solid, torch.zeros((), dtype=torch.float64, device=u.device), u)
    rho = torch.ones_like(u[0])
    return torch.stack([_equilibrium(i, rho, u, incompressible) for i in range(19)])


def _step(f, force, solid, moving, tau, wall_u, incompressible, in_place=False):
    pulled = torch.empty_like(f) if in_place else [None] * 19
    for i, c in enumerate(E):
        shift = (c[2], c[1], c[0])
        v = torch.roll(f[i], shift, (0, 1, 2))
        if solid is not None and i:
            back = f[OPP[i]]
            kick = 6 * W[i] * sum(a * b for a, b in zip(c, wall_u))
            if kick:
                back = back + kick * torch.roll(moving, shift, (0, 1, 2))
            v = torch.where(torch.roll(solid, shift, (0, 1, 2)), back, v)
        pulled[i] = v
    rho = sum(pulled[i] for i in range(19))
    if solid is not None:
        rho = torch.where(solid, torch.ones_like(rho), rho)
    u = []
    for d in range(3):
        j = sum(E[i][d] * pulled[i] for i in range(19) if E[i][d]) + 0.5 * force[d]
        u.append(j if incompressible else j / rho)
    om = 1.0 / tau
    uF = u[0] * force[0] + u[1] * force[1] + u[2] * force[2]
    out = f if in_place else []
    for i in range(19):
        eu = sum(c * u[d] for d, c in enumerate(E[i]) if c)
        eF = sum(c * force[d] for d, c in enumerate(E[i]) if c)
        guo = (1 - 0.5 * om) * W[i] * (3 * (eF - uF) + 9 * eu * eF)
        v = pulled[i] + om * (_equilibrium(i, rho, u, incompressible) - pulled[i]) + guo
        if solid is not None:
            v = torch.where(solid, torch.zeros_like(v), v)
        if in_place:
            out[i] = v
        else:
            out.append(v)
    return out if in_place else torch.stack(out)


def _fields(f, force, solid, incompressible):
    rho = f.sum(0)
    safe = rho if solid is None else torch.where(solid, torch.ones_like(rho), rho)
    j = torch.stack([sum(E[i][d] * f[i] for i in range(19) if E[i][d]) - 0.5 * force[d]
                     for d in range(3)])
    u = j if incompressible else j / safe
    if solid is not None:
        zero = torch.zeros((), dtype=torch.float64, device=f.device)
        rho, u = torch.where(solid, zero, rho), torch.where(solid, zero, u)
    return rho, u


def exact(case, seed):
    flags = _flags(case, seed)
    solid = None if flags is None else (flags & SOLID) != 0
    moving = None if flags is None else ((flags & MOVING) != 0).double()
    incompressible = case["equilibrium"] == "incompressible"
    u0 = _velocity(case, seed, 11)
    force = torch.tensor([case["fx"], 0.0, 0.0], dtype=torch.float64, device="cuda")
    args = (solid, moving, case["tau"], _wall_u(case), incompressible)
    if case["kind"] == "rollout":
        from torch.utils.checkpoint import checkpoint
        u0.requires_grad_()
        force.requires_grad_()
        f = _initial(u0, solid, incompressible)
        for _ in range(case["steps"]):
            f = checkpoint(_step, f, force, *args, use_reentrant=False)
        rho, u = _fields(f, force, solid, incompressible)
        loss = ((u - _velocity(case, seed, 21)) ** 2).mean() + ((rho - 1.0) ** 2).mean()
        du0, dg = torch.autograd.grad(loss, (u0, force))
        return {"rho": rho.detach(), "u": u.detach(), "du0": du0.double(), "dg": dg.cpu()}
    f = _initial(u0, solid, incompressible)
    for _ in range(case["steps"]):
        f = _step(f, force, *args, in_place=True)
    if case["kind"] == "steps":
        for i in range(19):
            f[i] -= W[i]
        f *= 2.0 ** _f16_scale(case)
        if solid is not None:
            for i in range(19):
                f[i][solid] = math.nan  # a solid cell holds no state
        return {"f": f}
    rho, u = _fields(f, force, solid, incompressible)
    m = u if incompressible else rho * u
    sums = torch.stack([rho.sum(), m[0].sum(), m[1].sum(), m[2].sum(),
                        0.5 * (m * u).sum()])
    return {"rho": rho, "u": u, "sums": sums}
