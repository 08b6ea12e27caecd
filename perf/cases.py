"""Performance cases: the work that a program built on this library has it do.

Four kinds of call, each through the package's public entry points:

  steps     `pic_step`: a simulation advanced by a few steps with the sort
            schedule of the run (or, with sort_every 0, on the binning that
            the program holds), diagnostics after every step
  adjoint   `pic_step_adjoint`: one reverse step on a binned state
  rollout   `rollout_loss` and its gradient: the differentiable simulation,
            forward and backward
  ops       the separate operations `pic_gather`, `pic_push`, `pic_deposit`
            and `pic_yee`, from which a program with several species (which
            `pic_step` does not take) composes its own step

A case gives the grid, the particles per cell, the shape order, the precision
and the options.  A pass starts from the same state each time: one device copy
puts it back (a program that restarts from a checkpoint does the same).

Particle arrays are returned where the order of the particles is the
caller's.  After a sort the order inside a cell is not specified, so a pass
that sorts returns the fields, the current and the diagnostics, which depend
on every particle.  Momenta are returned rather than cell indices and
offsets: a position next to a cell face may carry either cell after any
rounding, and the current that is returned holds the displacements.
"""
import math
import types

import numpy as np
import torch

from paper_2101_12149_amd import _lib
from paper_2101_12149_amd import rollout
from paper_2101_12149_amd import workloads as wl

DEV = "cuda"


def _case(name, kind, n, ppc, order, dtype, u_th=0.05, nsteps=1, sort_every=0, vay=False, ckc=False, filt=False,
          laser=False, tile=(0, 0, 0), drift=2.0, every=0):
    c = dict(kind=kind, nx=n[0], ny=n[1], nz=n[2], ppc=ppc, order=order, dtype=dtype, u_th=u_th, nsteps=nsteps,
             sort_every=sort_every, vay=vay, ckc=ckc, filt=filt, laser=laser, tx=tile[0], ty=tile[1], tz=tile[2],
             drift=drift, every=every)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the uniform plasma of the benchmark: 8 particles per cell, third-order shapes, a sort every 4 steps
        _case("uniform256_f32", "steps", (256, 256, 256), 8, 3, "f32", nsteps=8, sort_every=4),
        # the same physics in double precision at an eighth of the volume
        _case("uniform128_f64", "steps", (128, 128, 128), 8, 3, "f64", nsteps=4, sort_every=4),
        # laser wakefield stage: cold plasma with a density ramp and weights, a pulse in the box, the source plane
        _case("laser_f32", "steps", (128, 128, 1024), 2, 3, "f32", u_th=0.0, nsteps=4, sort_every=4, laser=True),
        # the largest box: hot plasma, 2 particles per cell, sorts 20 steps apart
        _case("hot512_f32", "steps", (512, 512, 512), 2, 3, "f32", u_th=0.1, nsteps=4, sort_every=20),
        # the small first-order plasma of the benchmark
        _case("uniform32_o1_f64", "steps", (32, 32, 32), 8, 1, "f64", u_th=0.01, nsteps=10, sort_every=4),
        # one step of the smallest box, on a binning that is kept: a call that is mostly launches and its read-back
        _case("step16_f64", "steps", (16, 16, 16), 2, 3, "f64", nsteps=1, sort_every=0, tile=(8, 8, 4)),
        # accelerator-stage options (Vay, CKC, a filter before the gather) on a grid of uneven extents
        _case("options_f32", "steps", (100, 84, 175), 4, 3, "f32", u_th=0.2, nsteps=6, sort_every=3, vay=True,
              ckc=True, filt=True),
        # reverse step at the headline's density and shapes
        _case("adjoint128_f32", "adjoint", (128, 128, 128), 8, 3, "f32", tile=(8, 8, 8)),
        # reverse step of the laser stage, with the gradient of the source map
        _case("adjoint_laser_f32", "adjoint", (128, 128, 1024), 2, 3, "f32", u_th=0.0, laser=True, tile=(8, 8, 8)),
        # the differentiable workload: 20 steps forward, checkpoints every 5, and the reverse sweep
        _case("rollout64_f64", "rollout", (64, 64, 64), 4, 3, "f64", nsteps=20, every=5),
        # a gradient of the smallest size, as in a fit that takes many of them
        _case("rollout16_f64", "rollout", (16, 16, 16), 2, 3, "f64", nsteps=8, every=3),
        # two species stepped with the separate operations
        _case("ops64_f32", "ops", (64, 64, 64), 8, 3, "f32", tile=(8, 8, 8)),
    ]


def draw(rng):
    kind = rng.choice(("steps", "steps", "steps", "adjoint", "rollout", "ops"))
    dtype = rng.choice(("f32", "f32", "f64"))
    order = rng.choice((3, 3, 1))
    ppc = rng.choice((1, 2, 3, 4, 6, 8, 12))
    top = {"steps": 6e7, "adjoint": 3e7, "rollout": 2e6, "ops": 1e7}[kind] / (2.0 if dtype == "f64" else 1.0)
    parts = math.exp(rng.uniform(math.log(8e3), math.log(top)))
    edge = max(10.0, (parts / ppc) ** (1.0 / 3.0))
    stretch = [math.exp(rng.uniform(-0.5, 0.5)) for _ in range(3)]
    tile, n = [], []
    for d, s in enumerate(stretch):
        # (a tile with its halo in double precision has to fit one workgroup)
        t = rng.choice((3, 4)) if dtype == "f64" and d == 2 else rng.choice((4, 5, 6, 7, 8, 8))
        tile.append(t)
        n.append(t * max(2, int(round(edge * s / t))))
    u_th = rng.choice((0.01, 0.05, 0.1, 0.2))
    opt = rng.random() < 0.25
    kw = dict(u_th=u_th, vay=opt, ckc=opt and kind != "ops", filt=opt and kind != "ops" and rng.random() < 0.5)
    if kind == "steps":
        se = rng.choice((0, 1, 3, 4, 4, 8, 20))
        steps = rng.randint(1, 10)
        return _case("", kind, n, ppc, order, dtype, nsteps=steps, sort_every=se, drift=rng.choice((0.5, 1.0, 2.0)), **kw)
    if kind == "adjoint":
        return _case("", kind, n, ppc, order, dtype, tile=tile, drift=rng.choice((0.0, 1.0, 2.0, 4.0)), **kw)
    if kind == "rollout":
        return _case("", kind, n, ppc, order, dtype, nsteps=rng.randint(4, 16), every=rng.randint(2, 6), **kw)
    return _case("", kind, n, ppc, order, dtype, tile=tile, **kw)


# ---------------------------------------------------------------------------
# inputs, from the seed alone

def _grid(c):
    n, tile = (c["nx"], c["ny"], c["nz"]), (c["tx"], c["ty"], c["tz"])
    if c["laser"]:   # spacing of the laser stage: 16 cells per wavelength along z, 80 wavelengths across
        lam = 2.0 * math.pi
        d = (80.0 * lam / n[0], 80.0 * lam / n[1], lam / 16.0)
        dt = 0.99 / math.sqrt(sum(1.0 / v ** 2 for v in d))
        g = wl.Grid(n, d, dt, order=c["order"], tile=tile)
    else:
        g = wl.plasma_grid(n, c["order"], tile=tile)
    g.pusher, g.solver = int(c["vay"]), int(c["ckc"])
    if c["filt"]:    # a binomial filter along z before the gather
        g.gather_filter = tuple((0.5, 0.25, 0.0, 0.0) for _ in range(6))
    return g


def _tdt(c):
    return torch.float64 if c["dtype"] == "f64" else torch.float32


def _ramp(c):
    """First plasma cell along z and the length of the density ramp (laser stage)."""
    return (c["nz"] // 32, max(1, c["nz"] // 10)) if c["laser"] else (0, 0)


def _cells(c, tile):
    """Exactly ppc particles in every cell (from the ramp's first plane on), in
    tile-major order, inside a tile one particle of every cell after the
    other: the order that the sort documents for such a load.  (3, N) int32."""
    n = (c["nx"], c["ny"], c["nz"])
    lin = torch.arange(n[0] * n[1] * n[2] * c["ppc"], device=DEV, dtype=torch.int64)

    def split(m):
        r = lin % m
        torch.div(lin, m, rounding_mode="floor", out=lin)
        return r.to(torch.int32)
    loc = [split(t) for t in tile]
    split(c["ppc"])
    cell = torch.stack([split(n[d] // tile[d]) * tile[d] + loc[d] for d in range(3)])
    k0 = _ramp(c)[0]
    return cell[:, cell[2] >= k0].contiguous() if k0 else cell


def _below_one(off):
    one = torch.ones((), dtype=off.dtype, device=off.device)
    return torch.where(off >= 1, torch.nextafter(one, 0 * one), off)


def _species(c, g, cell, seed, q=-1.0, m=1.0, u_th=None):
    """Offsets uniform in the cell, thermal momenta (in the pulse of a laser
    case also the quiver momentum), weights from the ramp."""
    gen = torch.Generator(device=DEV)
    gen.manual_seed(int(seed))
    dt, n = _tdt(c), int(cell.shape[1])
    u_th = c["u_th"] if u_th is None else u_th
    off = _below_one(torch.rand((3, n), generator=gen, dtype=dt, device=DEV))
    u = torch.randn((3, n), generator=gen, dtype=dt, device=DEV) * u_th
    w = None
    if c["laser"]:
        k0, length = _ramp(c)
        z = cell[2].to(dt) + off[2]
        w = (torch.clamp((z - k0) / length, 0.0, 1.0) * 0.01 * g.dV / c["ppc"]).contiguous()
        u[0] += _pulse(c, g, z, torch.cos)
    return wl.Species(cell, off, u, w, g.dV / c["ppc"] if w is None else 0.0, q, m)


def _pulse(c, g, z, osc, a0=1.0):
    """A plane pulse in mid-box, along z (z in cells)."""
    zc, s = 0.5 * c["nz"], c["nz"] / 16.0
    return a0 * torch.exp(-((z - zc) / s) ** 2) * osc((z - zc) * g.d[2])


def _move(c, g, sp):
    """The state some steps after its binning: every particle drifts freely."""
    if c["drift"] <= 0:
        return
    ig = 1.0 / torch.sqrt(1.0 + (sp.u.double() ** 2).sum(0))
    for d in range(3):
        x = sp.off[d].double() + (c["drift"] * g.dt / g.d[d]) * sp.u[d].double() * ig
        k = torch.floor(x)
        f = (x - k).to(sp.off.dtype)
        sp.off[d] = _below_one(f)
        sp.cell[d] = torch.remainder(sp.cell[d] + k.to(torch.int32), g.n[d])


def _fields(c, g, seed):
    """Thermal field noise; the laser's pulse travels along +z."""
    gen = torch.Generator(device=DEV)
    gen.manual_seed(int(seed) + 77)
    shape = (3, c["nz"], c["ny"], c["nx"])
    E = torch.randn(shape, generator=gen, dtype=_tdt(c), device=DEV) * 0.01
    B = torch.randn(shape, generator=gen, dtype=_tdt(c), device=DEV) * 0.01
    if c["laser"]:
        k = torch.arange(c["nz"], device=DEV, dtype=torch.float64)
        E[0] += _pulse(c, g, k, torch.sin).to(E.dtype)[:, None, None]
        B[1] += _pulse(c, g, k + 0.5, torch.sin).to(E.dtype)[:, None, None]
    return E, B


def _source(c, g, seed):
    """Plane source: the laser's, or the rollout's map of amplitudes."""
    if not (c["laser"] or c["kind"] == "rollout"):
        return None
    x = (torch.arange(c["nx"], dtype=torch.float64, device=DEV) + 0.5) / c["nx"] - 0.5
    y = torch.arange(c["ny"], dtype=torch.float64, device=DEV) / c["ny"] - 0.5
    gen = torch.Generator(device=DEV)
    gen.manual_seed(int(seed) + 99)
    amp = 1e-2 * torch.exp(-(y[:, None] ** 2 + x[None, :] ** 2) * 16.0)
    amp = amp * (1.0 + 0.1 * torch.randn(amp.shape, generator=gen, dtype=torch.float64, device=DEV))
    return wl.Source(2, amp.to(_tdt(c)).contiguous(), np.sin(2.0 * math.pi * (np.arange(64) + 1.0) / 16.0))


def _lam(c, g, n, seed):
    """Incoming gradients of a reverse step."""
    gen = torch.Generator(device=DEV)
    gen.manual_seed(int(seed) + 55)
    shape = (3, c["nz"], c["ny"], c["nx"])

    def draw_(s, a):
        return torch.randn(s, generator=gen, dtype=_tdt(c), device=DEV) * a
    return dict(lx=draw_((3, n), 0.1), lu=draw_((3, n), 0.1), lE=draw_(shape, 1.0), lB=draw_(shape, 1.0))


def _inputs(c, seed):
    """Grid, list of species, fields and source of a case.  The tile given by
    the case fixes the particles' order; a case without one lists the cells in
    tiles of one cell (cell by cell)."""
    g = _grid(c)
    tile = (c["tx"], c["ty"], c["tz"]) if c["tx"] else (1, 1, 1)
    cell = _cells(c, tile)
    sps = [_species(c, g, cell, seed)]
    if c["kind"] == "ops":
        sps.append(_species(c, g, cell.clone(), seed + 1, q=1.0, m=1836.0, u_th=c["u_th"] / 40.0))
    E, B = _fields(c, g, seed)
    return g, sps, E, B, _source(c, g, seed)


# ---------------------------------------------------------------------------
# states

def _pack(tensors):
    """Copies of the tensors in one buffer, and views of a second buffer of
    the same layout: state.copy_(initial) restores them all."""
    offs, o = [], 0
    for t in tensors:
        offs.append(o)
        o += (t.numel() * t.element_size() + 255) // 256 * 256
    first = torch.zeros(o, dtype=torch.uint8, device=DEV)
    live = torch.empty_like(first)

    def views(buf):
        return [buf[a:a + t.numel() * t.element_size()].view(t.dtype).view(t.shape) for a, t in zip(offs, tensors)]
    for v, t in zip(views(first), tensors):
        v.copy_(t)
    return first, live, views(first), views(live)


def _arrays(sp):
    return [sp.cell, sp.off, sp.u] + ([sp.w] if sp.w is not None else [])


def _like(sp, arrays):
    return wl.Species(arrays[0], arrays[1], arrays[2], arrays[3] if sp.w is not None else None, sp.w0, sp.q, sp.m)


def prepare(case, seed):
    c = case
    g, sps, E, B, src = _inputs(c, seed)
    sp, dt = sps[0], c["dtype"]
    s = types.SimpleNamespace(c=c, g=g, src=src)
    if c["kind"] == "rollout":
        f = wl.Fields(E, B, torch.zeros_like(E))
        s.u0 = sp.u.clone().requires_grad_(True)
        s.amp = src.amp.clone().requires_grad_(True)
        s.pb = rollout.Problem(g, sp, f, src, c["nsteps"], c["every"], _tdt(c))
        return s
    if c["kind"] == "ops":
        for q in sps:
            _move(c, g, q)
        ten = [a for q in sps for a in _arrays(q)] + [E, B]
        s.first, s.live, v0, v1 = _pack(ten)
        s.sps, s.before = [], []
        for q in sps:
            k = len(_arrays(q))
            s.before.append(_like(q, v0[:k]))
            s.sps.append(_like(q, v1[:k]))
            v0, v1 = v0[k:], v1[k:]
        s.f = wl.Fields(v1[0], v1[1], torch.zeros_like(E))
        s.EpBp = [(torch.empty_like(q.off), torch.empty_like(q.off)) for q in sps]
        return s
    s.ws = _lib.workspace(g, dt, sp.n)
    s.ts = torch.zeros(_lib.pic_tile_count(g, dt) + 1, dtype=torch.int32, device=DEV)
    if c["tx"]:
        # the binning of the cells: the particles' order inside a cell stays the drawn one
        cells = wl.Species(sp.cell.clone(), torch.zeros_like(sp.off), torch.zeros_like(sp.u), None, 1.0)
        _lib.pic_sort_tiles(g, cells, s.ts, s.ws)
        del cells
    else:
        _lib.pic_sort_tiles(g, sp, s.ts, s.ws)
    _move(c, g, sp)
    if c["kind"] == "steps":
        s.first, s.live, _, v = _pack(_arrays(sp) + [E, B])
        s.sp = _like(sp, v[:-2])
        s.f = wl.Fields(v[-2], v[-1], torch.zeros_like(E))
        s.diag = torch.zeros((c["nsteps"], 5), dtype=torch.float64, device=DEV)
        return s
    s.sp, s.f = sp, wl.Fields(E, B, torch.zeros_like(E))
    lam = _lam(c, g, sp.n, seed)
    dA = torch.zeros((c["ny"], c["nx"]), dtype=torch.float64, device=DEV)
    s.first, s.live, _, v = _pack(list(lam.values()) + [dA])
    s.lam = types.SimpleNamespace(**dict(zip(lam, v)))
    s.dA = v[4] if src is not None else None
    return s


def run(s):
    c, g = s.c, s.g
    if c["kind"] == "rollout":
        loss = rollout.rollout_loss(s.u0, s.amp, s.pb)
        du0, damp = torch.autograd.grad(loss, (s.u0, s.amp))
        return {"loss": loss.detach(), "du0": du0, "damp": damp}
    s.live.copy_(s.first)
    if c["kind"] == "steps":
        _lib.pic_step(g, s.sp, s.f, s.src, 0, c["nsteps"], c["sort_every"], s.ts, s.ws, s.diag)
        out = {"E": s.f.E, "B": s.f.B, "J": s.f.J, "diag": s.diag}
        if c["sort_every"] == 0 and c["tx"]:
            out["u"] = s.sp.u
        return out
    if c["kind"] == "adjoint":
        _lib.pic_step_adjoint(g, s.sp, s.f, s.src, 3, s.lam, s.dA, s.ws, tile_start=s.ts)
        out = {"lx": s.lam.lx, "lu": s.lam.lu, "lE": s.lam.lE, "lB": s.lam.lB}
        if s.dA is not None:
            out["dA"] = s.dA
        return out
    s.f.J.zero_()
    out = {}
    for k, (sp, before, (Ep, Bp)) in enumerate(zip(s.sps, s.before, s.EpBp)):
        _lib.pic_gather(g, sp, s.f, Ep, Bp)
        _lib.pic_push(g, sp, Ep, Bp)
        _lib.pic_deposit(g, before, sp, s.f)
        out["u%d" % k], out["Ep%d" % k], out["Bp%d" % k] = sp.u, Ep, Bp
    _lib.pic_yee(g, s.f)
    out.update(E=s.f.E, B=s.f.B, J=s.f.J)
    return out


def work(case):
    """Bytes: the particle state read and written once a step (cell, offset,
    momentum; the weight read), E and B read, E, B and J written once a step;
    a reverse step reads the state and reads and writes its gradients.  Flops:
    the arithmetic of a particle that stays in its cell (weights, six gathered
    components, push, Esirkepov sums), and for a reverse step the forward
    recomputation with three derivatives of each component, the deposit's
    transpose and the scatter of six components."""
    c = case
    n, ts = c["nx"] * c["ny"] * c["nz"], 8 if c["dtype"] == "f64" else 4
    npart = (c["nz"] - _ramp(c)[0]) * c["nx"] * c["ny"] * c["ppc"]
    state = 12 + 6 * ts
    wb = ts if c["laser"] else 0
    f_fwd = 2028 if c["order"] == 3 else 411
    f_adj = 3 * f_fwd
    fwd = {"bytes": npart * (2 * state + wb) + 15 * ts * n, "flops": npart * f_fwd + 36 * n}
    adj = {"bytes": npart * (state + wb + 12 * ts) + 18 * ts * n, "flops": npart * f_adj + 36 * n}
    if c["kind"] == "steps":
        per, k = fwd, c["nsteps"]
        return {"bytes": per["bytes"] * k, "flops": per["flops"] * k}
    if c["kind"] == "adjoint":
        return adj
    if c["kind"] == "ops":   # gathered fields written and read between the calls
        return {"bytes": 2 * npart * (2 * state + 12 * ts) + 15 * ts * n, "flops": 2 * npart * f_fwd + 36 * n}
    return {k: c["nsteps"] * (fwd[k] + adj[k]) for k in ("bytes", "flops")}


# ---------------------------------------------------------------------------
# the same results in 64 bits, with torch alone

CHUNK = 1 << 17
SX, SY, SZ = (1, 0, 0, 0, 1, 1), (0, 1, 0, 1, 0, 1), (0, 0, 1, 1, 1, 0)   # staggering of E_x .. B_z


def _spline(order, x):
    a = x.abs()
    if order == 1:
        return torch.clamp(1.0 - a, min=0.0)
    near = 2.0 / 3.0 - a * a + 0.5 * a ** 3
    far = torch.clamp(2.0 - a, min=0.0) ** 3 / 6.0
    return torch.where(a < 1.0, near, far)


def _weights(order, x, stag, lo, count):
    j = torch.arange(lo, lo + count, device=x.device, dtype=torch.float64)
    return _spline(order, x[None, :] - j[:, None] - 0.5 * stag)


def _nodes(n, cell, lo, count):
    j = torch.arange(lo, lo + count, device=cell.device)
    return torch.remainder(cell.long()[None, :] + j[:, None], n)


def _linear(g, idx):
    """Linear index of the nodes idx[x], idx[y], idx[z]: (z, y, x, particle)."""
    return (idx[2][:, None, None] * g.n[1] + idx[1][None, :, None]) * g.n[0] + idx[0][None, None, :]


def _gather(g, cell, off, EB):
    lo, cnt = (-2, 5) if g.order == 3 else (-1, 3)
    lin = _linear(g, [_nodes(g.n[d], cell[d], lo, cnt) for d in range(3)])
    wt = [[_weights(g.order, off[d], s, lo, cnt) for s in (0, 1)] for d in range(3)]
    got = []
    for m in range(6):
        v = EB[m].reshape(-1).gather(0, lin.reshape(-1)).reshape(lin.shape)
        v = (v * wt[0][SX[m]][None, None]).sum(2)
        v = (v * wt[1][SY[m]][None]).sum(1)
        got.append((v * wt[2][SZ[m]]).sum(0))
    return torch.stack(got[:3]), torch.stack(got[3:])


def _cross(a, b):
    return torch.stack([a[1] * b[2] - a[2] * b[1], a[2] * b[0] - a[0] * b[2], a[0] * b[1] - a[1] * b[0]])


def _push(g, sp, u, E, B):
    h, ic2 = sp.q * g.dt / (2.0 * sp.m), 1.0 / g.c ** 2
    if g.pusher == 0:
        um = u + h * E
        t = h * B / torch.sqrt(1.0 + (um * um).sum(0) * ic2)
        up = um + _cross(um, t)
        return um + _cross(up, 2.0 * t / (1.0 + (t * t).sum(0))) + h * E
    v0 = u / torch.sqrt(1.0 + (u * u).sum(0) * ic2)
    w, tau = u + 2.0 * h * E + h * _cross(v0, B), h * B
    tau2 = (tau * tau).sum(0)
    sg = 1.0 + (w * w).sum(0) * ic2 - tau2
    t = tau / torch.sqrt(0.5 * (sg + torch.sqrt(sg * sg + 4.0 * (tau2 + (w * tau).sum(0) ** 2 * ic2))))
    return (w + (w * t).sum(0) * t + _cross(w, t)) / (1.0 + (t * t).sum(0))


def _advance(g, sp, u, off, E, B):
    """u1 and the new position in the old cell's frame."""
    u1 = _push(g, sp, u, E, B)
    ig = 1.0 / torch.sqrt(1.0 + (u1 * u1).sum(0) / g.c ** 2)
    dtd = torch.tensor([g.dt / v for v in g.d], dtype=torch.float64, device=u.device)
    return u1, off + dtd[:, None] * u1 * ig


def _current(g, sp, cell, x0, x1, w):
    """Esirkepov's current of particles moving from x0 to x1 (frame of the
    cell): node indices and the three components' values there."""
    lo, cnt = (-2, 6) if g.order == 3 else (-1, 4)
    lin = _linear(g, [_nodes(g.n[d], cell[d], lo, cnt) for d in range(3)])
    S0 = [_weights(g.order, x0[d], 0, lo, cnt) for d in range(3)]
    S1 = [_weights(g.order, x1[d], 0, lo, cnt) for d in range(3)]
    vals = []
    for m in range(3):
        p, q = (m + 1) % 3, (m + 2) % 3

        def ax(v, d):
            return v[None, None] if d == 0 else (v[None, :, None] if d == 1 else v[:, None, None])
        a0, a1, b0, b1 = ax(S0[p], p), ax(S1[p], p), ax(S0[q], q), ax(S1[q], q)
        C = (a0 * b0 + a1 * b1) / 3.0 + (a1 * b0 + a0 * b1) / 6.0
        P = torch.cumsum(S1[m] - S0[m], 0) * (-sp.q * w / (g.dt * g.d[p] * g.d[q]))
        vals.append(ax(P, m) * C)
    return lin, vals


def _chunks(n):
    return [slice(a, min(a + CHUNK, n)) for a in range(0, n, CHUNK)]


def _weight(sp, s):
    return sp.w[s].double() if sp.w is not None else sp.w0


def _filtered(g, EB):
    if not g.gather_filter:
        return EB
    return [w[0] * F + sum(w[k] * (torch.roll(F, k, 0) + torch.roll(F, -k, 0)) for k in (1, 2, 3) if w[k])
            for F, w in zip(EB, g.gather_filter)]


def _diff(g, F, a, sign, ckc=False):
    """Difference of F along axis a divided by the spacing, to the next
    (sign 1) or previous node; with ckc averaged across the axis."""
    dim = 2 - a
    D = (torch.roll(F, -1, dim) - F) if sign > 0 else (F - torch.roll(F, 1, dim))
    if ckc:
        dl = min(g.d)
        r = [(dl / v) ** 2 for v in g.d]
        S = r[0] * r[1] + r[1] * r[2] + r[2] * r[0]
        p, q = (a + 1) % 3, (a + 2) % 3
        beta = (1.0 - r[0] * r[1] * r[2] / S) / 8.0
        bp, bq = r[p] * beta, r[q] * beta
        gm = r[p] * r[q] * (1.0 / 16.0 - r[p] * r[q] / (8.0 * S))

        def both(v, d):
            return torch.roll(v, 1, 2 - d) + torch.roll(v, -1, 2 - d)
        D = (1.0 - 2 * bp - 2 * bq - 4 * gm) * D + bp * both(D, p) + bq * both(D, q) + gm * both(both(D, p), q)
    return D / g.d[a]


def _curl(g, F, sign, ckc=False):
    def d(m, a):
        return _diff(g, F[m], a, sign, ckc)
    return [d(2, 1) - d(1, 2), d(0, 2) - d(2, 0), d(1, 0) - d(0, 1)]


def _field_step(g, E, B, J, amp, k_plane, gn):
    ckc = g.solver == 1
    B = [b - 0.5 * g.dt * v for b, v in zip(B, _curl(g, E, 1, ckc))]
    E = [e + g.dt * (g.c ** 2 * v - j / g.eps0) for e, v, j in zip(E, _curl(g, B, -1), J)]
    if amp is not None and gn:
        plane = torch.zeros_like(E[0])
        plane[k_plane] = 1.0
        E[0] = E[0] + plane * amp[None] * gn
    B = [b - 0.5 * g.dt * v for b, v in zip(B, _curl(g, E, 1, ckc))]
    return E, B


def _step64(g, sp, st, E, B, amp, src, step):
    """One step of the state st = (cell, off, u) in place of the caller's;
    returns cell, off, u, E, B, J."""
    cell, off, u = st
    EB = _filtered(g, list(E) + list(B))
    J = [torch.zeros_like(E[0]) for _ in range(3)]
    c1, o1, v1 = torch.empty_like(cell), torch.empty_like(off), torch.empty_like(u)
    for s in _chunks(cell.shape[1]):
        Ep, Bp = _gather(g, cell[:, s], off[:, s], EB)
        u1, x1 = _advance(g, sp, u[:, s], off[:, s], Ep, Bp)
        lin, vals = _current(g, sp, cell[:, s], off[:, s], x1, _weight(sp, s))
        for m in range(3):
            J[m].view(-1).index_add_(0, lin.reshape(-1), vals[m].reshape(-1))
        k = torch.floor(x1)
        v1[:, s], o1[:, s] = u1, x1 - k
        for d in range(3):
            c1[d, s] = torch.remainder(cell[d, s] + k[d].to(cell.dtype), g.n[d])
    gn = float(src.g[step]) if src is not None and step < len(src.g) else 0.0
    E, B = _field_step(g, E, B, J, amp, src.k_plane if src is not None else -1, gn)
    return (c1, o1, v1), E, B, J


def _diag64(g, sp, u, E, B):
    dV = g.d[0] * g.d[1] * g.d[2]
    w = sp.w.double() if sp.w is not None else torch.full_like(u[0], sp.w0)
    uu = (u * u).sum(0) / g.c ** 2
    return torch.stack([0.5 * dV * g.eps0 * sum((e * e).sum() for e in E),
                        0.5 * dV * g.eps0 * g.c ** 2 * sum((b * b).sum() for b in B),
                        sp.m * g.c ** 2 * (w * uu / (torch.sqrt(1.0 + uu) + 1.0)).sum(),
                        sp.q * w.sum(), sp.m * (w * u[2]).sum()])


def _reverse64(g, sp, st, E, B, amp, src, step, lam):
    """Gradients (lx, lu, lE, lB, damp) with respect to the step's inputs from
    those with respect to its outputs."""
    cell, off, u = st
    lx, lu, lE, lB = lam
    grid = [v.detach().clone().requires_grad_(True) for v in list(E) + list(B)]
    J = [torch.zeros_like(E[0]).requires_grad_(True) for _ in range(3)]
    am = amp.detach().clone().requires_grad_(True) if amp is not None else None
    gn = float(src.g[step]) if src is not None and step < len(src.g) else 0.0
    E1, B1 = _field_step(g, grid[:3], grid[3:], J, am, src.k_plane if src is not None else -1, gn)
    phi = sum((a * b).sum() for a, b in zip(E1 + B1, list(lE) + list(lB)))
    ins = grid + J + ([am] if am is not None and gn else [])
    got = torch.autograd.grad(phi, ins)
    gE, gJ = list(got[:6]), got[6:9]
    gA = got[9] if len(got) > 9 else (torch.zeros_like(amp) if amp is not None else None)
    EB = [v.detach().requires_grad_(True) for v in _filtered(g, [v.detach() for v in grid])]
    acc = [torch.zeros_like(v) for v in EB]
    gx, gu = torch.empty_like(off), torch.empty_like(u)
    for s in _chunks(cell.shape[1]):
        x = off[:, s].detach().clone().requires_grad_(True)
        v = u[:, s].detach().clone().requires_grad_(True)
        Ep, Bp = _gather(g, cell[:, s], x, EB)
        u1, x1 = _advance(g, sp, v, x, Ep, Bp)
        lin, vals = _current(g, sp, cell[:, s], x, x1, _weight(sp, s))
        p = (lx[:, s] * x1).sum() + (lu[:, s] * u1).sum()
        for m in range(3):
            p = p + (vals[m] * gJ[m].reshape(-1)[lin.reshape(-1)].reshape(lin.shape)).sum()
        d = torch.autograd.grad(p, [x, v] + EB)
        gx[:, s], gu[:, s] = d[0], d[1]
        for a, b in zip(acc, d[2:]):
            a += b
    acc = _filtered(g, acc)   # the filter is symmetric
    gE = [a + b for a, b in zip(gE, acc)]
    return (gx, gu, gE[:3], gE[3:]), gA


def exact(case, seed):
    c = case
    n = c["nx"] * c["ny"] * c["nz"] * c["ppc"]
    limit = {"steps": 1.5e8, "adjoint": 4e7, "rollout": 2.5e7, "ops": 1e7}[c["kind"]]
    if n * c["nsteps"] > limit:
        return None
    g, sps, E, B, src = _inputs(c, seed)
    E, B = [v.double() for v in E], [v.double() for v in B]
    amp = src.amp.double() if src is not None else None

    def state(sp):
        return sp.cell, sp.off.double(), sp.u.double()
    if c["kind"] == "ops":
        out, J = {}, [torch.zeros_like(E[0]) for _ in range(3)]
        for k, sp in enumerate(sps):
            _move(c, g, sp)
            cell, off, u = state(sp)
            u1s, Eps, Bps = torch.empty_like(u), torch.empty_like(u), torch.empty_like(u)
            for s in _chunks(cell.shape[1]):
                Eps[:, s], Bps[:, s] = _gather(g, cell[:, s], off[:, s], E + B)
                u1s[:, s], x1 = _advance(g, sp, u[:, s], off[:, s], Eps[:, s], Bps[:, s])
                lin, vals = _current(g, sp, cell[:, s], off[:, s], x1, _weight(sp, s))
                for m in range(3):
                    J[m].view(-1).index_add_(0, lin.reshape(-1), vals[m].reshape(-1))
            out["u%d" % k], out["Ep%d" % k], out["Bp%d" % k] = u1s, Eps, Bps
        E, B = _field_step(g, E, B, J, None, -1, 0.0)
        out.update(E=torch.stack(E), B=torch.stack(B), J=torch.stack(J))
        return out
    sp = sps[0]
    if c["kind"] == "adjoint":
        _move(c, g, sp)
        lam = {k: v.double() for k, v in _lam(c, g, sp.n, seed).items()}
        (gx, gu, gE, gB), gA = _reverse64(g, sp, state(sp), E, B, amp, src, 3,
                                          (lam["lx"], lam["lu"], lam["lE"], lam["lB"]))
        out = {"lx": gx, "lu": gu, "lE": torch.stack(gE), "lB": torch.stack(gB)}
        if gA is not None:
            out["dA"] = gA
        return out
    st = None
    if c["kind"] == "steps":
        _move(c, g, sp)
        st, diag = state(sp), []
        for i in range(c["nsteps"]):
            st, E, B, J = _step64(g, sp, st, E, B, amp, src, i)
            diag.append(_diag64(g, sp, st[2], E, B))
        out = {"E": torch.stack(E), "B": torch.stack(B), "J": torch.stack(J), "diag": torch.stack(diag)}
        if c["sort_every"] == 0 and c["tx"]:
            out["u"] = st[2]
        return out
    # rollout: the states of every step, then the reverse sweep
    st, states = state(sp), []
    for i in range(c["nsteps"]):
        states.append((st, E, B))
        st, E, B, _ = _step64(g, sp, st, E, B, amp, src, i)
    dV = g.d[0] * g.d[1] * g.d[2]
    k = (g.eps0 * dV, g.eps0 * g.c ** 2 * dV)
    loss = 0.5 * k[0] * sum((e * e).sum() for e in E) + 0.5 * k[1] * sum((b * b).sum() for b in B)
    lam = (torch.zeros_like(st[1]), torch.zeros_like(st[2]), [k[0] * e for e in E], [k[1] * b for b in B])
    damp = torch.zeros_like(amp)
    for i in reversed(range(c["nsteps"])):
        st, E, B = states[i]
        lam, gA = _reverse64(g, sp, st, E, B, amp, src, i, lam)
        damp += gA
    return {"loss": loss, "du0": lam[1], "damp": damp}
