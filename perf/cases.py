"""Timed cases of the force library: the calls that a program using it makes, at the sizes and
options it makes them with.

Every case goes through the Python binding of the C ABI (`paper_1601_03138_amd.fdx`).  A case
is a dict of plain values; its "kind" says which calls a pass makes:

  force    Context.calc_force on device-resident particles, forces fetched into device arrays
  step     Context.integrate, one eager leapfrog step, then forces and state
  graph    Context.integrate with graph=True, steps of several systems replayed as a HIP graph
  noalloc  calc_force_noalloc, the entry point for programs that may not allocate
  density  Context.calc_density, the neighbour search and SPH density
  treepm   Context.calc_force_cutoff, the tree part of TreePM
  exchange Context.build_exchange_lists and the lists on the host, as a sender ships them

Particles are drawn on the GPU from the seed: Plummer spheres, Plummer sub-clusters in a Plummer
background, uniform cubes -- the distributions of the benchmark and the tests.  Forces of the
FP32 path, and the velocities that it advances, are handed on in float32, the precision they
hold; FP64 results stay float64.
"""
from __future__ import annotations

import math
import os

import numpy as np
import torch

from paper_1601_03138_amd import fdx

WEIGHTS = os.path.join(os.path.dirname(os.path.abspath(fdx.__file__)),
                       "predictor_clustered16m_ng256.bin")
N_LEAF = 8
NMAX_NOALLOC = 1 << 16          # its scratch array holds the lists of this many particles
EXACT_PAIRS = 4e10              # direct sums up to this many pairs (a few seconds)


def listed():
    return [
        # smallest call: the plain-method configuration, FP64 monopole, one workgroup per group
        dict(name="plummer4k_fp64_mono", kind="force", dist="plummer", n=4096, theta=0.5,
             n_group=64, quad=False, fp32=False, persistent=False, predictor=False),
        # a serving loop that may not allocate: one small ragged set, FP32 quadrupole
        dict(name="noalloc21k_fp32", kind="noalloc", dist="plummer", n=21013, theta=0.6,
             n_group=64, quad=True, fp32=True, persistent=True),
        # the FP64 path of the million-body configuration
        dict(name="plummer1m_fp64", kind="force", dist="plummer", n=1 << 20, theta=0.5,
             n_group=256, quad=True, fp32=False, persistent=False, predictor=False),
        # its leapfrog step on the FP32 path, binding defaults (direct launch)
        dict(name="plummer1m_fp32_step", kind="step", dist="plummer", n=1 << 20, theta=0.5,
             n_group=256, quad=True, fp32=True, persistent=False, predictor=False,
             dt=1.0 / 256.0),
        # an ordinary odd-sized clustered set, exact two-pass walk, smaller groups
        dict(name="clustered3m_fp32", kind="force", dist="clustered", n=3000017, theta=0.6,
             n_group=128, quad=True, fp32=True, persistent=True, predictor=False),
        # the headline workload: 2^24 clustered, learned list sizes, one leapfrog step
        dict(name="clustered16m_fp32_step", kind="step", dist="clustered", n=1 << 24, theta=0.5,
             n_group=256, quad=True, fp32=True, persistent=True, predictor=True,
             dt=1.0 / 1024.0),
        # the batched ensemble: 512 Plummer systems of 1024..65536, graph-replayed steps
        dict(name="ensemble512_graph", kind="graph", dist="ensemble", n_sys=512, nmin=1024,
             nmax=65536, theta=0.6, n_group=128, quad=True, fp32=True, fused=False,
             dt=1.0 / 256.0, steps=1),
        # a small ensemble, walk and force in one launch: launches and latency count
        dict(name="ensemble24_fused_graph", kind="graph", dist="ensemble", n_sys=24, nmin=500,
             nmax=8000, theta=0.6, n_group=64, quad=True, fp32=True, fused=True,
             dt=1.0 / 256.0, steps=1),
        # SPH density of the benchmark: fixed cutoff of 4.2 mean spacings, about 300 neighbours
        dict(name="density16m_fixed", kind="density", dist="cube", n=1 << 24, mode=0, k=4.2,
             n_group=64),
        # per-particle radii in both directions on a ragged set
        dict(name="density700k_symmetric", kind="density", dist="cube", n=700001, mode=3, k=4.2,
             n_group=64),
        # tree part of TreePM: monopole with the S2 cutoff of three mesh widths
        dict(name="treepm16m_fp32", kind="treepm", dist="cube", n=1 << 24, theta=0.5,
             n_group=256, fp32=True, persistent=True),
        # lists that 27 domains send each other
        dict(name="exchange600k_27domains", kind="exchange", dist="plummer", n=600011, domains=3,
             theta=0.5),
    ]


def draw(rng):
    def logint(a, b):
        return int(round(math.exp(rng.uniform(math.log(a), math.log(b))))) | rng.randint(0, 1)

    kind = rng.choice(["force", "force", "step", "graph", "noalloc", "density", "treepm",
                       "exchange"])
    theta = round(rng.uniform(0.45, 0.8), 3)
    n_group = rng.choice([32, 64, 100, 128, 256, 512])
    if kind in ("force", "step"):
        fp32 = rng.random() < 0.7
        n = logint(1500, 12_000_000 if fp32 else 3_000_000)
        c = dict(kind=kind, dist=rng.choice(["plummer", "clustered", "cube"]), n=n, theta=theta,
                 n_group=n_group, quad=rng.random() < 0.8, fp32=fp32,
                 persistent=rng.random() < 0.5, predictor=False)
        if kind == "step":
            c["dt"] = rng.choice([1.0 / 128.0, 1.0 / 256.0, 1.0 / 1024.0])
        return c
    if kind == "graph":
        nmin = logint(300, 4000)
        return dict(kind=kind, dist="ensemble", n_sys=rng.randint(2, 200), nmin=nmin,
                    nmax=nmin * rng.randint(1, 12), theta=theta, n_group=min(n_group, 256),
                    quad=rng.random() < 0.8, fp32=True, fused=rng.random() < 0.5,
                    dt=1.0 / 256.0, steps=rng.randint(1, 3))
    if kind == "noalloc":
        return dict(kind=kind, dist=rng.choice(["plummer", "cube"]), n=logint(300, NMAX_NOALLOC),
                    theta=theta, n_group=rng.choice([32, 64, 128]), quad=rng.random() < 0.5,
                    fp32=rng.random() < 0.5, persistent=rng.random() < 0.5)
    if kind == "density":
        return dict(kind=kind, dist="cube", n=logint(2000, 6_000_000), mode=rng.randint(0, 3),
                    k=round(rng.uniform(2.0, 4.6), 2), n_group=rng.choice([32, 64, 128]))
    if kind == "treepm":
        return dict(kind=kind, dist="cube", n=logint(4000, 10_000_000), theta=theta,
                    n_group=n_group, fp32=rng.random() < 0.7, persistent=rng.random() < 0.5)
    return dict(kind=kind, dist=rng.choice(["plummer", "cube"]), n=logint(30_000, 590_000),
                domains=rng.randint(2, 3), theta=theta)


# -- particles ---------------------------------------------------------------------------------

def _rand(g, *shape):
    return torch.rand(*shape, generator=g, device="cuda", dtype=torch.float64)


def _directions(g, n):
    cth = 2.0 * _rand(g, n) - 1.0
    phi = (2.0 * math.pi) * _rand(g, n)
    sth = torch.sqrt(1.0 - cth * cth)
    return torch.stack([sth * torch.cos(phi), sth * torch.sin(phi), cth])


def _plummer(g, n, a=1.0, mass=1.0, rmax=20.0):
    """Positions and velocities [3, n] of a Plummer sphere (Aarseth, Henon & Wielen)."""
    # radii from the inverted mass profile, truncated at rmax scale radii
    umax = (rmax * rmax / (1.0 + rmax * rmax)) ** 1.5
    u = (1e-12 + (1.0 - 1e-12) * _rand(g, n)) * umax
    r = a / torch.sqrt(u ** (-2.0 / 3.0) - 1.0)
    # speed fraction q with density q^2 (1 - q^2)^{7/2}, by rejection (43 % pass)
    q = torch.empty(0, device="cuda", dtype=torch.float64)
    while q.numel() < n:
        k = 3 * (n - q.numel()) + 64
        t, y = _rand(g, k), 0.1 * _rand(g, k)
        q = torch.cat([q, t[y < t * t * (1.0 - t * t) ** 3.5]])
    vesc = math.sqrt(2.0 * mass) * (r * r + a * a) ** -0.25
    return _directions(g, n) * r, _directions(g, n) * (q[:n] * vesc)


def _sizes(case):
    """The systems' sizes: part of the configuration, the same for every seed."""
    rng = np.random.default_rng(case["n_sys"])
    lo, hi = math.log(case["nmin"]), math.log(case["nmax"])
    # an even spread over the logarithm, shuffled
    u = (np.arange(case["n_sys"]) + rng.random(case["n_sys"])) / case["n_sys"]
    return rng.permutation(np.rint(np.exp(lo + u * (hi - lo))).astype(np.int64))


def _particles(case, seed):
    """dict of float64 device arrays x .. vz, m, eps, and the system offsets (or None)."""
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 7919 + 13)
    off = None
    if case["dist"] == "ensemble":
        sizes = _sizes(case)
        off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
        n = int(off[-1])
        pos, vel = _plummer(g, n)
        ns = torch.repeat_interleave(torch.from_numpy(sizes), torch.from_numpy(sizes)).cuda().double()
        m, eps = 1.0 / ns, 4.0 / ns ** (1.0 / 3.0)
    elif case["dist"] == "cube":
        n = case["n"]
        pos = _rand(g, 3, n) - 0.5
        vel = torch.zeros_like(pos)
        m = (0.5 + _rand(g, n)) / n
        mesh = max(1, round(n ** (1.0 / 3.0)))
        eps = torch.full((n,), 0.025 / mesh if case["kind"] == "treepm" else 0.3 / mesh,
                         device="cuda", dtype=torch.float64)
    else:
        n = case["n"]
        if case["dist"] == "clustered":
            # half the particles in sub-clusters of scale 0.02 inside the unit sphere
            k = 64 if n >= 1 << 20 else 8
            per = n // (2 * k)
            pos, vel = _plummer(g, n - k * per, mass=0.5)
            pc, vc = _plummer(g, k * per, a=0.02, mass=0.5 / k)
            centre = _directions(g, k) * _rand(g, k) ** (1.0 / 3.0)
            pos = torch.cat([pos, pc + centre.repeat_interleave(per, dim=1)], dim=1)
            vel = torch.cat([vel, vc], dim=1)
            e = 1e-3
        else:
            pos, vel = _plummer(g, n)
            e = 0.3 * n ** (-1.0 / 3.0)
        m = torch.full((n,), 1.0 / n, device="cuda", dtype=torch.float64)
        eps = torch.full((n,), e, device="cuda", dtype=torch.float64)
    p = dict(zip(("x", "y", "z"), (t.contiguous() for t in pos)))
    p.update(zip(("vx", "vy", "vz"), (t.contiguous() for t in vel)))
    p["m"], p["eps"] = m.contiguous(), eps.contiguous()
    return p, off


def _domains(p, k):
    """The particles regrouped into k^3 domains of equal count: slabs along x, columns along y,
    blocks along z."""
    runs = [torch.arange(p["x"].numel(), device="cuda")]
    for axis in ("x", "y", "z"):
        nxt = []
        for r in runs:
            r = r[torch.argsort(p[axis][r], stable=True)]
            nxt += list(torch.tensor_split(r, k))
        runs = nxt
    order = torch.cat(runs)
    off = np.concatenate([[0], np.cumsum([r.numel() for r in runs])]).astype(np.int64)
    return {a: t[order].contiguous() for a, t in p.items()}, off


def _radii(case, n, seed):
    """Support radius of every particle: k mean spacings within +-10 %."""
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 7919 + 29)
    return case["k"] * n ** (-1.0 / 3.0) * (0.9 + 0.2 * _rand(g, n))


# -- a pass --------------------------------------------------------------------------------------

class _State:
    pass


def _outputs(n, fp32):
    out = [torch.empty(n, device="cuda", dtype=torch.float64) for _ in range(4)]
    low = [torch.empty(n, device="cuda", dtype=torch.float32) for _ in range(4)] if fp32 else None
    return out, low


def prepare(case, seed):
    s = _State()
    s.case = case
    kind = case["kind"]
    p, off = _particles(case, seed)
    if kind == "exchange":
        p, off = _domains(p, case["domains"])
    n = s.n = p["x"].numel()
    s.p = p
    fp32 = bool(case.get("fp32"))
    if kind in ("force", "step", "graph", "noalloc", "treepm"):
        s.out, s.low = _outputs(n, fp32)
    if kind in ("step", "graph") and fp32:
        s.vlow = [torch.empty(n, device="cuda", dtype=torch.float32) for _ in range(3)]
    torch.cuda.synchronize()
    if kind == "noalloc":
        s.flags = fdx.Context.flags(quad=case["quad"], fp32=fp32, persistent=case["persistent"])
        s.stream = torch.cuda.current_stream()
        return s
    s.ctx = fdx.Context(0)
    s.ctx.set_particles_device(p, off)
    if kind == "density":
        s.h = _radii(case, n, seed) if case["mode"] != fdx.CUT_FIXED else None
        s.r_cut = case["k"] * n ** (-1.0 / 3.0)
        s.rho = torch.empty(n, device="cuda", dtype=torch.float64)
        s.nngb = torch.empty(n, device="cuda", dtype=torch.int32)
        torch.cuda.synchronize()
    if kind == "exchange":
        # send buffers kept by the program: the lists fill them from the front
        cap = min(case["domains"] ** 3 - 1, 24) * n
        s.epj, s.spj = np.zeros(cap, np.uint32), np.zeros(cap, np.uint32)
    if kind == "treepm":
        s.r_cut = 3.0 / max(1, round(n ** (1.0 / 3.0)))
    if case.get("predictor"):
        s.ctx.predictor_load(WEIGHTS)
    if kind in ("step", "graph"):
        # the sample program evaluates the force once before its loop
        _calc(s)
    return s


def _calc(s):
    c = s.case
    s.ctx.calc_force(c["theta"], N_LEAF, c["n_group"], 0.0, quad=c["quad"], fp32=c["fp32"],
                     predictor=bool(c.get("predictor")),
                     persistent=bool(c.get("persistent", c["kind"] == "graph")),
                     fused=bool(c.get("fused")))


def _forces(s):
    s.ctx.forces_device(*s.out)
    return _lowered(s)


def _lowered(s):
    if s.low is None:
        return s.out
    for a, b in zip(s.low, s.out):
        a.copy_(b)
    return s.low


def run(s):
    c = s.case
    kind = c["kind"]
    if kind == "force":
        _calc(s)
        return {"force": _forces(s)}
    if kind in ("step", "graph"):
        if kind == "step":
            s.ctx.integrate(c["dt"], 1)
        else:
            s.ctx.integrate(c["dt"], c["steps"], graph=True)
        v = [s.p[a] for a in ("vx", "vy", "vz")]
        if s.low is not None:
            for a, b in zip(s.vlow, v):
                a.copy_(b)
            v = s.vlow
        return {"force": _forces(s), "pos": [s.p[a] for a in ("x", "y", "z")], "vel": v}
    if kind == "noalloc":
        p = s.p
        fdx.calc_force_noalloc(0, s.stream, p["x"], p["y"], p["z"], p["m"], p["eps"], 0.0,
                               c["theta"], N_LEAF, c["n_group"], s.flags, *s.out)
        return {"force": _lowered(s)}
    if kind == "treepm":
        s.ctx.calc_force_cutoff(c["theta"], N_LEAF, c["n_group"], 0.0, s.r_cut, fp32=c["fp32"],
                                persistent=c["persistent"])
        return {"force": _forces(s)[:3]}
    if kind == "density":
        s.ctx.calc_density(c["mode"], s.r_cut if s.h is None else 0.0, s.h, N_LEAF, c["n_group"])
        # the C entry itself: the binding's density() brings the result to the host
        s.ctx._check(s.ctx.lib.fdx_get_density(s.ctx.h, s.rho.data_ptr(), s.nngb.data_ptr(),
                                               fdx.MEM_DEVICE), "get_density")
        return {"rho": s.rho, "nngb": s.nngb}
    s.ctx.build_exchange_lists(c["theta"], N_LEAF)
    ne, ns = s.ctx.exchange_counts()
    if max(int(ne.sum()), int(ns.sum())) > s.epj.size:
        raise RuntimeError("the send buffers are too small")
    s.ctx._check(s.ctx.lib.fdx_get_exchange_lists(s.ctx.h, s.epj.ctypes.data,
                                                  s.spj.ctypes.data), "get_exchange_lists")
    return {"n_epj": ne, "n_spj": ns, "epj": s.epj, "spj": s.spj}


# -- what a pass cannot do without ---------------------------------------------------------------

def _list_model(n, theta, n_group):
    """Particle and superparticle interactions per particle: the lists of the 2^24 clustered set
    at theta 0.5 and n_group 256 (940 and 3100), scaled with the group's size and log n."""
    lg = max(1.0, math.log2(max(2.0, n / 64.0))) / 18.0
    pp = min(float(n), 940.0 * (n_group / 256.0) ** 0.5 * min(1.0, 0.5 / theta))
    pc = min(float(n), 3100.0 * (0.5 / theta) ** 2.5 * lg * (n_group / 256.0) ** 0.3)
    return pp, pc


def work(case):
    kind = case["kind"]
    n = float(_sizes(case).sum()) if case["dist"] == "ensemble" else float(case["n"])
    if kind == "density":
        ngb = 4.0 / 3.0 * math.pi * case["k"] ** 3
        h = 8.0 if case["mode"] else 0.0
        return {"bytes": n * (32.0 + h + 12.0), "flops": n * ngb * 30.0}
    if kind == "treepm":
        ngb = 4.0 / 3.0 * math.pi * 27.0
        return {"bytes": n * (40.0 + 32.0), "flops": n * 3.0 * ngb * 35.0}
    if kind == "exchange":
        d = float(case["domains"]) ** 3
        per = 14.0 * (n / d) ** (2.0 / 3.0) / case["theta"]
        return {"bytes": n * 32.0 + d * per * 4.0, "flops": 0.0}
    pp, pc = _list_model(n / case.get("n_sys", 1), case["theta"], case["n_group"])
    flops = n * (20.0 * pp + (54.0 if case["quad"] else 20.0) * pc)
    move = 120.0 + 72.0 if kind in ("step", "graph") else 0.0
    k = case.get("steps", 1)
    return {"bytes": k * n * (40.0 + 32.0 + move), "flops": k * flops}


# -- the same quantities in 64 bits, summed over all pairs ------------------------------------------

def _direct(p, off, pair, width):
    """Sum over every particle's system of pair(dx, dy, dz, r2, j slice, i slice) -> width sums."""
    n = p["x"].numel()
    off = [0, n] if off is None else off
    out = torch.zeros(width, n, device="cuda", dtype=torch.float64)
    for a, b in zip(off[:-1], off[1:]):
        a, b = int(a), int(b)
        rows = max(1, int(3e7) // max(1, b - a))
        for i0 in range(a, b, rows):
            i, j = slice(i0, min(b, i0 + rows)), slice(a, b)
            d = [p[q][j][None, :] - p[q][i][:, None] for q in ("x", "y", "z")]
            r2 = (d[0] * d[0] + d[1] * d[1]) + d[2] * d[2]
            for k, v in enumerate(pair(d, r2, i, j)):
                out[k, i] = v
    return out


def _gravity(p, off):
    def pair(d, r2, i, j):
        rinv = torch.rsqrt(r2 + p["eps"][i][:, None] ** 2)
        mr = p["m"][j][None, :] * rinv
        own = torch.arange(j.start, j.stop, device="cuda")[None, :] == \
            torch.arange(i.start, i.stop, device="cuda")[:, None]
        mr = torch.where(own, torch.zeros_like(mr), mr)
        f = mr * rinv * rinv
        return [(f * d[0]).sum(1), (f * d[1]).sum(1), (f * d[2]).sum(1), -mr.sum(1)]
    return list(_direct(p, off, pair, 4))


def _s2(xi):
    """1 - xi^3 (...) of the S2 pair force (Hockney & Eastwood), 0 beyond xi = 2."""
    a = 1 - xi ** 3 * (224 - 224 * xi ** 2 + 70 * xi ** 3 + 48 * xi ** 4 - 21 * xi ** 5) / 140
    b = 1 - (12 - 224 * xi ** 2 + 896 * xi ** 3 - 840 * xi ** 4 + 224 * xi ** 5 + 70 * xi ** 6
             - 48 * xi ** 7 + 7 * xi ** 8) / 140
    return torch.where(xi <= 1, a, torch.where(xi < 2, b, torch.zeros_like(xi)))


def _wendland(r2, h):
    q = (torch.sqrt(r2) / h).clamp(max=1.0)
    return 1365.0 / (64.0 * math.pi) / h ** 3 * (1 - q) ** 8 * (1 + 8 * q + 25 * q * q + 32 * q ** 3)


def exact(case, seed):
    kind = case["kind"]
    if kind == "exchange":
        return None
    sizes = _sizes(case).astype(float) if case["dist"] == "ensemble" else \
        np.array([float(case["n"])])
    if (sizes ** 2).sum() * (case.get("steps", 1) + 1 if kind in ("step", "graph") else 1) \
            > EXACT_PAIRS:
        return None
    p, off = _particles(case, seed)
    n = p["x"].numel()
    if kind in ("force", "noalloc"):
        return {"force": _gravity(p, off)}
    if kind in ("step", "graph"):
        a, dt = _gravity(p, off), case["dt"]
        for _ in range(case.get("steps", 1)):
            for q, ak in zip("xyz", a):
                p["v" + q] += 0.5 * dt * ak
                p[q] += dt * p["v" + q]
            a = _gravity(p, off)
            for q, ak in zip("xyz", a):
                p["v" + q] += 0.5 * dt * ak
        return {"force": a, "pos": [p[q] for q in "xyz"], "vel": [p["v" + q] for q in "xyz"]}
    if kind == "treepm":
        r_cut = 3.0 / max(1, round(n ** (1.0 / 3.0)))

        def pair(d, r2, i, j):
            rinv = torch.rsqrt(r2 + p["eps"][i][:, None] ** 2)
            f = p["m"][j][None, :] * rinv ** 3 * _s2(2.0 / r_cut * torch.sqrt(r2))
            return [(f * d[0]).sum(1), (f * d[1]).sum(1), (f * d[2]).sum(1)]
        return {"force": list(_direct(p, off, pair, 3))}
    mode = case["mode"]
    h = _radii(case, n, seed) if mode else torch.full(
        (n,), case["k"] * n ** (-1.0 / 3.0), device="cuda", dtype=torch.float64)

    def pair(d, r2, i, j):
        hi, hj, m = h[i][:, None], h[j][None, :], p["m"][j][None, :]
        gather = torch.where(r2 < hi * hi, _wendland(r2, hi), torch.zeros_like(r2)) \
            if mode != 1 else None
        scatter = torch.where(r2 < hj * hj, _wendland(r2, hj), torch.zeros_like(r2)) \
            if mode in (1, 3) else None
        w = scatter if mode == 1 else gather if mode != 3 else 0.5 * (gather + scatter)
        return [(m * w).sum(1)]
    return {"rho": _direct(p, off, pair, 1)[0], "nngb": None}
