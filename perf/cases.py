"""The work a user of this library has it do, as cases that can be timed and
compared: one domain on the device, many uneven domains in one launch, the
repeated timestep as a graph, and a domain that lives in host memory.

A case is a dict of plain values:
  kind     "single" (pw_advect), "batch" (pw_advect_batched), "noalloc"
           (pw_advect_batched_noalloc), "step" (a replayed graph of perturb +
           halo fill + advect) or "host" (pw_advect_host, overlapped slabs)
  storage  "f64", "f32", "bf16", "f16", "i16" or "i32"
  nx ny nz, pad    one domain and the elements between its columns
  domains, heights, shapes   a batch: how many, its column heights, and the
           seed of its x-y extents (16..96 each)
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2107_13500_amd import binding as B
from paper_2107_13500_amd import inputs

DEV = "cuda:0"
STORAGE = {"f64": B.F64, "f32": B.F32, "bf16": B.BF16, "f16": B.F16, "i16": B.I16, "i32": B.I32}
ELEM = {"f64": 8, "f32": 4, "bf16": 2, "f16": 2, "i16": 2, "i32": 4}
TARGET = {"f16": 2.0 ** 14, "i16": 2.0 ** 14, "i32": 2.0 ** 30}   # largest scaled magnitude
AMPLITUDE = 1e-3
KEY = 20210713   # the perturbation's own seed (a program keeps one; the fields' seed differs from it)


def listed():
    return [
        # one small domain, as a test run or a subdomain of a decomposed model calls it: latency
        dict(name="pw64-f64", kind="single", storage="f64", nx=64, ny=64, nz=64, pad=0),
        # the paper's Table I grid, 16.8 M points
        dict(name="pw512-f64", kind="single", storage="f64", nx=512, ny=512, nz=64, pad=0),
        # the benchmark's headline grid, 268 M points
        dict(name="pw2048-f64", kind="single", storage="f64", nx=2048, ny=2048, nz=64, pad=0),
        # the headline grid in the narrowest floating storage
        dict(name="pw2048-bf16", kind="single", storage="bf16", nx=2048, ny=2048, nz=64, pad=0),
        # fixed point with per-field scales on a taller column
        dict(name="fixed1024-i16", kind="single", storage="i16", nx=1024, ny=1000, nz=96, pad=0),
        # a column height with no kernel of its own, even
        dict(name="levels80-f64", kind="single", storage="f64", nx=300, ny=420, nz=80, pad=0),
        # an odd column height, odd extents
        dict(name="levels63-f32", kind="single", storage="f32", nx=257, ny=391, nz=63, pad=0),
        # columns padded to a round pitch, as a model with aligned columns stores them
        dict(name="padded60-f64", kind="single", storage="f64", nx=250, ny=310, nz=60, pad=4),
        # the 384 uneven subdomains of a decomposed model in one launch
        dict(name="batch384-f64", kind="batch", storage="f64", domains=384, heights="64,96,128", shapes=4),
        # their repeated timestep (perturb, halos, advect), one graph replay per step
        dict(name="step384-f32", kind="step", storage="f32", domains=384, heights="64,96,128", shapes=4),
        # a smaller batch without a plan, for callers that may not allocate
        dict(name="noalloc96-f16", kind="noalloc", storage="f16", domains=96, heights="64,96,128", shapes=9),
        # the Table I grid resident in host memory, transfers overlapped with the kernel
        dict(name="host512-f64", kind="host", storage="f64", nx=512, ny=512, nz=64, pad=0),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _height(rng):
    """Half the common heights (which have kernels of their own), most of the
    rest between 20 and 200 levels, odd or even, and some tall columns."""
    r = rng.random()
    if r < 0.5:
        return rng.choice((64, 64, 96, 128))
    return rng.randint(20, 200) if r < 0.9 else rng.randint(201, 400)


def draw(rng):
    r = rng.random()
    storage = rng.choice(("f64", "f64", "f64", "f32", "f32", "bf16", "f16", "i16", "i32"))
    if r < 0.62:
        nz = _height(rng)
        while True:
            nx, ny = _log_int(rng, 16, 2048), _log_int(rng, 16, 2048)
            if nx * ny * nz * ELEM[storage] <= 2048 * 2048 * 64 * 8:
                break
        return dict(kind="single", storage=storage, nx=nx, ny=ny, nz=nz,
                    pad=rng.choice((1, 2, 4, 8)) if r < 0.08 else 0)
    if r < 0.92:
        heights = rng.choice(("64,96,128", "64,96,128", "64", "40,80", "48,63,100"))
        return dict(kind=rng.choice(("batch", "batch", "step", "noalloc")), storage=storage,
                    domains=_log_int(rng, 4, 384), heights=heights, shapes=rng.randint(100, 10 ** 6))
    return dict(kind="host", storage=rng.choice(("f64", "f32")), nx=_log_int(rng, 64, 512),
                ny=_log_int(rng, 64, 512), nz=rng.choice((64, 96, rng.randint(20, 100))), pad=0)


# ----------------------------------------------------------------------------
# inputs
# ----------------------------------------------------------------------------
def _shapes(case):
    if case["kind"] in ("single", "host"):
        return [(case["nx"], case["ny"], case["nz"])]
    rng = np.random.Generator(np.random.PCG64(case["shapes"]))
    heights = [int(h) for h in case["heights"].split(",")]
    return [(int(rng.integers(16, 97)), int(rng.integers(16, 97)), heights[int(rng.integers(0, len(heights)))])
            for _ in range(case["domains"])]


def _coefficients(nz, d):
    """Domain d's coefficients (its own grid spacing and density profile)."""
    g = inputs.vertical_grid(nz, rho0=1.1 + 0.02 * (d % 11), scale_height=6000.0 + 400.0 * (d % 11))
    return inputs.coefficients(g, dx=25.0 + 5.0 * (d % 16))


def _halo(a):
    """Periodic one-point x-y halo of a (nx + 2, ny + 2, nz) tensor, in place."""
    a[0, 1:-1] = a[-2, 1:-1]
    a[-1, 1:-1] = a[1, 1:-1]
    a[:, 0] = a[:, -2]
    a[:, -1] = a[:, 1]


def _scales(storage, fields, c):
    """Power-of-two input and output scales (1 where the type needs none)."""
    if storage not in TARGET:
        return (1.0, 1.0, 1.0), (1.0, 1.0, 1.0)
    mu, mv, mw = (float(t) for t in torch.stack([f.abs().max() for f in fields]).cpu())
    zc, zd = float(np.max(c.tzc1 + c.tzc2)), float(np.max(c.tzd1 + c.tzd2))
    bounds = (4 * c.tcx * mu * mu + 4 * c.tcy * mu * mv + 2 * zc * mu * mw,
              4 * c.tcy * mv * mv + 4 * c.tcx * mv * mu + 2 * zc * mv * mw,
              4 * c.tcx * mw * mu + 4 * c.tcy * mw * mv + 2 * zd * mw * mw)
    t = TARGET[storage]
    return tuple(inputs.pow2_scale(m, t) for m in (mu, mv, mw)), tuple(inputs.pow2_scale(b, t) for b in bounds)


def _fill(views, storage, c, gen):
    """Seeded winds u = 5 + N(0, 1), v = 2 + N(0, 1), w = 0.3 N(0, 1) (w = 0 at
    the lid and the ground) with periodic halos into the three views, in the
    storage type; returns the scales."""
    work = views if storage in ("f64", "f32") else [
        torch.empty(v.shape, dtype=torch.float64 if storage == "i32" else torch.float32, device=v.device) for v in views]
    for a, (mean, std) in zip(work, ((5.0, 1.0), (2.0, 1.0), (0.0, 0.3))):
        a.normal_(mean, std, generator=gen)
    work[2][:, :, 0] = 0
    work[2][:, :, -1] = 0
    for a in work:
        _halo(a)
    ins, outs = _scales(storage, work, c)
    if work is not views:
        for v, a, s in zip(views, work, ins):
            a *= s
            if storage in ("i16", "i32"):
                a.round_()
            v.copy_(a)
    return ins, outs


def _inputs(case, seed):
    """Device memory of every domain: dict with per-domain records of views,
    coefficients and scales, and the whole output arrays."""
    storage, shapes = case["storage"], _shapes(case)
    dt = B.torch_dtype(STORAGE[storage])
    gen = torch.Generator(device=DEV).manual_seed(seed)
    doms = []
    if case["kind"] in ("single", "host"):
        nx, ny, nz = shapes[0]
        pool = B.pooled_fields((nx + 2, ny + 2, nz + case["pad"]), dt, DEV)
        for o in pool:
            o.zero_()
        f = [o[:, :, :nz] for o in pool]
        c = _coefficients(nz, 0)
        doms.append((f, c, _fill(f[:3], storage, c, gen)))
        return {"doms": doms, "out": f[3:]}
    # a batch in one allocation: every domain's u, v, w, then all su, all sv,
    # all sw, each array 256-byte aligned
    unit = 256 // ELEM[storage]
    size = [-(-(nx + 2) * (ny + 2) * nz // unit) * unit for nx, ny, nz in shapes]
    total = sum(size)
    pool = torch.zeros(6 * total, dtype=dt, device=DEV)
    at = 0
    for d, (nx, ny, nz) in enumerate(shapes):
        n = (nx + 2) * (ny + 2) * nz
        starts = [3 * at, 3 * at + size[d], 3 * at + 2 * size[d], 3 * total + at, 4 * total + at, 5 * total + at]
        f = [pool[s:s + n].view(nx + 2, ny + 2, nz) for s in starts]
        at += size[d]
        c = _coefficients(nz, d)
        doms.append((f, c, _fill(f[:3], storage, c, gen)))
    return {"doms": doms, "in": pool[:3 * total], "out": [pool[(3 + q) * total:(4 + q) * total] for q in range(3)],
            "pool": pool}


def prepare(case, seed):
    s = _inputs(case, seed)
    s["kind"], s["storage"] = case["kind"], STORAGE[case["storage"]]
    if case["kind"] == "single":
        f, c, (ins, outs) = s["doms"][0]
        tz = [torch.from_numpy(a).to(DEV) for a in c.arrays()]
        sc = B.make_scales(ins, outs) if s["storage"] in B.SCALED else None
        s["domain"] = B.DeviceDomain(*f[:3], c.tcx, c.tcy, *tz, scales=sc, outputs=f[3:])
        s["plan"] = B.Plan(s["storage"], [B.shape_of(f[0])])
        return s
    if case["kind"] == "host":
        f, c, _ = s["doms"][0]
        s["h_in"] = [torch.empty(a.shape, dtype=a.dtype, pin_memory=True).copy_(a) for a in f[:3]]
        s["out"] = [torch.zeros(a.shape, dtype=a.dtype, pin_memory=True) for a in f[3:]]
        s["coef"] = (c.tcx, c.tcy) + tuple(torch.from_numpy(a.copy()) for a in c.arrays())
        s["plan"] = B.StreamPlan(s["storage"], B.shape_of(s["h_in"][0]))
        del s["doms"], f
        return s
    coef = torch.from_numpy(np.concatenate([np.concatenate(c.arrays()) for _, c, _ in s["doms"]])).to(DEV)
    recs, at = [], 0
    for f, c, (ins, outs) in s["doms"]:
        nz = f[0].shape[2]
        tz = [coef[at + q * nz:at + (q + 1) * nz] for q in range(4)]
        at += 4 * nz
        recs.append(B.domain_record(*f, c.tcx, c.tcy, *tz, scales=B.make_scales(ins, outs)))
    s["coef"], s["shapes"] = coef, [r.shape for r in recs]
    s["d_args"] = B.domain_args_tensor(recs, DEV)
    if case["kind"] != "noalloc":
        s["plan"] = B.Plan(s["storage"], s["shapes"])
    if case["kind"] == "step":
        s["call"] = torch.zeros(1, dtype=torch.int64, device=DEV)
        s["graph"] = B.Graph.timestep(s["plan"], s["d_args"], KEY, s["call"], AMPLITUDE)
    return s


def run(s):
    if s["kind"] == "single":
        s["domain"].run(s["plan"])
    elif s["kind"] == "batch":
        B.advect_batched(s["plan"], s["d_args"])
    elif s["kind"] == "noalloc":
        B.advect_batched_noalloc(s["storage"], s["shapes"], s["d_args"])
    elif s["kind"] == "step":
        s["graph"].launch()
        return [*s["out"], s["in"], s["call"]]   # the step also moves u and v and their halos
    else:
        s["plan"].run(*s["h_in"], *s["out"], *s["coef"])
    return list(s["out"])


def work(case):
    e, nbytes, points = ELEM[case["storage"]], 0, 0
    for nx, ny, nz in _shapes(case):
        inner, halo = nx * ny * nz, (nx + 2) * (ny + 2) * nz
        points += inner
        if case["kind"] == "step":   # interiors of u, v, w in; u, v, the halos of all three and the outputs out
            nbytes += e * (3 * inner + 2 * inner + 3 * (halo - inner) + 3 * inner) + 32 * nz
        else:
            nbytes += e * (3 * halo + 3 * inner) + 32 * nz
    return {"bytes": nbytes, "flops": 63 * points}


# ----------------------------------------------------------------------------
# the same in 64 bits, plain torch
# ----------------------------------------------------------------------------
def _reference(u, v, w, c, out):
    """su, sv, sw of the interior of float64 u, v, w into the interiors of the
    three float64 tensors `out`, a few x planes at a time."""
    t1, t2, e1, e2 = (torch.from_numpy(a).to(u.device) for a in c.arrays())
    nx, nz = u.shape[0] - 2, u.shape[2]
    step = max(1, int(2 ** 25 // (u.shape[1] * nz)))
    for i in range(0, nx, step):
        U, V, W = (a[i:min(i + step, nx) + 2] for a in (u, v, w))

        def at(a, di, dj, lo, hi):   # levels lo .. hi - 1 at x offset di, y offset dj
            return a[1 + di:a.shape[0] - 1 + di, 1 + dj:a.shape[1] - 1 + dj, lo:hi]

        # k = 2 .. nz (index 1 .. nz - 1) for the parts that exist at every level
        r = (1, nz)
        lo = (0, nz - 1)
        su = c.tcx * (at(U, -1, 0, *r) * (at(U, 0, 0, *r) + at(U, -1, 0, *r))
                      - at(U, 1, 0, *r) * (at(U, 0, 0, *r) + at(U, 1, 0, *r)))
        su += c.tcy * (at(U, 0, -1, *r) * (at(V, 0, -1, *r) + at(V, 1, -1, *r))
                       - at(U, 0, 1, *r) * (at(V, 0, 0, *r) + at(V, 1, 0, *r)))
        su += t1[1:] * at(U, 0, 0, *lo) * (at(W, 0, 0, *lo) + at(W, 1, 0, *lo))
        sv = c.tcy * (at(V, 0, -1, *r) * (at(V, 0, 0, *r) + at(V, 0, -1, *r))
                      - at(V, 0, 1, *r) * (at(V, 0, 0, *r) + at(V, 0, 1, *r)))
        sv += c.tcx * (at(V, -1, 0, *r) * (at(U, -1, 0, *r) + at(U, -1, 1, *r))
                       - at(V, 1, 0, *r) * (at(U, 0, 0, *r) + at(U, 0, 1, *r)))
        sv += t1[1:] * at(V, 0, 0, *lo) * (at(W, 0, 0, *lo) + at(W, 0, 1, *lo))
        o = [a[1 + i:1 + min(i + step, nx), 1:-1] for a in out]
        if nz > 2:   # k = 2 .. nz - 1: the upper vertical flux, and sw
            m, up, dn = (1, nz - 1), (2, nz), (0, nz - 2)
            su[:, :, :-1] -= t2[1:-1] * at(U, 0, 0, *up) * (at(W, 0, 0, *m) + at(W, 1, 0, *m))
            sv[:, :, :-1] -= t2[1:-1] * at(V, 0, 0, *up) * (at(W, 0, 0, *m) + at(W, 0, 1, *m))
            sw = c.tcx * (at(W, -1, 0, *m) * (at(U, -1, 0, *m) + at(U, -1, 0, *up))
                          - at(W, 1, 0, *m) * (at(U, 0, 0, *m) + at(U, 0, 0, *up)))
            sw += c.tcy * (at(W, 0, -1, *m) * (at(V, 0, -1, *m) + at(V, 0, -1, *up))
                           - at(W, 0, 1, *m) * (at(V, 0, 0, *m) + at(V, 0, 0, *up)))
            sw += e1[1:-1] * at(W, 0, 0, *dn) * (at(W, 0, 0, *m) + at(W, 0, 0, *dn))
            sw -= e2[1:-1] * at(W, 0, 0, *up) * (at(W, 0, 0, *m) + at(W, 0, 0, *up))
            o[2][:, :, 1:-1] = sw
        o[0][:, :, 1:] = su
        o[1][:, :, 1:] = sv


def _mix64(x):
    """SplitMix64's finaliser (Steele, Lea and Flood, OOPSLA 2014)."""
    m = (1 << 64) - 1
    x = (x + 0x9E3779B97F4A7C15) & m
    x = ((x ^ (x >> 30)) * 0xBF58476D1CE4E5B9) & m
    x = ((x ^ (x >> 27)) * 0x94D049BB133111EB) & m
    return x ^ (x >> 31)


def _mix32(x):
    """lowbias32 (C. Wellons, 2018) on 32-bit values in an int64 tensor."""
    def times(a, k):   # the low 32 bits of a k, without overflow of 63 bits
        return ((a & 0xFFFF) * k + (((a >> 16) * k & 0xFFFF) << 16)) & 0xFFFFFFFF
    x = times(x ^ (x >> 16), 0x7FEB352D)
    x = times(x ^ (x >> 15), 0x846CA68B)
    return x ^ (x >> 16)


def _noise(d, nx, ny, nz, q):
    """The documented perturbation of the first call, r in [-1, 1)."""
    k = _mix64(KEY ^ _mix64(d))
    key = (k ^ (k >> 32)) & 0xFFFFFFFF
    g = torch.arange(nx * ny * nz, dtype=torch.int64, device=DEV).view(nx, ny, nz)
    h = _mix32(_mix32((2 * g + q) & 0xFFFFFFFF) ^ key)
    return (h >> 8).to(torch.float64) * 2.0 ** -23 - 1.0


def exact(case, seed):
    s = _inputs(case, seed)
    whole = case["storage"] in ("i16", "i32")
    if whole:
        return None   # whole numbers: they stay equal
    outs = [torch.zeros(o.shape, dtype=torch.float64, device=DEV) for o in s["out"]]
    moved = torch.zeros(s["in"].shape, dtype=torch.float64, device=DEV) if case["kind"] == "step" else None
    for d, (f, c, (in_s, out_s)) in enumerate(s["doms"]):
        nx, ny, nz = (f[0].shape[0] - 2, f[0].shape[1] - 2, f[0].shape[2])
        fields = [a.to(torch.float64) / k for a, k in zip(f[:3], in_s)]
        if moved is not None:
            for q in range(2):
                fields[q][1:-1, 1:-1] += AMPLITUDE * _noise(d, nx, ny, nz, q)
            for a, g, k in zip(fields, f, in_s):
                _halo(a)
                moved[g.storage_offset():g.storage_offset() + g.numel()] = (a * k).view(-1)
        if case["kind"] in ("single", "host"):
            o = outs
        else:
            n, total = f[3].numel(), s["in"].numel() // 3
            o = [outs[q][a.storage_offset() - (3 + q) * total:][:n].view(f[3].shape) for q, a in enumerate(f[3:])]
        _reference(*fields, c, o)
        for a, k in zip(o, out_s):
            if k != 1.0:
                a *= k
    return outs if moved is None else [*outs, moved, None]
