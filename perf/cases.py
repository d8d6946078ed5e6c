"""The calls a user of this package makes, as cases that can be timed.

A case is a dict of plain values; `prepare` makes its volumes on the GPU (and
the workspace, plan or server a program keeps between calls), `run` is one
pass through the package's public entry points, `work` the bytes and
operations the pass cannot do without, and `exact` the same outputs in 64
bits from plain torch.  Sizes are those of the package's own workloads and
tests, and generic ones of the same range.

Kinds of case:

  step      select_and_window_stats + the prepared search, with workspaces
            that the program keeps: the time-critical registration of 12-bit
            volumes, and what the benchmark times
  register  select_blocks + block_match, nothing kept: the one-off call
  aniso     the same with block edges, strides and half windows per axis
            (slices thicker than the pixels are wide)
  batch     a BatchPlan run: the parametric search of one volume pair
  mask      select_blocks_ex: selection inside a mask, with a pattern that
            keeps the blocks apart
  conf      structure_confidence: the directional weights of matched blocks
  serve     a Server's queue: several requests naming resident volumes
"""

from __future__ import annotations

import math

import torch

import paper_2308_10868_amd as nrr

DEV = "cuda"


# ----------------------------------------------------------------- the cases

def listed():
    return [
        # the smallest call: a sub-volume around a lesion, a few dozen blocks,
        # where launches and their latency are all there is
        {"name": "register_u16_48", "kind": "register", "dtype": "u16", "nx": 48, "ny": 40,
         "nz": 36, "block": 5, "stride": 5, "fraction": 0.3, "window": 4},
        # the small float workload (64^3, translated): one plain registration
        {"name": "register_f32_64", "kind": "register", "dtype": "f32", "nx": 64, "ny": 64,
         "nz": 64, "block": 7, "stride": 7, "fraction": 0.2, "window": 5},
        # the headline workload: a clinical MRI pair, selection, statistics, search
        {"name": "step_u16_mri", "kind": "step", "dtype": "u16", "nx": 256, "ny": 256, "nz": 124,
         "block": 7, "stride": 7, "fraction": 0.25, "window": 10},
        # a resampled atlas-sized pair: every axis odd, larger blocks, a part of them
        {"name": "step_u16_odd", "kind": "step", "dtype": "u16", "nx": 181, "ny": 217, "nz": 181,
         "block": 9, "stride": 8, "fraction": 0.2, "window": 8},
        # the largest: dense overlapping blocks of a 512 x 512 x 256 pair
        {"name": "step_u16_dense", "kind": "step", "dtype": "u16", "nx": 512, "ny": 512,
         "nz": 256, "block": 9, "stride": 5, "fraction": 0.7, "window": 12},
        # large blocks (edges above 9): few, for low-contrast regions
        {"name": "register_u16_b13", "kind": "register", "dtype": "u16", "nx": 192, "ny": 192,
         "nz": 96, "block": 13, "stride": 13, "fraction": 0.3, "window": 6},
        # the headline sizes on float volumes (intensities after bias correction)
        {"name": "register_f32_mri", "kind": "register", "dtype": "f32", "nx": 256, "ny": 256,
         "nz": 124, "block": 7, "stride": 7, "fraction": 0.25, "window": 10},
        # the parametric search: 32 sets over block, window and fraction
        {"name": "batch_f32_64_32sets", "kind": "batch", "dtype": "f32", "nx": 64, "ny": 64,
         "nz": 64, "sets": 32, "draw": 1},
        # thick slices: blocks and windows thinner along z
        {"name": "aniso_u16_mri", "kind": "aniso", "dtype": "u16", "nx": 256, "ny": 256,
         "nz": 124, "bx": 7, "by": 7, "bz": 3, "sx": 7, "sy": 7, "sz": 3, "fraction": 0.25,
         "wx": 10, "wy": 10, "wz": 4},
        # selection inside the brain's mask, blocks sharing no face
        {"name": "mask_u16_mri", "kind": "mask", "dtype": "u16", "nx": 256, "ny": 256, "nz": 124,
         "block": 7, "stride": 7, "fraction": 0.25, "connectivity": 6},
        # the directional confidence of the headline workload's blocks
        {"name": "conf_u16_mri", "kind": "conf", "dtype": "u16", "nx": 256, "ny": 256, "nz": 124,
         "block": 7, "stride": 7, "fraction": 0.25},
        # a queue of eight requests of mixed parameters on resident volumes
        {"name": "serve_u16_192", "kind": "serve", "dtype": "u16", "nx": 192, "ny": 192,
         "nz": 96, "requests": 8, "draw": 4, "slots": 4},
    ]


# nominal voxel pairs (block voxels x displacements, summed over the blocks)
# a drawn case may cost, by the path that serves it
MOST_PAIRS = {"u16": 4.0e11, "f32": 6.0e10, "big": 4.0e10, "aniso": 6.0e10}


def draw(rng):
    kind = rng.choice(["step", "step", "step", "register", "register", "register", "aniso",
                       "aniso", "batch", "mask", "conf", "serve"])

    def size(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    dtype = "u16" if kind in ("step", "serve") else rng.choice(["u16", "f32"])
    c = {"kind": kind, "dtype": dtype, "nx": size(40, 360), "ny": size(40, 360),
         "nz": size(32, 200)}
    if kind == "batch":
        c.update(nx=size(40, 72), ny=size(40, 72), nz=size(40, 72), sets=rng.randint(8, 32),
                 draw=rng.randint(0, 1 << 20))
        return c
    if kind == "serve":
        c.update(nx=size(96, 256), ny=size(96, 256), nz=size(64, 128),
                 requests=rng.randint(4, 10), draw=rng.randint(0, 1 << 20),
                 slots=rng.randint(1, 4))
        return c
    if kind == "aniso":
        c.update(bx=rng.choice([5, 7, 9]), by=rng.choice([5, 7, 9]), bz=rng.choice([3, 5]))
        c.update(sx=c["bx"] + rng.randint(-1, 2), sy=c["by"] + rng.randint(-1, 2),
                 sz=c["bz"] + rng.randint(0, 2), wx=rng.randint(4, 12), wy=rng.randint(4, 12),
                 wz=rng.randint(1, 5), fraction=rng.uniform(0.05, 0.5))
    else:
        c["block"] = rng.choice([5, 7, 9] if kind == "step" else [3, 5, 7, 7, 9, 9, 11, 13, 15])
        c["stride"] = max(3, c["block"] + rng.randint(-3, 2))
        c["fraction"] = rng.uniform(0.05, 0.5)
        if kind in ("step", "register"):
            c["window"] = rng.randint(3, 12)
        if kind == "mask":
            c["connectivity"] = rng.choice([0, 6, 18, 26])
    if kind in ("step", "register", "aniso"):
        path = "aniso" if kind == "aniso" else "f32" if dtype == "f32" else \
            "big" if c["block"] > 9 else "u16"
        while _pairs(c) > MOST_PAIRS[path]:
            c["fraction"] /= 2
    return c


def _sets(c):
    """(block, window, stride, fraction) of a batch or the requests of a queue."""
    import random

    r = random.Random(c["draw"])
    if c["kind"] == "batch":
        out = []
        for _ in range(c["sets"]):
            b = r.choice([5, 7, 9])
            out.append((b, r.choice([5, 8, 12]), b, r.choice([0.05, 0.1, 0.25, 0.5])))
        return out
    out = []
    for _ in range(c["requests"]):
        b = r.choice([5, 7, 9])
        out.append((b, r.randint(5, 12), b, round(r.uniform(0.1, 0.3), 3)))
    return out


def _axes(c):
    """Per-axis (x, y, z) block edges, strides and half windows of a case."""
    if c["kind"] == "aniso":
        return ((c["bx"], c["by"], c["bz"]), (c["sx"], c["sy"], c["sz"]),
                (c["wx"], c["wy"], c["wz"]))
    return (c["block"],) * 3, (c["stride"],) * 3, (c.get("window", 0),) * 3


def _count(dims, b, s, fraction):
    n = 1
    for d, e, t in zip(dims, b, s):
        n *= (d - e) // t + 1
    return n, min(n, int(math.floor(0.5 + n * fraction)))


def _pairs(c):
    b, s, w = _axes(c)
    _, k = _count((c["nx"], c["ny"], c["nz"]), b, s, c["fraction"])
    return float(k) * math.prod(b) * math.prod(2 * a + 1 for a in w)


def work(case):
    c = case
    vox = c["nx"] * c["ny"] * c["nz"]
    size = 2 if c["dtype"] == "u16" else 4
    dims = (c["nx"], c["ny"], c["nz"])
    if c["kind"] in ("batch", "serve"):
        pairs, rows = 0.0, 0
        for b, w, s, f in _sets(c):
            _, k = _count(dims, (b,) * 3, (s,) * 3, f)
            pairs += float(k) * b ** 3 * (2 * w + 1) ** 3
            rows += k
        return {"bytes": 2.0 * vox * size + 32.0 * rows, "flops": 2.0 * pairs}
    b, s, _ = _axes(c)
    n, k = _count(dims, b, s, c["fraction"])
    if c["kind"] == "mask":  # a variance per candidate: an add and a multiply-add per voxel
        return {"bytes": float(vox) * (size + 1) + 12.0 * k, "flops": 3.0 * n * math.prod(b)}
    if c["kind"] == "conf":  # gradients (6) and six products per voxel of a block
        return {"bytes": float(min(vox, k * (b[0] + 2) ** 3)) * size + 40.0 * k,
                "flops": 18.0 * k * math.prod(b)}
    return {"bytes": 2.0 * vox * size + 32.0 * k, "flops": 2.0 * _pairs(c)}


# -------------------------------------------------------------------- inputs

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _field(g, dims, spacing):
    """A smooth random field of about unit variance: white noise on a coarse
    grid of `spacing` voxels, interpolated."""
    nx, ny, nz = dims
    shape = [1, 1] + [max(2, -(-n // spacing) + 1) for n in (nz, ny, nx)]
    coarse = torch.randn(shape, generator=g, device=DEV)
    f = torch.nn.functional.interpolate(coarse, size=(nz, ny, nx), mode="trilinear",
                                        align_corners=True)[0, 0]
    return f * 1.8


def _smooth3(v):
    """Partial volume: a 1-2-1 filter per axis, edges repeated."""
    for d in range(3):
        n = v.shape[d]
        lo = torch.cat([v.narrow(d, 0, 1), v.narrow(d, 0, n - 1)], d)
        hi = torch.cat([v.narrow(d, 1, n - 1), v.narrow(d, n - 1, 1)], d)
        v = 0.25 * lo + 0.5 * v + 0.25 * hi
    return v


def _sag(v, g, peak):
    """v warped by a smooth brain shift of up to `peak` voxels (trilinear)."""
    nz, ny, nx = v.shape
    u = [_field(g, (nx, ny, nz), 48) for _ in range(3)]
    zz, yy, xx = torch.meshgrid(torch.arange(nz, device=DEV), torch.arange(ny, device=DEV),
                                torch.arange(nx, device=DEV), indexing="ij")
    out = torch.empty_like(v)
    pos = []
    for p, d, n in zip((zz, yy, xx), u, (nz, ny, nx)):
        q = (p.float() - (d * (0.5 * peak)).clamp(-peak, peak)).clamp(0, n - 1)
        i = q.floor().clamp(max=max(n - 2, 0)).to(torch.int64)
        pos.append((i, q - i))
    (iz, fz), (iy, fy), (ix, fx) = pos
    flat = v.reshape(-1)
    acc = torch.zeros_like(out)
    for az in (0, 1):
        for ay in (0, 1):
            for ax in (0, 1):
                w = (fz if az else 1 - fz) * (fy if ay else 1 - fy) * (fx if ax else 1 - fx)
                acc += w * flat[((iz + az) * ny + iy + ay) * nx + ix + ax]
    return acc


def _volumes(c, seed):
    """(ref, flt) of a case: tissue classes with Rician noise (12-bit, or the
    same magnitudes as float), or, for float volumes up to 72 voxels a side,
    textured blobs of unit range with Gaussian noise."""
    g = _gen(seed)
    dims = (c["nx"], c["ny"], c["nz"])
    small = c["dtype"] == "f32" and max(dims) <= 72
    if small:
        clean = _field(g, dims, 9) * 0.3 + 0.6
        moved = torch.roll(clean, (1, -2, 3), (0, 1, 2))
        ref = clean + 0.02 * torch.randn(clean.shape, generator=g, device=DEV)
        flt = moved + 0.02 * torch.randn(clean.shape, generator=g, device=DEV)
        return ref.float().contiguous(), flt.float().contiguous()
    f = _field(g, dims, 22) + 0.3 * _field(g, dims, 7)
    clean = torch.where(f < -0.43, 600.0, torch.where(f < 0.43, 1400.0, 2600.0))
    clean = _smooth3(_smooth3(clean))
    moved = _sag(clean, g, min(8.0, max(2.0, 0.5 * c.get("window", 8))))
    del f

    def noisy(v):
        a = v + 40.0 * torch.randn(v.shape, generator=g, device=DEV)
        b = 40.0 * torch.randn(v.shape, generator=g, device=DEV)
        return torch.sqrt(a * a + b * b)

    ref, flt = noisy(clean), noisy(moved)
    if c["dtype"] == "f32":
        return ref.contiguous(), flt.contiguous()
    return tuple(v.round().clamp(0, 4095).to(torch.int16).contiguous().view(torch.uint16)
                 for v in (ref, flt))


def _mask(c):
    """An ellipsoid of the volume's shape (uint8)."""
    nz, ny, nx = c["nz"], c["ny"], c["nx"]
    ax = [((torch.arange(n, device=DEV) - 0.5 * (n - 1)) / (0.45 * n)) ** 2 for n in (nz, ny, nx)]
    return ((ax[0][:, None, None] + ax[1][None, :, None] + ax[2][None, None, :]) <= 1
            ).to(torch.uint8).contiguous()


def prepare(case, seed):
    c = case
    ref, flt = _volumes(c, seed)
    s = {"c": c, "ref": ref, "flt": flt}
    kind, dims = c["kind"], (c["nx"], c["ny"], c["nz"])
    if kind == "step":
        dt = nrr.U16 if c["dtype"] == "u16" else nrr.F32
        s["select_ws"] = torch.empty(nrr.select_workspace_bytes(dims, c["block"], c["stride"]),
                                     dtype=torch.uint8, device=DEV)
        s["match_ws"] = torch.empty(nrr.match_workspace_bytes(dt, dims, c["block"]),
                                    dtype=torch.uint8, device=DEV)
    elif kind == "batch":
        s["plan"] = nrr.BatchPlan(ref, flt, _sets(c))
    elif kind == "mask":
        s["mask"] = _mask(c)
    elif kind == "conf":
        s["centers"] = nrr.select_blocks(ref, c["block"], c["stride"], c["fraction"])
        g = _gen(seed + 1)
        s["conf"] = torch.rand(s["centers"].shape[0], generator=g, device=DEV)
    elif kind == "serve":
        need = sum(nrr.request_footprint(ref, flt, b, st, w, f) for b, w, st, f in _sets(c))
        s["server"] = nrr.Server(device_bytes=need + 6 * ref.numel() * ref.element_size(),
                                 slots=c["slots"])
        s["vols"] = (s["server"].add_volume(ref), s["server"].add_volume(flt))
    torch.cuda.synchronize()
    return s


def run(state):
    s, c = state, state["c"]
    kind, ref, flt = c["kind"], s["ref"], s["flt"]
    if kind == "step":
        centers, ws = nrr.select_and_window_stats(ref, flt, c["block"], c["stride"],
                                                  c["fraction"], c["window"],
                                                  select_workspace=s["select_ws"],
                                                  match_workspace=s["match_ws"])
        disp, ncc, conf = nrr.block_match(ref, flt, centers, c["block"], c["window"],
                                          workspace=ws, prepared=True)
        return {"centers": centers, "disp": disp, "ncc": ncc, "conf": conf}
    if kind == "register":
        centers = nrr.select_blocks(ref, c["block"], c["stride"], c["fraction"])
        disp, ncc, conf = nrr.block_match(ref, flt, centers, c["block"], c["window"])
        return {"centers": centers, "disp": disp, "ncc": ncc, "conf": conf}
    if kind == "aniso":
        b, st, w = _axes(c)
        centers = nrr.select_blocks_aniso(ref, b, st, c["fraction"])
        disp, ncc, conf = nrr.block_match_aniso(ref, flt, centers, b, w)
        return {"centers": centers, "disp": disp, "ncc": ncc, "conf": conf}
    if kind == "batch":
        p = s["plan"]
        p.run()
        return {"centers": p.centers, "disp": p.disp, "ncc": p.ncc, "conf": p.conf}
    if kind == "mask":
        return {"centers": nrr.select_blocks_ex(ref, c["block"], c["stride"], c["fraction"],
                                                mask=s["mask"], connectivity=c["connectivity"])}
    if kind == "conf":
        return {"S": nrr.structure_confidence(ref, s["centers"], c["block"], s["conf"])}
    jobs = [s["server"].submit(*s["vols"], b, st, w, f) for b, w, st, f in _sets(c)]
    for j in jobs:
        j.wait()
    return [{"centers": j.centers, "disp": j.disp, "ncc": j.ncc, "conf": j.conf} for j in jobs]


# ------------------------------------------------------------- 64-bit values

MOST_EXACT_PAIRS = 4.0e10  # the plain torch search of more takes too long


def _origins(dims, b, s):
    """Candidate origins (x, y, z) in grid order, int64 [n, 3]."""
    ax = [torch.arange((d - e) // t + 1, device=DEV) * t for d, e, t in zip(dims, b, s)]
    zz, yy, xx = torch.meshgrid(ax[2], ax[1], ax[0], indexing="ij")
    return torch.stack([xx.reshape(-1), yy.reshape(-1), zz.reshape(-1)], 1)


def _offsets(dims, b):
    nx, ny, _ = dims
    ax = [torch.arange(e, device=DEV) for e in b]
    return ((ax[2][:, None, None] * ny + ax[1][None, :, None]) * nx + ax[0][None, None, :]
            ).reshape(-1)


def _flat(vol):
    return vol.view(torch.int16).to(torch.int64).reshape(-1) if vol.dtype == torch.uint16 \
        else vol.to(torch.float64).reshape(-1)


def _select64(vol, dims, b, s, fraction):
    """Centres by variance rank, ties to the lower grid index, in grid order."""
    org, off, v = _origins(dims, b, s), _offsets(dims, b), _flat(vol)
    _, k = _count(dims, b, s, fraction)
    base = (org[:, 2] * dims[1] + org[:, 1]) * dims[0] + org[:, 0]
    keys = []
    for part in base.split(max(1, 20_000_000 // off.numel())):
        t = v[part[:, None] + off[None, :]]
        if t.dtype == torch.int64:
            keys.append(off.numel() * (t * t).sum(1) - t.sum(1) ** 2)
        else:
            keys.append((t - t.mean(1, keepdim=True)).square().mean(1))
    order = torch.sort(torch.cat(keys), descending=True, stable=True).indices[:k]
    half = torch.tensor([(e - 1) // 2 for e in b], device=DEV)
    return (org[torch.sort(order).values] + half).to(torch.int32)


def _search64(ref, flt, dims, centers, b, w):
    """The exhaustive NCC search in 64 bits: (disp, ncc) with the smallest
    shift index among equal values."""
    nx, ny, nz = dims
    off, N = _offsets(dims, b), math.prod(b)
    fr, ff = _flat(ref).double(), _flat(flt).double()
    half = [(e - 1) // 2 for e in b]
    org = centers.to(torch.int64) - torch.tensor(half, device=DEV)
    n = org.shape[0]
    base = (org[:, 2] * ny + org[:, 1]) * nx + org[:, 0]
    t = fr[base[:, None] + off[None, :]]
    t = t - t.mean(1, keepdim=True)
    vt = t.square().sum(1)
    best = torch.full((n,), -math.inf, dtype=torch.float64, device=DEV)
    disp = torch.zeros((n, 3), dtype=torch.int32, device=DEV)
    lim = torch.tensor([d - e for d, e in zip(dims, b)], device=DEV)
    row = torch.arange(-w[0], w[0] + 1, device=DEV)
    take = max(1, 30_000_000 // (N * max(n, 1)))
    for dz in range(-w[2], w[2] + 1):
        for dy in range(-w[1], w[1] + 1):
            for dx in row.split(take):
                m = dx.numel()
                o = org[:, None, :].expand(n, m, 3).clone()
                o[:, :, 0] += dx
                o[:, :, 1] += dy
                o[:, :, 2] += dz
                ok = ((o >= 0) & (o <= lim)).all(2)
                o = torch.minimum(o.clamp(min=0), lim)
                f = ff[((o[:, :, 2] * ny + o[:, :, 1]) * nx + o[:, :, 0])[:, :, None] + off]
                f = f - f.mean(2, keepdim=True)
                den = vt[:, None] * f.square().sum(2)
                q = (f * t[:, None, :]).sum(2) / den.clamp(min=1e-300).sqrt()
                q = torch.where(den > 0, q, torch.zeros_like(q))
                q = torch.where(ok, q, torch.full_like(q, -math.inf))
                v, i = q.max(1)
                i = (q == v[:, None]).to(torch.int8).argmax(1)
                up = v > best
                best = torch.where(up, v, best)
                d = torch.stack([dx[i], torch.full_like(i, dy), torch.full_like(i, dz)], 1)
                disp = torch.where(up[:, None], d.to(torch.int32), disp)
    return disp, best


def _registration64(ref, flt, dims, b, s, w, fraction):
    centers = _select64(ref, dims, b, s, fraction)
    disp, ncc = _search64(ref, flt, dims, centers, b, w)
    return {"centers": centers, "disp": disp, "ncc": ncc, "conf": ncc.clamp(min=0)}


def _confidence64(ref, dims, centers, block, conf):
    nx, ny, nz = dims
    v = _flat(ref).double().reshape(nz, ny, nx)
    grad = []
    for d in (2, 1, 0):
        g, n = torch.empty_like(v), v.shape[d]
        g.narrow(d, 1, n - 2).copy_((v.narrow(d, 2, n - 2) - v.narrow(d, 0, n - 2)) / 2)
        g.narrow(d, 0, 1).copy_(v.narrow(d, 1, 1) - v.narrow(d, 0, 1))
        g.narrow(d, n - 1, 1).copy_(v.narrow(d, n - 1, 1) - v.narrow(d, n - 2, 1))
        grad.append(g.reshape(-1))
    org = centers.to(torch.int64) - (block - 1) // 2
    base = (org[:, 2] * ny + org[:, 1]) * nx + org[:, 0]
    at = base[:, None] + _offsets(dims, (block,) * 3)[None, :]
    gx, gy, gz = (g[at] for g in grad)
    j = torch.stack([(a * b).sum(1) for a, b in
                     ((gx, gx), (gy, gy), (gz, gz), (gx, gy), (gx, gz), (gy, gz))], 1)
    tr = j[:, :3].sum(1, keepdim=True)
    return torch.where(tr > 0, conf.double()[:, None] * j / tr.clamp(min=1e-300),
                       torch.zeros_like(j))


def exact(case, seed):
    c = case
    dims = (c["nx"], c["ny"], c["nz"])
    if c["kind"] == "mask":
        return None  # centres only: whole numbers
    if c["kind"] in ("batch", "serve"):
        sets = [((b,) * 3, (s,) * 3, (w,) * 3, f) for b, w, s, f in _sets(c)]
    else:
        sets = [_axes(c) + (c["fraction"],)]
    pairs = sum(_count(dims, b, s, f)[1] * math.prod(b) * math.prod(2 * a + 1 for a in w)
                for b, s, w, f in sets)
    if c["kind"] != "conf" and pairs > MOST_EXACT_PAIRS:
        return None
    ref, flt = _volumes(c, seed)
    if c["kind"] == "conf":
        b, s, _, f = sets[0]
        centers = _select64(ref, dims, b, s, f)
        g = _gen(seed + 1)
        conf = torch.rand(centers.shape[0], generator=g, device=DEV)
        return {"S": _confidence64(ref, dims, centers, c["block"], conf)}
    got = [_registration64(ref, flt, dims, b, s, w, f) for b, s, w, f in sets]
    if c["kind"] == "serve":
        return got
    return {k: torch.cat([g[k] for g in got]) for k in ("centers", "disp", "ncc", "conf")}
