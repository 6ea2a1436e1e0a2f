"""Performance cases of the filtering library: the calls its users make, each
with its inputs, the work it cannot do without, and its results in 64 bits.

listed() names the cases, draw(rng) gives further ones of the same ranges,
prepare(case, seed) makes what a program holds before the call (textures,
query streams, output buffers), run(state) is one pass through the public
entry points, work(case) the bytes and operations of a pass, and
exact(case, seed) the results by plain torch arithmetic in binary64.

Inputs are made on the GPU from the seed alone: sparse grids of thresholded
fBm noise with ray samples through them, textures and DCT-compressed sets of
fBm noise seen by a pinhole camera over a ground plane, materials of bumps
with scattered shading records, and latent grids with a small decoder.
"""
import math

import numpy as np
import torch

import paper_2305_05810_amd as stf

DEV = "cuda:0"
F64 = torch.float64

FILTERS = {"linear": stf.STF_LINEAR, "cubic": stf.STF_CUBIC_BSPLINE, "keys": stf.STF_CUBIC_KEYS,
           "mitchell": stf.STF_CUBIC_MITCHELL}
MODES = {"deterministic": stf.STF_DETERMINISTIC, "stochastic": stf.STF_STOCHASTIC, "fis": stf.STF_STOCHASTIC_FIS}
GAUSS = {"fis": stf.STF_GAUSS_FIS, "fis_mean": stf.STF_GAUSS_FIS_MEAN, "discrete": stf.STF_GAUSS_DISCRETE,
         "discrete_mean": stf.STF_GAUSS_DISCRETE_MEAN}
SHADE = {"shade_after_filter": stf.STF_SHADE_AFTER_FILTER, "filter_after_shade": stf.STF_FILTER_AFTER_SHADE,
         "stochastic": stf.STF_SHADE_STOCHASTIC}
TAPS = {"linear": 2, "cubic": 4, "keys": 4, "mitchell": 4}
FMT_TORCH = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16, "fp8_e4m3": torch.float8_e4m3fn,
             "u8": torch.uint8}
DECODE_FLOPS = 2 * (8 * 64 + 64 * 64 + 64 * 8)


def listed():
    return [
        # The library's headline: one stochastic tap per sample of a ray
        # march through a sparse volume, most samples in empty space.
        {"name": "grid_ray_stochastic", "kind": "grid", "dim": 512, "fmt": "f32", "stream": "ray", "n": 1 << 24,
         "filter": "cubic", "mode": "stochastic"},
        # The 64-tap reference filter where a renderer that skips empty space
        # calls it: every sample inside the medium.  An odd count.
        {"name": "grid_medium_deterministic", "kind": "grid", "dim": 512, "fmt": "f32", "stream": "medium",
         "n": 4194301, "filter": "cubic", "mode": "deterministic"},
        # The same lookups on 16-bit voxels, ordered by the library first and
        # scattered back: sort and filter of one batch.
        {"name": "grid_sorted_f16", "kind": "sorted", "dim": 512, "fmt": "f16", "n": 1 << 22, "filter": "cubic",
         "mode": "deterministic"},
        # The smallest call: a 256^2 RGBA texture and 65,536 lookups, where
        # the launch and the binding count.
        {"name": "tex2d_small", "kind": "tex2d", "width": 256, "height": 256, "channels": 4, "fmt": "f32",
         "n": 65536, "view": "random", "filter": "cubic", "mode": "stochastic"},
        # A 1080p frame of an 8-bit RGBA texture magnified with the 16-tap
        # B-spline (the deterministic image a renderer compares with).
        {"name": "tex2d_frame_u8", "kind": "tex2d", "width": 4096, "height": 4096, "channels": 4, "fmt": "u8",
         "n": 1920 * 1080, "view": "frame", "filter": "cubic", "mode": "deterministic"},
        # The DCT-compressed nine-channel set over a 4K frame, 16 taps each.
        {"name": "dct_frame_deterministic", "kind": "dct", "size": 4096, "channels": 9, "n": 3840 * 2160,
         "view": "frame", "filter": "cubic", "mode": "deterministic"},
        # Gaussian magnification by filter importance sampling on that set
        # (one decode per lookup; the sigma the benchmark reports).
        {"name": "gauss_frame_fis", "kind": "gauss", "size": 4096, "channels": 9, "n": 3840 * 2160, "sigma": 0.5,
         "mode": "fis"},
        # Anisotropic minification of a frame: a MIP level and one texel of
        # the ellipse per lookup.
        {"name": "ewa_frame_stochastic", "kind": "ewa", "size": 4096, "channels": 4, "fmt": "u8",
         "n": 3840 * 2160, "aniso": 8.0, "mode": "stochastic"},
        # Filter-after-shading: 16 GGX evaluations per scattered record.
        {"name": "shade_filter_after", "kind": "shade", "size": 4096, "n": 1 << 22, "filter": "cubic",
         "mode": "filter_after_shade"},
        # The neural texture decoded at all 16 taps of scattered lookups.
        {"name": "neural_decode", "kind": "neural", "size": 4096, "lat": 1024, "n": 1 << 22, "filter": "cubic",
         "mode": "deterministic"},
        # Fitting a neural texture: a run of Adam steps, the parameters read
        # back at its end.
        {"name": "neural_train", "kind": "train", "size": 2048, "lat": 512, "batch": 1 << 18, "steps": 32},
        # Serving: a burst of requests of mixed sizes on two resident
        # textures, waited for.
        {"name": "serve_burst", "kind": "serve", "dim": 256, "size": 2048, "fmt": "f16", "requests": 192,
         "median": 16384},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["grid", "grid", "sorted", "tex2d", "tex2d", "dct", "dct", "gauss", "ewa", "shade", "neural",
                       "train", "serve"])
    fmt3 = rng.choice(["f32", "f16", "bf16", "fp8_e4m3"])
    fmt2 = rng.choice(["f32", "f16", "bf16", "u8"])
    filt = rng.choice(["linear", "cubic", "cubic", "keys", "mitchell"])
    mode = rng.choice(["deterministic", "stochastic"])
    if kind == "grid":
        stream = rng.choice(["ray", "medium"])
        return {"kind": kind, "dim": rng.choice([128, 256, 384, 512]), "fmt": fmt3, "stream": stream,
                "n": _log_int(rng, 50_000, 8_000_000 if stream == "ray" else 4_000_000), "filter": filt, "mode": mode}
    if kind == "sorted":
        return {"kind": kind, "dim": rng.choice([256, 512]), "fmt": fmt3, "n": _log_int(rng, 100_000, 4_000_000),
                "filter": rng.choice(["linear", "cubic", "keys"]), "mode": mode}
    if kind == "tex2d":
        view = rng.choice(["random", "frame"])
        return {"kind": kind, "width": _log_int(rng, 37, 4096), "height": _log_int(rng, 37, 4096),
                "channels": rng.choice([1, 2, 3, 4, 4]), "fmt": fmt2, "n": _log_int(rng, 10_000, 8_000_000),
                "view": view, "filter": filt, "mode": mode}
    if kind == "dct":
        return {"kind": kind, "size": rng.choice([512, 1024, 2048, 4096]), "channels": rng.choice([1, 3, 4, 9, 16]),
                "n": _log_int(rng, 50_000, 6_000_000), "view": rng.choice(["random", "frame"]), "filter": filt,
                "mode": mode}
    if kind == "gauss":
        return {"kind": kind, "size": rng.choice([1024, 2048, 4096]), "channels": rng.choice([3, 4, 9]),
                "n": _log_int(rng, 50_000, 2_000_000), "sigma": rng.choice([0.3, 0.5, 0.8]),
                "mode": rng.choice(["fis", "discrete", "fis_mean", "discrete_mean"])}
    if kind == "ewa":
        return {"kind": kind, "size": rng.choice([512, 1024, 2048, 4096]), "channels": rng.choice([1, 3, 4]),
                "fmt": rng.choice(["u8", "f16", "f32"]), "n": _log_int(rng, 50_000, 6_000_000),
                "aniso": rng.choice([1.0, 4.0, 8.0, 16.0, 64.0]), "mode": mode}
    if kind == "shade":
        return {"kind": kind, "size": rng.choice([512, 1024, 2048, 4096]), "n": _log_int(rng, 50_000, 4_000_000),
                "filter": rng.choice(["linear", "cubic"]), "mode": rng.choice(list(SHADE))}
    if kind == "neural":
        size = rng.choice([512, 1024, 2048, 4096])
        return {"kind": kind, "size": size, "lat": size // rng.choice([2, 4, 8]), "n": _log_int(rng, 20_000, 4_000_000),
                "filter": rng.choice(["linear", "cubic"]), "mode": mode}
    if kind == "train":
        size = rng.choice([512, 1024, 2048])
        return {"kind": kind, "size": size, "lat": size // rng.choice([2, 4, 8]),
                "batch": _log_int(rng, 5_000, 200_000), "steps": rng.choice([4, 8, 16])}
    return {"kind": "serve", "dim": rng.choice([128, 256]), "size": rng.choice([512, 1024, 2048]), "fmt": fmt3,
            "requests": rng.randrange(16, 160), "median": _log_int(rng, 2048, 20000)}


# ----------------------------------------------------------------------------
# inputs
# ----------------------------------------------------------------------------
def _gen(seed, salt):
    g = torch.Generator(device=DEV)
    g.manual_seed((int(seed) * 1_000_003 + salt) & 0x7FFFFFFFFFFFFFFF)
    return g


def _rand(g, *shape, dtype=torch.float32):
    return torch.rand(*shape, generator=g, device=DEV, dtype=dtype)


def _lerp_axis(lat, axis, n, period, offset):
    x = (torch.arange(n, device=DEV, dtype=F64) + offset) / period
    c = x.floor().long()
    f = (x - c)
    w = (f * f * (3 - 2 * f)).float()
    shape = [1] * lat.dim()
    shape[axis] = n
    w = w.view(shape)
    return lat.index_select(axis, c) * (1 - w) + lat.index_select(axis, c + 1) * w


def _fbm(g, dims, period, octaves=5):
    """Value-noise fBm with smoothstep-faded multilinear interpolation."""
    out = torch.zeros(dims, device=DEV)
    for o in range(octaves):
        p = period / 2 ** o
        offs = [float(v) * p for v in _rand(g, len(dims)).cpu()]
        lat = _rand(g, *[int((n + p) / p) + 3 for n in dims]) * 2 - 1
        for a in reversed(range(len(dims))):
            lat = _lerp_axis(lat, a, dims[a], p, offs[a])
        out += lat * 0.5 ** o
    return out


def _rays(g, dims, n_rays, spr=256):
    """Ray samples in voxel index space, ray-major: random chords of the box."""
    hi = torch.tensor(dims, device=DEV, dtype=F64) - 1
    o = _rand(g, n_rays, 3, dtype=F64) * hi
    z = _rand(g, n_rays, dtype=F64) * 2 - 1
    phi = _rand(g, n_rays, dtype=F64) * (2 * math.pi)
    r = (1 - z * z).clamp_min(0).sqrt()
    d = torch.stack([r * phi.cos(), r * phi.sin(), z], 1)
    d = torch.where(d.abs() < 1e-12, torch.full_like(d, 1e-12), d)
    ta, tb = -o / d, (hi - o) / d
    t0 = torch.minimum(ta, tb).amax(1)
    t1 = torch.maximum(ta, tb).amin(1)
    k = torch.arange(spr, device=DEV, dtype=F64) + _rand(g, n_rays, 1, dtype=F64)
    t = t0[:, None] + k * ((t1 - t0) / spr)[:, None]
    return (o[:, None, :] + t[:, :, None] * d[:, None, :]).float().reshape(-1, 3)


def _grid_inputs(case, seed):
    """Density (z, y, x) in the storage format, leaf occupancy, queries."""
    g, dim = _gen(seed, 1), case["dim"]
    dens = (_fbm(g, (dim, dim, dim), 64.0) * 0.65 - 0.55).clamp_min(0)
    nb = dim // 8
    leaves = dens.view(nb, 8, nb, 8, nb, 8).permute(0, 2, 4, 1, 3, 5).reshape(nb, nb, nb, 512)
    active = leaves.amax(3) > 0
    if not bool(active.any()):
        active[0, 0, 0] = True
    return dens.to(FMT_TORCH[case["fmt"]]), leaves, active


def _grid_queries(case, seed, active):
    g, dim, n = _gen(seed, 2), case["dim"], case["n"]
    if case.get("stream") == "ray":
        return _rays(g, (dim,) * 3, -(-n // 256))[:n].contiguous()
    nb = dim // 8
    occ = torch.zeros((nb + 2,) * 3, dtype=torch.bool, device=DEV)   # one empty border leaf
    occ[1:-1, 1:-1, 1:-1] = active
    kept, total = [], 0
    while total < n:
        p = _rays(g, (dim,) * 3, 65536)
        c = p.floor().long() - 1
        lo, hi = (c >> 3).clamp(-1, nb) + 1, ((c + 3) >> 3).clamp(-1, nb) + 1
        hit = torch.zeros(p.shape[0], dtype=torch.bool, device=DEV)
        for sx in (lo[:, 0], hi[:, 0]):
            for sy in (lo[:, 1], hi[:, 1]):
                for sz in (lo[:, 2], hi[:, 2]):
                    hit |= occ[sz, sy, sx]
        kept.append(p[hit])
        total += int(kept[-1].shape[0])
        if total == 0 or len(kept) >= 8:   # a nearly empty medium: its samples again
            kept = (kept * (n // max(total, 1) + 1)) if total else [p]
            break
    q = torch.cat(kept)
    if q.shape[0] < n:
        q = q.repeat(-(-n // q.shape[0]), 1)
    return q[:n].contiguous()


def _host(t):
    return t.contiguous().view(torch.uint8).cpu().numpy() if t.dtype in (torch.bfloat16, torch.float8_e4m3fn) \
        else t.contiguous().cpu().numpy()


def _make_grid(case, stored, leaves, active):
    dim = case["dim"]
    kz, ky, kx = torch.nonzero(active, as_tuple=True)
    origins = torch.stack([kx, ky, kz], 1).int() * 8
    vals = leaves[kz, ky, kx].to(FMT_TORCH[case["fmt"]])
    return stf.stf_create_sparse_grid3d((dim,) * 3, stf.FORMATS[case["fmt"]], origins.cpu().numpy(), _host(vals))


def _tex_inputs(case, seed):
    g = _gen(seed, 3)
    h, w, c = case.get("height", case.get("size")), case.get("width", case.get("size")), case["channels"]
    t = torch.stack([(0.5 + 0.5 * _fbm(g, (h, w), 64.0)).clamp(0, 1) for _ in range(c)], 2)
    if case["fmt"] == "u8":
        return (t * 255).round().to(torch.uint8)
    return t.to(FMT_TORCH[case["fmt"]])


def _frame_dirs(g, n):
    """Pixels of a 16:9 frame of at least n pixels, pixel order: directions of
    a camera pitched 25 degrees down (60-degree field of view)."""
    h = max(9, math.ceil(math.sqrt(n * 9 / 16)))
    w = -(-n // h)
    jx, jy = (float(v) for v in _rand(g, 2).cpu())
    px = ((torch.arange(w, device=DEV, dtype=F64) + jx) / w * 2 - 1) * math.tan(math.radians(30))
    py = (1 - (torch.arange(h, device=DEV, dtype=F64) + jy) / h * 2) * math.tan(math.radians(30)) * h / w
    y, x = torch.meshgrid(py, px, indexing="ij")
    s, c = math.sin(math.radians(25)), math.cos(math.radians(25))
    return x, c + y * s, -s + y * c, w, h


def _uv(case, seed):
    g, n = _gen(seed, 4), case["n"]
    if case.get("view", "frame") == "random":
        return _rand(g, n, 2)
    dx, dy, dz, w, h = _frame_dirs(g, n)
    hit = dz < -1e-6
    t = torch.where(hit, 2 / (-dz).clamp_min(1e-6), torch.zeros_like(dz))
    u, v = dx * t / 8, dy * t / 8   # the texture tiled every 8 units
    uv = torch.stack([u - u.floor(), v - v.floor()], 2)
    sky = _rand(g, h, w, 2, dtype=F64)
    return torch.where(hit[:, :, None], uv, sky).float().reshape(-1, 2)[:n].clamp_max(1 - 2.0 ** -24).contiguous()


def _ewa_queries(case, seed):
    g, n = _gen(seed, 5), case["n"]
    dx, dy, dz, w, h = _frame_dirs(g, n)
    hit = dz < -1e-6
    t = torch.where(hit, 2 / (-dz).clamp_min(1e-6), torch.zeros_like(dz))
    su, sv = dx * t / 2, dy * t / 2   # tiled every 2 units: minified, anisotropic
    dif = lambda a, d: torch.diff(a, dim=d, append=a.narrow(d, -1, 1) * 2 - a.narrow(d, -2, 1))
    rec = torch.stack([su - su.floor(), sv - sv.floor(), dif(su, 1), dif(sv, 1), dif(su, 0), dif(sv, 0)], 2)
    sky = torch.zeros_like(rec)
    sky[:, :, 0:2] = _rand(g, h, w, 2, dtype=F64)
    sky[:, :, 2] = sky[:, :, 5] = 1.0 / 4096
    low = hit.clone()   # a pixel whose lower neighbour misses the plane has no difference
    low[:-1] &= hit[1:]
    return torch.where(low[:, :, None], rec, sky).float().reshape(-1, 6)[:n].contiguous()


def _mips(t):
    lv, cur = [t], t.to(F64)
    while cur.shape[0] > 1 or cur.shape[1] > 1:
        cur = torch.nn.functional.avg_pool2d(cur.permute(2, 0, 1), 2).permute(1, 2, 0)
        lv.append(cur.round().to(t.dtype) if t.dtype == torch.uint8 else cur.to(t.dtype))
    return lv


def _dct_inputs(case, seed):
    """(H/8, W/8, C) words: six DCT codes of 8-bit noise channels per block."""
    g, s, c = _gen(seed, 6), case["size"], case["channels"]
    i = torch.arange(8, device=DEV, dtype=F64)
    D = torch.cos((2 * i[None, :] + 1) * i[:, None] * math.pi / 16) * 0.5
    D[0] *= math.sqrt(0.5)
    words = torch.zeros(s // 8, s // 8, c, dtype=torch.int64, device=DEV)
    for ch in range(c):
        t = (_fbm(g, (s, s), 64.0 if ch % 3 else 32.0) * 0.5 + 0.5).clamp(0, 1)
        t = (t * 255).round().to(F64) / 255
        b = t.view(s // 8, 8, s // 8, 8).permute(0, 2, 1, 3)
        k = D[:3] @ b @ D[:3].T
        w = (k[..., 0, 0] * 127 / 8).round().clamp(0, 127).long()
        for j, (v, u) in enumerate(((0, 1), (1, 0), (2, 0), (1, 1), (0, 2))):
            w |= ((k[..., v, u] * 7.5).round().clamp(-15, 15).long() + 16) << (7 + 5 * j)
        words[:, :, ch] = w
    return words


def _material_inputs(case, seed):
    """Level 0 of a material: (H, W, 4) uint8 albedo and roughness, (H, W, 2)
    float16 normals of a bumpy height field, and its two coarser levels."""
    g, s = _gen(seed, 7), case["size"]
    a = torch.randint(0, 256, (s, s, 4), generator=g, device=DEV, dtype=torch.uint8)
    r = _rand(g, s, s)
    a[:, :, 3] = (255 * (1 - (1 - r) ** 0.4) * 0.9).to(torch.uint8)   # mostly low roughness
    hgt = _fbm(g, (s, s), 32.0) * 2.0
    hx, hy = (torch.roll(hgt, -1, 1) - torch.roll(hgt, 1, 1)) * 0.5, (torch.roll(hgt, -1, 0) - torch.roll(hgt, 1, 0)) * 0.5
    inv = 1 / (hx * hx + hy * hy + 1).sqrt()
    nrm = torch.stack([-hx * inv, -hy * inv], 2).half()
    lv = [(a, nrm)]
    for _ in range(2):
        pa, pn = lv[-1]
        h2 = pa.shape[0] // 2
        qa = pa.int().view(h2, 2, h2, 2, 4).sum((1, 3))
        qn = pn.float().view(h2, 2, h2, 2, 2).sum((1, 3)) / 4
        lv.append((((qa + 2) >> 2).to(torch.uint8), qn.half()))
    return lv


def _material_bytes(lv):
    return [torch.cat([a, n.contiguous().view(torch.uint8).view(*a.shape[:2], 4)], 2).contiguous().cpu().numpy()
            for a, n in lv]


def _shade_queries(case, seed):
    g, n = _gen(seed, 8), case["n"]
    rec = torch.empty(n, 9, device=DEV)
    rec[:, 0:2] = _rand(g, n, 2)
    rec[:, 2] = torch.exp2(_rand(g, n) * 4 - 2)
    for k in (3, 6):
        z, phi = _rand(g, n, dtype=F64), _rand(g, n, dtype=F64) * (2 * math.pi)
        r = (1 - z * z).clamp_min(0).sqrt()
        rec[:, k], rec[:, k + 1], rec[:, k + 2] = r * phi.cos(), r * phi.sin(), z
    return rec


def _neural_inputs(case, seed):
    g = _gen(seed, 9)
    L = case["lat"]
    lat = torch.randn(L, L, 8, generator=g, device=DEV) * 0.1
    w = [torch.randn(64 * 8, generator=g, device=DEV) * 0.5, torch.randn(64, generator=g, device=DEV) * 0.05,
         torch.randn(64 * 64, generator=g, device=DEV) * math.sqrt(2 / 64),
         torch.randn(64, generator=g, device=DEV) * 0.05,
         torch.randn(8 * 64, generator=g, device=DEV) * 0.125, torch.randn(8, generator=g, device=DEV) * 0.05]
    return lat, torch.cat(w)


def _target(case, seed):
    g, s = _gen(seed, 10), case["size"]
    return torch.stack([0.5 + 0.5 * _fbm(g, (s, s), 64.0 if c % 2 else 32.0) for c in range(8)], 2).contiguous()


def _requests(case):
    """Sizes, textures, filters and offsets of a burst of requests (the
    burst's shape belongs to the case; the queries come from the seed)."""
    k = case["requests"]
    r = np.random.default_rng([k, case["median"], 11])
    sizes = np.clip(np.exp(r.normal(np.log(case["median"]), 1.0, k)), 256, 1 << 17).astype(np.int64)
    which = r.integers(0, 2, k)
    which[:2] = (0, 1)
    cubic = r.random(k) < 0.5
    offs = np.zeros(k, np.int64)
    for t in (0, 1):
        m = which == t
        offs[m] = np.concatenate([[0], np.cumsum(sizes[m])[:-1]])
    totals = [int(sizes[which == t].sum()) for t in (0, 1)]
    return sizes, which, cubic, offs, totals


def prepare(case, seed):
    kind, s = case["kind"], {"case": case}
    s["seed"] = 0x5EED + int(seed) * 7919
    if kind in ("grid", "sorted"):
        stored, leaves, active = _grid_inputs(case, seed)
        s["tex"] = _make_grid(case, stored, leaves, active)
        s["q"] = _grid_queries(case, seed, active)
        s["out"] = torch.empty(case["n"], 1, device=DEV)
        if kind == "sorted":
            s["sq"] = torch.empty_like(s["q"])
            s["order"] = torch.empty(case["n"], dtype=torch.int32, device=DEV)
            s["ws"] = torch.empty(stf.stf_sort_workspace_bytes(case["n"]), dtype=torch.uint8, device=DEV)
    elif kind == "tex2d":
        s["tex"] = stf.stf_create_texture2d(case["width"], case["height"], case["channels"],
                                            stf.FORMATS[case["fmt"]], [_host(_tex_inputs(case, seed))])
        s["q"] = _uv(case, seed)
        s["out"] = torch.empty(case["n"], case["channels"], device=DEV)
    elif kind in ("dct", "gauss"):
        words = _dct_inputs(case, seed).cpu().numpy().astype(np.uint32)
        s["tex"] = stf.stf_create_dct_texture2d(case["size"], case["size"], case["channels"], words)
        s["q"] = _uv(case, seed)
        s["out"] = torch.empty(case["n"], case["channels"], device=DEV)
    elif kind == "ewa":
        lv = [_host(t) for t in _mips(_tex_inputs(case, seed))]
        s["tex"] = stf.stf_create_texture2d(case["size"], case["size"], case["channels"],
                                            stf.FORMATS[case["fmt"]], lv)
        s["q"] = _ewa_queries(case, seed)
        s["out"] = torch.empty(case["n"], case["channels"], device=DEV)
    elif kind == "shade":
        s["tex"] = stf.stf_create_material2d(case["size"], case["size"], _material_bytes(_material_inputs(case, seed)))
        s["q"] = _shade_queries(case, seed)
        s["out"] = torch.empty(case["n"], 3, device=DEV)
    elif kind == "neural":
        lat, mlp = _neural_inputs(case, seed)
        s["nt"] = stf.stf_ntex_create(case["size"], case["size"], lat.cpu().numpy(), mlp.cpu().numpy())
        stf.stf_ntex_prepare_inference(s["nt"])
        s["q"] = _rand(_gen(seed, 12), case["n"], 2)
        s["out"] = torch.empty(case["n"], 8, device=DEV)
    elif kind == "train":
        lat, mlp = _neural_inputs(case, seed)
        s["nt"] = stf.stf_ntex_create(case["size"], case["size"], lat.cpu().numpy(), mlp.cpu().numpy())
        s["target"] = _target(case, seed)
        s["loss"] = torch.empty(case["steps"], device=DEV)
    elif kind == "serve":
        stored, leaves, active = _grid_inputs(case, seed)
        s["texs"] = [_make_grid(case, stored, leaves, active),
                     stf.stf_create_material2d(case["size"], case["size"],
                                               _material_bytes(_material_inputs(case, seed))[:1])]
        sizes, which, cubic, offs, totals = _requests(case)
        s["q"] = _serve_queries(case, seed, totals)
        s["out"] = [torch.empty(totals[0], 1, device=DEV), torch.empty(totals[1], 6, device=DEV)]
        s["srv"] = stf.stf_server_create(1 << 28, 4096, 1 << 18)
        s["reqs"] = [(s["texs"][t], s["q"][t].data_ptr() + 4 * (3, 2)[t] * int(o), int(n),
                      stf.STF_CUBIC_BSPLINE if c else stf.STF_LINEAR, k,
                      s["out"][t].data_ptr() + 4 * (1, 6)[t] * int(o), None, 0.0)
                     for k, (n, t, c, o) in enumerate(zip(sizes, which, cubic, offs))]
    return s


def _serve_queries(case, seed, totals):
    return [_rays(_gen(seed, 13), (case["dim"],) * 3, -(-totals[0] // 256))[:totals[0]].contiguous(),
            _rand(_gen(seed, 14), totals[1], 2)]


def run(s):
    c = s["case"]
    kind = c["kind"]
    if kind in ("grid", "tex2d", "dct"):
        stf.stf_filter(s["tex"], s["q"], FILTERS[c["filter"]], MODES[c["mode"]], s["seed"], s["out"])
    elif kind == "sorted":
        stf.stf_sort_queries(s["tex"], s["q"], s["sq"], s["order"], s["ws"])
        stf.stf_filter_ordered(s["tex"], s["sq"], s["order"], FILTERS[c["filter"]], MODES[c["mode"]], s["seed"],
                               s["out"], flags=stf.STF_ORDER_SCATTER)
        return s["out"], s["order"]
    elif kind == "gauss":
        stf.stf_filter_gaussian(s["tex"], s["q"], c["sigma"], GAUSS[c["mode"]], s["seed"], s["out"])
    elif kind == "ewa":
        stf.stf_filter_ewa(s["tex"], s["q"], c["aniso"], MODES[c["mode"]], s["seed"], s["out"])
    elif kind == "shade":
        stf.stf_shade_filter(s["tex"], s["q"], FILTERS[c["filter"]], SHADE[c["mode"]], s["seed"], s["out"])
    elif kind == "neural":
        stf.stf_ntex_filter(s["nt"], s["q"], FILTERS[c["filter"]], MODES[c["mode"]], s["seed"], s["out"])
    elif kind == "train":
        stf.stf_ntex_train(s["nt"], s["target"], c["steps"], c["batch"], 1e-2, 1e-3, 7, s["loss"])
        lat, mlp = stf.stf_ntex_get_params(s["nt"])
        return s["loss"], lat, mlp
    elif kind == "serve":
        stf.stf_server_replay(s["srv"], s["reqs"],
                              stf.STF_SERVE_QUERIES_ON_DEVICE | stf.STF_SERVE_RESULTS_ON_DEVICE, 60.0)
        return s["out"]
    return s["out"]


def work(case):
    """Each query read once and each result written once; texels as far as the
    lookups can touch them, at most the texture once."""
    kind, n = case["kind"], case.get("n", 0)
    if kind in ("grid", "sorted"):
        nt = 1 if case["mode"] == "stochastic" else TAPS[case["filter"]] ** 3
        vox = stf.FORMAT_BYTES[stf.FORMATS[case["fmt"]]]
        held = 0.07 * case["dim"] ** 3 * vox   # the stored leaves
        b = n * 16 + min(n * nt * vox, held)
        if kind == "sorted":   # queries read and written in order, the order array, the filter's own streams
            b += n * (12 + 12 + 4 + 4)
        return {"bytes": b, "flops": 2 * nt * n}
    if kind in ("tex2d", "dct", "gauss"):
        taps = 1 if case["mode"] in ("stochastic", "fis", "discrete") else 16
        if kind == "tex2d":
            if case["mode"] == "deterministic":
                taps = TAPS[case["filter"]] ** 2
            c = case["channels"]
            tex = case["width"] * case["height"] * c * stf.FORMAT_BYTES[stf.FORMATS[case["fmt"]]]
        else:
            if kind == "dct" and case["mode"] == "deterministic":
                taps = TAPS[case["filter"]] ** 2
            if case["mode"] == "fis_mean":
                taps = (2 * math.ceil(6 * case["sigma"]) + 4) ** 2
            c = case["channels"]
            tex = case["size"] ** 2 // 64 * c * 4
        return {"bytes": n * (8 + 4 * c) + min(tex, n * taps * c * 4), "flops": 2.0 * taps * c * n}
    if kind == "ewa":
        c = case["channels"]
        tex = case["size"] ** 2 * c * stf.FORMAT_BYTES[stf.FORMATS[case["fmt"]]] * 4 // 3
        return {"bytes": n * (24 + 4 * c) + min(tex, n * 16 * c), "flops": 40.0 * 8 * n}
    if kind == "shade":
        taps = 1 if case["mode"] == "stochastic" else TAPS[case["filter"]] ** 2
        ev = taps if case["mode"] == "filter_after_shade" else 1
        return {"bytes": n * 48 + min(n * taps * 8, case["size"] ** 2 * 8 * 21 // 16), "flops": 120.0 * ev * n}
    if kind == "neural":
        taps = 1 if case["mode"] == "stochastic" else TAPS[case["filter"]] ** 2
        return {"bytes": n * 40 + min(n * taps * 64, case["lat"] ** 2 * 64), "flops": DECODE_FLOPS * taps * n}
    if kind == "train":
        per = case["batch"] * (32 + 4 * 32) + case["lat"] ** 2 * 8 * 28
        return {"bytes": case["steps"] * per, "flops": 3.0 * DECODE_FLOPS * case["batch"] * case["steps"]}
    total = case["requests"] * case["median"] * 1.6
    return {"bytes": total * (16 + 32) / 2, "flops": total * 2}


# ----------------------------------------------------------------------------
# results in binary64
# ----------------------------------------------------------------------------
M32 = 0xFFFFFFFF


def _pcg(x):
    state = (x * 747796405 + 2891336453) & M32
    word = (((state >> ((state >> 28) + 4)) ^ state) * 277803737) & M32
    return (word >> 22) ^ word


def _key(seed):
    lo, hi = torch.tensor(seed & M32), torch.tensor((seed >> 32) & M32)
    return int(_pcg(lo ^ _pcg(hi)))


def _uniform(seed, ids, a):
    """u * 2^24 of hash index a (exact in binary32)."""
    b = _pcg(ids ^ _key(seed))
    return (_pcg((b + a) & M32) >> 8).float()


def _cells(x):
    f = x.floor()
    return f.long(), x - f


def _choose(filt, t, m):
    """Tap offset of the linear or cubic draw in its defined binary32 steps."""
    if filt == "linear":
        return (m < t * 16777216.0).long()
    k6 = torch.tensor(float.fromhex("0x1.555556p-3") * 16777216.0, device=DEV)
    s = 1 - t
    c1 = (s * s) * s * k6
    c2 = c1 + (4 + (3 * (t * t)) * (t - 2)) * k6
    c3 = 16777216.0 - (t * t) * t * k6
    return -1 + (m >= c1).long() + (m >= c2).long() + (m >= c3).long()


def _weights(filt, t):
    """Offsets and binary64 weights of the per-axis taps."""
    t = t.to(F64)
    s = 1 - t
    if filt == "linear":
        return 0, [s, t]
    if filt == "cubic":
        return -1, [s ** 3 / 6, (4 + 3 * t * t * (t - 2)) / 6, (4 + 3 * s * s * (s - 2)) / 6, t ** 3 / 6]
    if filt == "keys":
        return -1, [-t * s * s / 2, s * (2 + t * (2 - 3 * t)) / 2, t * (2 + s * (2 - 3 * s)) / 2, -t * t * s / 2]
    return -1, [s * s * (1 - 7 * t) / 18, (1 + s * (9 + s * (27 - 21 * s))) / 18,
                (1 + t * (9 + t * (27 - 21 * t))) / 18, t * t * (1 - 7 * s) / 18]


def _chunks(n, size=1 << 20):
    return [(a, min(n, a + size)) for a in range(0, n, size)]


def _exact_grid(case, seed, stored, q, seed_run, filt, ids=None):
    dim, n = case["dim"], q.shape[0]
    vol = stored.to(F64)
    out = torch.empty(n, 1, dtype=F64, device=DEV)

    def at(x, y, z):
        ok = (x >= 0) & (x < dim) & (y >= 0) & (y < dim) & (z >= 0) & (z < dim)
        return vol[z.clamp(0, dim - 1), y.clamp(0, dim - 1), x.clamp(0, dim - 1)] * ok

    for a, b in _chunks(n):
        (cx, tx), (cy, ty), (cz, tz) = (_cells(q[a:b, k]) for k in range(3))
        if seed_run is not None:
            i = torch.arange(a, b, device=DEV) if ids is None else ids[a:b]
            v = at(cx + _choose(filt, tx, _uniform(seed_run, i, 0)), cy + _choose(filt, ty, _uniform(seed_run, i, 1)),
                   cz + _choose(filt, tz, _uniform(seed_run, i, 2)))
        else:
            o, wx = _weights(filt, tx)
            _, wy = _weights(filt, ty)
            _, wz = _weights(filt, tz)
            v = 0
            for k, c in enumerate(wz):
                for j, e in enumerate(wy):
                    row = sum(w * at(cx + o + m, cy + o + j, cz + o + k) for m, w in enumerate(wx))
                    v = v + c * e * row
        out[a:b, 0] = v
    return out


def _raster(uv, w, h):
    return _cells(uv[:, 0] * float(w) - 0.5), _cells(uv[:, 1] * float(h) - 0.5)


def _exact_2d(load, w, h, chans, filt, uv, seed_run):
    n = uv.shape[0]
    out = torch.empty(n, chans, dtype=F64, device=DEV)
    for a, b in _chunks(n):
        (cx, tx), (cy, ty) = _raster(uv[a:b], w, h)
        if seed_run is not None:
            i = torch.arange(a, b, device=DEV)
            out[a:b] = load((cx + _choose(filt, tx, _uniform(seed_run, i, 0))).clamp(0, w - 1),
                            (cy + _choose(filt, ty, _uniform(seed_run, i, 1))).clamp(0, h - 1))
        else:
            o, wx = _weights(filt, tx)
            _, wy = _weights(filt, ty)
            out[a:b] = _tensor_sum(load, w, h, cx + o, cy + o, wx, wy)
    return out


def _tensor_sum(load, w, h, x0, y0, wx, wy):
    v = 0
    for j, e in enumerate(wy):
        row = sum(c[:, None] * load((x0 + m).clamp(0, w - 1), (y0 + j).clamp(0, h - 1)) for m, c in enumerate(wx))
        v = v + e[:, None] * row
    return v


def _dct_load(words):
    def load(x, y):
        w = words[y >> 3, x >> 3]
        cx = [torch.cos((2 * (x & 7) + 1).to(F64) * k * math.pi / 16)[:, None] for k in (1, 2)]
        cy = [torch.cos((2 * (y & 7) + 1).to(F64) * k * math.pi / 16)[:, None] for k in (1, 2)]
        c = [(((w >> (7 + 5 * j)) & 31) - 16).to(F64) * (2 / 15) for j in range(5)]
        s = 1 / (4 * math.sqrt(2.0))
        return (w & 127).to(F64) / 127 + s * (c[0] * cx[0] + c[1] * cy[0] + c[2] * cy[1] + c[4] * cx[1]) \
            + 0.25 * c[3] * cx[0] * cy[0]
    return load


def _exact_gauss(case, load, uv, seed_run):
    n, s, sg, mode = uv.shape[0], case["size"], float(np.float32(case["sigma"])), case["mode"]
    out = torch.empty(n, case["channels"], dtype=F64, device=DEV)
    for a, b in _chunks(n, 1 << 19):
        (cx, tx), (cy, ty) = _raster(uv[a:b], s, s)
        i = torch.arange(a, b, device=DEV)
        tx, ty = tx.to(F64), ty.to(F64)
        if mode == "fis":
            u0, u1 = (_uniform(seed_run, i, k).to(F64) / 2 ** 24 for k in (0, 1))
            r = (-2 * torch.log(1 - u0)).sqrt() * sg
            x = (cx + tx + r * torch.cos(2 * math.pi * u1) + 0.5).floor().long()
            y = (cy + ty + r * torch.sin(2 * math.pi * u1) + 0.5).floor().long()
            out[a:b] = load(x.clamp(0, s - 1), y.clamp(0, s - 1))
            continue
        if mode == "fis_mean":
            rad = math.ceil(6 * np.float32(sg)) + 1
            offs = range(-rad, rad + 2)
            phi = lambda z: 0.5 * torch.erfc(-z / math.sqrt(2))
            ws = [[phi((k - t + 0.5) / sg) - phi((k - t - 0.5) / sg) for k in offs] for t in (tx, ty)]
            out[a:b] = _tensor_sum(load, s, s, cx - rad, cy - rad, ws[0], ws[1])
            continue
        ws = [[torch.exp(-((k - t) ** 2) / (2 * sg * sg)) for k in range(-1, 3)] for t in (tx, ty)]
        if mode == "discrete_mean":
            ws = [[v / sum(w) for v in w] for w in ws]
            out[a:b] = _tensor_sum(load, s, s, cx - 1, cy - 1, ws[0], ws[1])
            continue
        pick = []
        for k, w in enumerate(ws):
            T = _uniform(seed_run, i, k).to(F64) / 2 ** 24 * sum(w)
            pick.append(sum((T >= sum(w[:m])).long() for m in (1, 2, 3)) - 1)
        out[a:b] = load((cx + pick[0]).clamp(0, s - 1), (cy + pick[1]).clamp(0, s - 1))
    return out


def _ggx(alb, rough, nx, ny, wo, wi):
    n = torch.stack([nx, ny, (1 - nx * nx - ny * ny).clamp_min(0).sqrt()], 1)
    alpha = (rough * rough).clamp_min(1e-3)
    a2 = alpha * alpha
    dot = lambda u, v: (u * v).sum(1)
    cr2 = lambda u, v: torch.linalg.cross(u, v).square().sum(1)
    no, ni = dot(n, wo), dot(n, wi)
    h = wo + wi
    h = h / h.norm(dim=1, keepdim=True)
    nh = dot(n, h)
    D = a2 / (math.pi * (nh * nh * a2 + cr2(n, h)) ** 2)
    lam = lambda w, c: 0.5 * (-1 + (1 + a2 * cr2(n, w) / (c * c)).sqrt())
    f = 0.04 + 0.96 * (1 - dot(wi, h)) ** 5
    spec = D / (1 + lam(wo, no) + lam(wi, ni)) * f / (4 * no * ni)
    v = (alb / math.pi + spec[:, None]) * ni[:, None]
    return torch.where(((no > 0) & (ni > 0))[:, None], v, torch.zeros_like(v))


def _exact_shade(case, lv, q, seed_run):
    n, filt, mode = q.shape[0], case["filter"], case["mode"]
    out = torch.empty(n, 3, dtype=F64, device=DEV)
    sc = q[:, 2]
    level = (sc >= 1.41421354).long() + (sc >= 2.82842708).long()
    for l, (a, nrm) in enumerate(lv):
        s = a.shape[0]
        flat = torch.cat([a.to(F64) / 255, nrm.to(F64)], 2)
        sel = torch.nonzero(level == l)[:, 0]
        for x, y in _chunks(sel.shape[0]):
            ids = sel[x:y]
            r = q[ids]
            (cx, tx), (cy, ty) = _raster(r[:, :2], s, s)
            wo, wi = r[:, 3:6].to(F64), r[:, 6:9].to(F64)
            load = lambda i, j: flat[j, i]
            lit = lambda m: _ggx(m[:, :3], m[:, 3], m[:, 4], m[:, 5], wo, wi)
            if mode == "stochastic":
                out[ids] = lit(load((cx + _choose(filt, tx, _uniform(seed_run, ids, 0))).clamp(0, s - 1),
                                    (cy + _choose(filt, ty, _uniform(seed_run, ids, 1))).clamp(0, s - 1)))
                continue
            o, wx = _weights(filt, tx)
            _, wy = _weights(filt, ty)
            if mode == "shade_after_filter":
                out[ids] = lit(_tensor_sum(load, s, s, cx + o, cy + o, wx, wy))
            else:
                out[ids] = _tensor_sum(lambda i, j: lit(load(i, j)), s, s, cx + o, cy + o, wx, wy)
    return out


def _latent_at(lat, size, i, j):
    """Bilinear latents of texels (i, j) with their corners and weights."""
    L = lat.shape[0]
    r = L / size
    corners = []
    X, Y = (i.to(F64) + 0.5) * r - 0.5, (j.to(F64) + 0.5) * r - 0.5
    x0, y0 = X.floor(), Y.floor()
    fx, fy = X - x0, Y - y0
    z = 0
    for dy, wy in ((0, 1 - fy), (1, fy)):
        for dx, wx in ((0, 1 - fx), (1, fx)):
            k = (y0.long() + dy).clamp(0, L - 1) * L + (x0.long() + dx).clamp(0, L - 1)
            corners.append((k, wx * wy))
            z = z + (wx * wy)[:, None] * lat.view(-1, 8)[k]
    return z, corners


def _split_mlp(m):
    o = np.cumsum([0, 512, 64, 4096, 64, 512, 8])
    p = [m[o[k]:o[k + 1]] for k in range(6)]
    return p[0].view(64, 8), p[1], p[2].view(64, 64), p[3], p[4].view(8, 64), p[5]


def _exact_neural(case, lat, mlp, uv, seed_run):
    lat = lat.half().to(F64)   # the decoder's stored precision: binary16 latents, bfloat16 weights
    w1, b1, w2, b2, w3, b3 = _split_mlp(mlp)
    w1, w2, w3 = (w.bfloat16().to(F64) for w in (w1, w2, w3))
    b1, b2, b3 = (b.to(F64) for b in (b1, b2, b3))

    def load(x, y):
        z, _ = _latent_at(lat, case["size"], x, y)
        return torch.relu(torch.relu(z @ w1.T + b1) @ w2.T + b2) @ w3.T + b3

    s = case["size"]
    return _exact_2d(load, s, s, 8, case["filter"], uv, seed_run)


def _exact_train(case, seed):
    """The Adam steps in binary64 on the same batches."""
    lat, mlp = (t.to(F64) for t in _neural_inputs(case, seed))
    tgt, s, B = _target(case, seed).to(F64), case["size"], case["batch"]
    L = case["lat"]
    lat = lat.reshape(-1, 8).clone()
    mlp = mlp.clone()
    ml, vl, mm, vm = (torch.zeros_like(t) for t in (lat, lat, mlp, mlp))
    key, losses = _key(7), []
    ids = torch.arange(B, device=DEV)
    for step in range(1, case["steps"] + 1):
        ks = int(_pcg(torch.tensor(key ^ step)))
        h = _pcg(ids ^ ks)
        i, j = h % s, _pcg((h + 1) & M32) % s
        z, corners = _latent_at(lat.view(L, L, 8), s, i, j)
        w1, b1, w2, b2, w3, b3 = _split_mlp(mlp)
        h1 = torch.relu(z @ w1.T + b1)
        h2 = torch.relu(h1 @ w2.T + b2)
        e = h2 @ w3.T + b3 - tgt[j, i]
        losses.append((e * e).sum() / (8 * B))
        dy = e * (2 / (8 * B))
        d2 = (dy @ w3) * (h2 > 0)
        d1 = (d2 @ w2) * (h1 > 0)
        gm = torch.cat([(d1.T @ z).reshape(-1), d1.sum(0), (d2.T @ h1).reshape(-1), d2.sum(0),
                        (dy.T @ h2).reshape(-1), dy.sum(0)])
        dz = d1 @ w1
        gl = torch.zeros_like(lat)
        for k, w in corners:
            gl.index_add_(0, k, w[:, None] * dz)
        c1, c2 = 1 / (1 - 0.9 ** step), 1 / (1 - 0.999 ** step)
        for p, g, m, v, lr in ((mlp, gm, mm, vm, 1e-3), (lat, gl, ml, vl, 1e-2)):
            m.mul_(0.9).add_(0.1 * g)
            v.mul_(0.999).add_(0.001 * g * g)
            p -= lr * (m * c1) / ((v * c2).sqrt() + 1e-8)
    return torch.stack(losses), lat.view(L, L, 8).cpu().numpy(), mlp.cpu().numpy()


def exact(case, seed):
    kind, mode = case["kind"], case.get("mode")
    seed_run = 0x5EED + int(seed) * 7919 if mode == "stochastic" else None
    filt = case.get("filter")
    if mode == "stochastic" and filt in ("keys", "mitchell"):
        return None   # a signed pair of binary32 draws, defined by the library's own steps
    if kind in ("grid", "sorted"):
        stored, _, active = _grid_inputs(case, seed)
        v = _exact_grid(case, seed, stored, _grid_queries(case, seed, active), seed_run, filt)
        return (v, None) if kind == "sorted" else v
    if kind == "tex2d":
        t = _tex_inputs(case, seed)
        t = t.to(F64) / 255 if case["fmt"] == "u8" else t.to(F64)
        return _exact_2d(lambda x, y: t[y, x], case["width"], case["height"], case["channels"], filt,
                         _uv(case, seed), seed_run)
    if kind == "dct":
        return _exact_2d(_dct_load(_dct_inputs(case, seed)), case["size"], case["size"], case["channels"], filt,
                         _uv(case, seed), seed_run)
    if kind == "gauss":
        return _exact_gauss(case, _dct_load(_dct_inputs(case, seed)), _uv(case, seed), 0x5EED + int(seed) * 7919)
    if kind == "shade":
        return _exact_shade(case, _material_inputs(case, seed), _shade_queries(case, seed), seed_run)
    if kind == "neural":
        lat, mlp = _neural_inputs(case, seed)
        return _exact_neural(case, lat, mlp, _rand(_gen(seed, 12), case["n"], 2), seed_run)
    if kind == "train":
        return _exact_train(case, seed)
    if kind == "serve":
        stored, _, _ = _grid_inputs(case, seed)
        a, nrm = _material_inputs(case, seed)[0]
        flat = torch.cat([a.to(F64) / 255, nrm.to(F64)], 2)
        sizes, which, cubic, offs, totals = _requests(case)
        qs = _serve_queries(case, seed, totals)
        out = [torch.empty(totals[0], 1, dtype=F64, device=DEV), torch.empty(totals[1], 6, dtype=F64, device=DEV)]
        for k, (n, t, c, o) in enumerate(zip(sizes, which, cubic, offs)):
            q, f = qs[t][o:o + n], "cubic" if c else "linear"
            out[t][o:o + n] = _exact_grid(case, seed, stored, q, k, f) if t == 0 else \
                _exact_2d(lambda x, y: flat[y, x], case["size"], case["size"], 6, f, q, k)
        return out
    return None   # EWA: its tap weights are table entries picked by binary32 comparisons
