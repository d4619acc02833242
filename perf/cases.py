"""The work that a user of this framework has it do, as cases that can be timed.

Every case goes through the package's public classes (`GpuScene`, `Cache`,
`Octree`, `PrefetchRows`, `Mlp`, `Server`) as a viewer or a server does:

  frame     one frame of a bricked multi-channel volume (plain, LOD-adaptive,
            per-channel rates or render-and-skip), with the request readback
            where part of the volume is missing
  cold      the first frame of a slide of which nothing is resident yet: every
            visible brick is requested and the requests are read back
  stream    a frame's uploads into a full cache (LRU eviction, page tables,
            brick copies) and the residency update, optionally with the leaf
            metadata refined from the inserted bricks
  exchange  another data channel takes a cache channel's place at run time
  predict   one frame of the request predictor: history, features, logits,
            candidate bricks, labels
  train     the predictor's training steps of one frame
  serve     a batch of requests of several viewports and channel subsets

Volumes are cell-like tissue (ellipsoidal cells of lognormal intensity under a
low-frequency mask), made on the GPU from the seed; sizes are those of the
repository's configurations, tests and benchmark or lie between them.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2309_04393_amd import resoct
from paper_2309_04393_amd.pipeline import GpuScene

FLAGS = {"plain": 0, "adaptive": resoct.RENDER_ADAPTIVE_STEP,
         "rates": resoct.RENDER_ADAPTIVE_STEP | resoct.RENDER_CHANNEL_RATES,
         "homogeneous": resoct.RENDER_HOMOGENEOUS}
TERM = 0.99  # the renderer's default early-termination opacity


def listed():
    return [
        # A thumbnail of a small 8-bit volume (the smoke check's): a pass is launches and one ray's latency.
        dict(name="frame 64x64 1ch u8", kind="frame", dims="64x64x64", zs=1.0, m=1, bits=8, brick=16, levels=3,
             W=64, H=64, proj="ortho", view=70.0, tilt=35.0, tf="ramp", mode="plain", resident=1.0, mixed=False),
        # Interactive preview of a 4-channel tissue block, the whole block in view.
        dict(name="frame 512x512 4ch", kind="frame", dims="1024x1024x64", zs=4.0, m=4, bits=16, brick=32, levels=6,
             W=512, H=512, proj="persp", view=1100.0, tilt=50.0, tf="hue", mode="plain", resident=1.0, mixed=False),
        # The benchmark's view: 16 channels at full HD, about one voxel per pixel, everything resident.
        dict(name="frame 1080p 16ch", kind="frame", dims="1024x1024x192", zs=3.0, m=16, bits=16, brick=32, levels=6,
             W=1920, H=1080, proj="persp", view=580.0, tilt=30.0, tf="hue", mode="plain", resident=1.0, mixed=False),
        # While a view fills up: 60 % of the bricks resident, substitution, a ragged viewport, per-channel level
        # ranges, and the frame's requests read back.
        dict(name="frame 1001x563 6ch partly resident", kind="frame", dims="1000x900x60", zs=4.0, m=6, bits=16,
             brick=32, levels=6, W=1001, H=563, proj="persp", view=800.0, tilt=40.0, tf="hue", mode="plain",
             resident=0.6, mixed=True),
        # Whole-slide overview at 720p with the LOD-adaptive step.
        dict(name="frame 720p 8ch adaptive", kind="frame", dims="2048x2048x64", zs=4.0, m=8, bits=16, brick=32,
             levels=7, W=1280, H=720, proj="persp", view=2300.0, tilt=45.0, tf="hue", mode="adaptive", resident=1.0,
             mixed=False),
        # Opening a 16-channel whole-slide volume: nothing resident, 8.1 million miss counters read back.
        dict(name="cold 960x540 16ch slide", kind="cold", dims="8192x8192x192", zs=3.0, m=16, levels=9, W=960, H=540,
             view=6000.0, tilt=30.0),
        # A frame's uploads on the benchmark's cache (16 GiB), full from the start.
        dict(name="stream 2048 bricks 218551 slots", kind="stream", dims="8192x8192x192", zs=3.0, m=16, levels=9,
             slots=218551, U=2048, refine=False),
        # Streaming without a metadata server: few bricks, leaf metadata from their voxels.
        dict(name="stream 256 bricks refined", kind="stream", dims="2048x2048x64", zs=4.0, m=4, levels=7, slots=9000,
             U=256, refine=True),
        # The user swaps the stain shown in one of 16 channels of a slide.
        dict(name="exchange 16ch slide", kind="exchange", dims="8192x8192x192", zs=3.0, m=16, levels=9, slots=27318,
             U=512),
        # The prefetcher's share of a frame on the benchmark's 4-channel volume: 32,768 rows.
        dict(name="predict 32768 rows", kind="predict", dims="2048x2048x64", zs=4.0, m=4, levels=7, U=4096),
        # Its four training steps of a frame.
        dict(name="train 4x32768 rows", kind="train", rows=32768, steps=4),
        # A serving batch: mixed viewports, 3 to 16 of 16 channels.
        dict(name="serve 12 requests", kind="serve", dims="1024x1024x64", zs=4.0, m=16, levels=6, requests=12,
             small=256, large=640, mode="batch"),
    ]


def draw(rng):
    """One more case of the ranges above."""
    def logint(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["frame", "frame", "frame", "frame", "cold", "stream", "stream", "exchange", "predict", "train",
                       "serve"])
    if kind == "frame":
        m = rng.choice([1, 2, 3, 4, 5, 7, 8, 12, 16])
        small = rng.random() < 0.25
        if small:
            n = rng.choice([48, 64, 100, 128])
            c = dict(dims="%dx%dx%d" % (n, n, n), zs=1.0, bits=rng.choice([8, 16]), brick=16, levels=3,
                     W=logint(32, 400), H=logint(32, 400), view=n * rng.uniform(0.6, 1.3))
        else:
            x, y = rng.randint(400, 1024), rng.randint(400, 1024)
            c = dict(dims="%dx%dx%d" % (x, y, rng.randint(40, 96)), zs=rng.choice([2.0, 3.0, 4.0]),
                     bits=rng.choice([8, 16, 16, 16]), brick=rng.choice([16, 32, 32, 32, 64]), levels=5,
                     W=logint(200, 1920), H=logint(150, 1080), view=min(x, y) * rng.uniform(0.4, 1.3))
        mode = rng.choice(["plain", "plain", "plain", "adaptive", "rates", "homogeneous"])
        resident = rng.choice([1.0, 1.0, rng.uniform(0.2, 0.9)])
        return dict(kind=kind, m=m, proj=rng.choice(["persp", "persp", "ortho"]), tilt=rng.uniform(5.0, 60.0),
                    tf=rng.choice(["hue", "hue", "ramp"]), mode=mode, resident=resident,
                    mixed=rng.random() < 0.3, **c)
    if kind == "cold":
        n = logint(1000, 8192)
        return dict(kind=kind, dims="%dx%dx%d" % (n, n, rng.randint(40, 192)), zs=3.0, m=rng.choice([2, 4, 7, 16]),
                    levels=6, W=logint(160, 960), H=logint(120, 540), view=n * rng.uniform(0.3, 1.2),
                    tilt=rng.uniform(5.0, 60.0))
    if kind in ("stream", "exchange"):
        n = logint(1500, 8000)
        U = logint(16, 3000)
        c = dict(kind=kind, dims="%dx%dx%d" % (n, n, rng.randint(64, 192)), zs=3.0, m=rng.choice([3, 4, 8, 16]),
                 levels=6, slots=max(logint(6000, 100000), 2 * U), U=U)
        if kind == "stream":
            c["refine"] = rng.random() < 0.4
        return c
    if kind == "predict":
        n = logint(700, 4096)
        return dict(kind=kind, dims="%dx%dx%d" % (n, n, rng.randint(30, 130)), zs=4.0, m=rng.choice([1, 3, 4, 8]),
                    levels=rng.randint(4, 7), U=logint(200, 6000))
    if kind == "train":
        return dict(kind=kind, rows=logint(100, 100000), steps=rng.randint(1, 6))
    return dict(kind=kind, dims="%dx%dx%d" % (rng.randint(500, 1024), rng.randint(500, 1024), rng.randint(40, 64)),
                zs=4.0, m=rng.choice([4, 8, 16]), levels=5, requests=rng.randint(1, 16), small=logint(64, 200),
                large=logint(240, 640), mode=rng.choice(["batch", "graph", "continuous"]))


# ------------------------------------------------------------------ geometry

def _dims(case):
    return tuple(int(v) for v in case["dims"].split("x"))


class _Source:
    """What GpuScene asks of a data source (bricks come from device memory here)."""

    def __init__(self, dims, spacing, m, bits, n_levels):
        self.dims, self.spacing, self.n_channels, self.bits, self.n_levels = dims, spacing, m, bits, n_levels


def _leaf(brick, depth_z):
    return (8, 8, 8) if brick == 16 else (16, 16, 8 if depth_z > 64 else 4)


def _depth(dims, leaf):
    return max(max(0, (-(-dims[a] // leaf[a]) - 1).bit_length()) for a in range(3))


def _schedule(dims, spacing, n_levels):
    """Per level: its dims and L0 factors (an axis is halved iff its spacing is below twice the smallest)."""
    d, s, f = list(dims), list(spacing), [1, 1, 1]
    out = [(tuple(d), tuple(f))]
    for _ in range(1, n_levels):
        mn = min(s)
        h = [s[a] < 2 * mn for a in range(3)]
        for a in range(3):
            if h[a]:
                d[a], s[a], f[a] = (d[a] + 1) // 2, s[a] * 2, f[a] * 2
        out.append((tuple(d), tuple(f)))
    return out


def _norm(v):
    v = np.asarray(v, np.float64)
    return v / math.sqrt(float(v @ v))


def _camera(dims, spacing, view, tilt, proj, aspect, rng):
    """Looks at a point near the middle from above, tilted; `view` world units fill the height there."""
    ext = np.asarray(dims, np.float64) * np.asarray(spacing, np.float64)
    target = ext * (0.5 + rng.uniform(-0.04, 0.04, 3))
    az, ti = rng.uniform(0, 2 * math.pi), math.radians(tilt)
    back = np.array([math.sin(ti) * math.cos(az), math.sin(ti) * math.sin(az), math.cos(ti)])
    F = _norm(-back)
    R = _norm(np.cross(F, [-math.sin(az), math.cos(az), 0.1]))
    U = np.cross(R, F)
    if proj == "ortho":
        eye = target + back * (float(np.linalg.norm(ext)) / 2 + 1.0)
        tx, ty = view / 2 * aspect, view / 2
    else:
        ty = math.tan(math.radians(22.5))
        eye, tx = target + back * (view / (2 * ty)), aspect * ty
    return dict(proj=proj, eye=[float(x) for x in eye], F=[float(x) for x in F], R=[float(x) for x in R],
                U=[float(x) for x in U], tx=float(tx), ty=float(ty))


def _channels(case, m, n_levels, bits, rng, vis=None):
    """Window and table of each visible channel: the hue tables of the benchmark or a grey ramp."""
    out = []
    x = np.arange(256) / 255.0
    top = 255.0 if bits == 8 else 8000.0
    for j, c in enumerate(range(m) if vis is None else vis):
        w = rng.uniform(0.8, 1.2, 2)
        tf = np.zeros((256, 4), np.float32)
        if case.get("tf") == "ramp":
            tf[:] = (x * (1.0 if m == 1 else 0.3))[:, None]
        else:
            h = (c / max(m, 1)) * 6.0
            k, f = int(h) % 6, h - int(h)
            tf[:, :3] = [(1, f, 0), (1 - f, 1, 0), (0, 1, f), (0, 1 - f, 1), (f, 0, 1), (1, 0, 1 - f)][k]
            tf[:, 3] = 0.1 * x
        if case.get("mode") == "homogeneous" and c % 2 == 0:
            tf[:9] = tf[8]
            tf[:9, 3] = 0.05
        lo = min(2 * (c % 3), n_levels - 1) if case.get("mixed") else 0
        out.append(dict(c=c, lo=lo, hi=n_levels - 1, W0=int(round(top * 0.0375 * w[0] * 256)),
                        W1=int(round(top * w[1] * 256)) if bits == 16 else 255 * 256, tf=tf))
    return out


# -------------------------------------------------------------------- volumes

def _cells(dims, m, bits, seed):
    """[m][z][y][x] int16 (bits of uint16) or uint8 voxels: Poisson cells under a tissue mask."""
    nx, ny, nz = dims
    g = torch.Generator(device="cuda").manual_seed(seed)

    def rand(*shape):
        return torch.rand(*shape, generator=g, device="cuda")

    n = max(8, int(2e-4 * nx * ny * nz * (4.0 if nx <= 128 else 1.0)))
    n = min(n, 65000)
    pos = rand(n, 3) * torch.tensor([nx, ny, nz], device="cuda", dtype=torch.float32)
    rad = 4.0 + 6.0 * rand(n, 3)
    # low-frequency mask: cells outside the tissue are dropped
    mask = rand(1, 1, max(2, ny // 200 + 2), max(2, nx // 200 + 2))
    mask = torch.nn.functional.interpolate(mask, size=(ny, nx), mode="bilinear", align_corners=True)[0, 0]
    keep = mask[pos[:, 1].long().clamp(max=ny - 1), pos[:, 0].long().clamp(max=nx - 1)] > 0.42
    pos, rad = pos[keep], rad[keep]
    n = pos.shape[0]
    inten = torch.exp(7.0 + torch.randn(m, n + 1, generator=g, device="cuda"))
    gain = 0.3 + 0.7 * rand(m, n + 1)
    inten = (inten * gain).clamp(max=65535.0)
    if bits == 8:
        inten = (inten / 16.0).clamp(max=255.0)
    # key = weight << 16 | cell, the strongest cell of each voxel
    key = torch.zeros(nz * ny * nx, dtype=torch.int32, device="cuda")
    o = torch.arange(-10, 11, device="cuda")
    for s in range(0, n, 4096):
        p, r = pos[s:s + 4096], rad[s:s + 4096]
        q = p.floor().long()
        ax = [q[:, a, None] + o for a in range(3)]
        w = [((ax[a] + 0.5 - p[:, a, None]) / r[:, a, None]) ** 2 for a in range(3)]
        ok = [(ax[a] >= 0) & (ax[a] < dims[a]) for a in range(3)]
        d2 = w[2][:, :, None, None] + w[1][:, None, :, None] + w[0][:, None, None, :]
        ins = (d2 < 1.0) & ok[2][:, :, None, None] & ok[1][:, None, :, None] & ok[0][:, None, None, :]
        lin = (ax[2][:, :, None, None] * ny + ax[1][:, None, :, None]) * nx + ax[0][:, None, None, :]
        wq = (torch.exp(-2.0 * d2) * 32767.0).to(torch.int32)
        cell = torch.arange(s + 1, s + 1 + p.shape[0], device="cuda", dtype=torch.int32)[:, None, None, None]
        key.scatter_reduce_(0, lin[ins], ((wq << 16) | cell)[ins], "amax")
    wt, cell = (key >> 16).float() / 32767.0, (key & 0xFFFF).long()
    del key
    out = torch.empty((m, nz, ny, nx), dtype=torch.uint8 if bits == 8 else torch.int16, device="cuda")
    for c in range(m):
        v = (inten[c][cell] * wt + 0.5).to(torch.int32)
        out[c] = v.view(nz, ny, nx).to(out.dtype)
    return out


def _raw(t):
    """Voxel values as int32."""
    return t.to(torch.int32) & (0xFF if t.dtype == torch.uint8 else 0xFFFF)


def _pyramid(l0, dims, spacing, n_levels):
    """Level arrays by the box filter (an odd edge counts twice), rounded half up."""
    out, sch = [l0], _schedule(dims, spacing, n_levels)
    for l in range(1, n_levels):
        per = []
        for c in range(l0.shape[0]):
            a = _raw(out[-1][c])
            n = 1
            for ax, k in ((0, 2), (1, 1), (2, 0)):
                if sch[l][1][k] != sch[l - 1][1][k]:
                    if a.shape[ax] % 2:
                        a = torch.cat([a, a.narrow(ax, a.shape[ax] - 1, 1)], ax)
                    sl = [slice(None)] * 3
                    sl[ax] = slice(0, None, 2)
                    sm = list(sl)
                    sm[ax] = slice(1, None, 2)
                    a = a[tuple(sl)] + a[tuple(sm)]
                    n *= 2
            per.append(torch.div(a + n // 2, n, rounding_mode="floor").to(l0.dtype))
        out.append(torch.stack(per))
    return out


def _leaf_range(l0c, leaf, grid):
    """[n_leaves][2] (min, max) of one channel over each leaf box grown by one voxel, int32."""
    f = _raw(l0c).float()[None, None]
    k = (leaf[2] + 2, leaf[1] + 2, leaf[0] + 2)
    s = (leaf[2], leaf[1], leaf[0])
    pad = []
    for a in (0, 1, 2):  # x, y, z: one voxel before, up to the padded grid plus one after
        pad += [1, grid[a] * leaf[a] + 1 - f.shape[4 - a]]

    def pool(v):
        v = torch.nn.functional.pad(v, pad, value=-1e9)
        return torch.nn.functional.max_pool3d(v, k, s)[0, 0]

    hi, lo = pool(f), -pool(-f)
    void = hi < 0
    return torch.stack([lo.masked_fill(void, 0), hi.masked_fill(void, 0)], -1).to(torch.int32).reshape(-1, 2)


def _u16(t):
    return t.to(torch.int16).contiguous().view(-1).view(torch.uint16)


def _brick_ids(nb, c, l, n_levels):
    """IDs of every brick of a channel's level in z, y, x order."""
    nx, ny, nz = (int(v) for v in nb[l])
    z, y, x = np.meshgrid(np.arange(nz), np.arange(ny), np.arange(nx), indexing="ij")
    return (((c * n_levels + l) << 24) | (z << 16) | (y << 8) | x).astype(np.uint32).reshape(-1)


def _bricks(arr, nb, B):
    """[n][(B + 2)^3] halo bricks of one channel's level array, in z, y, x order."""
    for a, d in ((0, 2), (1, 1), (2, 0)):
        n = arr.shape[a]
        idx = torch.arange(-1, int(nb[d]) * B + 1, device=arr.device).clamp(0, n - 1)
        arr = arr.index_select(a, idx)
    w = arr.unfold(0, B + 2, B).unfold(1, B + 2, B).unfold(2, B + 2, B)
    return w.reshape(-1, (B + 2) ** 3)


def _volume_scene(case, seed, bits=16):
    """A scene with its voxels: (scene, per-level arrays, residency [m][level] bool, leaf ranges [m])."""
    dims, m, L, B = _dims(case), case["m"], case["levels"], case.get("brick", 32)
    spacing = (1.0, 1.0, float(case["zs"]))
    leaf = _leaf(B, dims[2])
    levels = _pyramid(_cells(dims, m, bits, seed), dims, spacing, L)
    gen = np.random.default_rng(seed + 1)
    nb = [[-(-d // B) for d in s[0]] for s in _schedule(dims, spacing, L)]
    frac = case.get("resident", 1.0)
    res = [[(gen.random(nb[l][0] * nb[l][1] * nb[l][2]) < frac) | (l == L - 1) for l in range(L)] for _ in range(m)]
    return levels, res, leaf, spacing, nb


def _upload(scene, levels, res, nb, B):
    cache = scene.cache
    L, m = len(levels), levels[0].shape[0]
    words = cache.slot_stride // (1 if levels[0].dtype == torch.uint8 else 2)
    for c in range(m):
        for l in range(L):
            pick = np.nonzero(res[c][l])[0]
            ids = _brick_ids(nb, c, l, L)[pick]
            br = _bricks(levels[l][c], nb[l], B)
            for s in range(0, len(ids), cache.max_batch):
                part = ids[s:s + cache.max_batch]
                staged = torch.zeros((len(part), words), dtype=br.dtype, device="cuda")
                at = torch.from_numpy(pick[s:s + len(part)]).cuda()
                staged[:, :br.shape[1]] = br.index_select(0, at)
                cache.stream_bricks(0, part, staged.view(-1).view(torch.uint8))
    scene.tree.update_residency()


def _frame_scene(case, seed):
    bits = case.get("bits", 16)
    dims, m, L, B = _dims(case), case["m"], case["levels"], case.get("brick", 32)
    levels, res, leaf, spacing, nb = _volume_scene(case, seed, bits)
    n = sum(r.size for per in res for r in per)
    scene = GpuScene(_Source(dims, spacing, m, bits, L), B, leaf, _depth(dims, leaf), n, max_batch=2048,
                     start_level=min(2, _depth(dims, leaf)), set_metadata=False)
    for c in range(m):
        scene.tree.set_leaf_metadata(c, _u16(_leaf_range(levels[0][c], leaf, scene.tree.leaf_grid)))
    _upload(scene, levels, res, nb, B)
    return scene


def _slide_scene(case, seed, slots, max_batch, known=True):
    """A scene without voxels: tissue-like leaf metadata only."""
    dims, m, L = _dims(case), case["m"], case["levels"]
    spacing = (1.0, 1.0, float(case["zs"]))
    leaf = _leaf(32, dims[2])
    scene = GpuScene(_Source(dims, spacing, m, 16, L), 32, leaf, _depth(dims, leaf), slots, max_batch=max_batch,
                     start_level=min(2, _depth(dims, leaf)), set_metadata=False)
    if known:
        for c in range(m):
            scene.tree.set_leaf_metadata(c, _u16(_slide_ranges(scene.tree.leaf_grid, seed, c)))
    else:
        for c in range(m):
            scene.set_unknown(c)
    return scene


def _slide_ranges(grid, seed, c):
    """Leaf ranges of one channel: cells in tissue, about half of the leaves empty."""
    g = torch.Generator(device="cuda").manual_seed(seed)  # one tissue for all channels
    nx, ny, nz = grid
    t = torch.rand(1, 1, max(2, ny // 40 + 2), max(2, nx // 40 + 2), generator=g, device="cuda")
    t = torch.nn.functional.interpolate(t, size=(ny, nx), mode="bilinear", align_corners=True)[0, 0]
    g.manual_seed(seed * 31 + c + 1)
    v = torch.exp(7.0 + torch.randn(nz, ny, nx, generator=g, device="cuda")).clamp(max=65535.0)
    v = torch.where(t[None] > 0.48, v, torch.zeros_like(v)).to(torch.int32)
    return torch.stack([torch.zeros_like(v), v], -1).reshape(-1, 2)


# -------------------------------------------------------------------- prepare

def prepare(case, seed):
    return globals()["_prepare_" + case["kind"]](case, seed)


def _view(case, seed, m=None, n_levels=None, bits=16):
    rng = np.random.default_rng(seed + 2)
    cam = _camera(_dims(case), (1.0, 1.0, float(case["zs"])), case["view"], case["tilt"], case.get("proj", "persp"),
                  case["W"] / case["H"], rng)
    return cam, _channels(case, case["m"], case["levels"], bits, rng)


def _pairs(cap, dtype=np.int64):
    """Host arrays that take up to cap (ID, value) pairs of a readback."""
    return dict(cap=cap, ids=np.zeros(cap, np.int64), val=np.zeros(cap, dtype), last=0)


def _keep(s, ids, val):
    n = len(ids)
    s["ids"][:n], s["val"][:n] = ids, val
    s["ids"][n:s["last"]], s["val"][n:s["last"]] = 0, 0
    s["last"] = n
    return dict(ids=s["ids"], val=s["val"], n=n)


def _prepare_frame(case, seed):
    scene = _frame_scene(case, seed)
    cam, chans = _view(case, seed, bits=case["bits"])
    out = torch.empty(case["W"] * case["H"] * 4, dtype=torch.float32, device="cuda")
    return dict(kind="frame", scene=scene, cam=cam, chans=chans, tf=scene.tf_tensor(chans), out=out, W=case["W"],
                H=case["H"], flags=FLAGS[case["mode"]], f=0, **_pairs(1 << 16 if case["resident"] < 1.0 else 0))


def _prepare_cold(case, seed):
    scene = _slide_scene(case, seed, 64, 64)
    cam, chans = _view(case, seed)
    out = torch.empty(case["W"] * case["H"] * 4, dtype=torch.float32, device="cuda")
    return dict(kind="frame", scene=scene, cam=cam, chans=chans, tf=scene.tf_tensor(chans), out=out, W=case["W"],
                H=case["H"], flags=0, f=0, **_pairs(1 << 19))


def _cycle(scene, m, L, count, rng):
    """Brick IDs in upload order: every channel of a brick position together, levels mixed, positions in runs."""
    nb = scene.nb
    rows = []
    for l in range(L):
        per = np.stack([_brick_ids(nb, c, l, L) for c in range(m)], 1)
        rows.append(per)
    # runs of 16 consecutive positions, shuffled over the levels
    runs = [r[i:i + 16].reshape(-1) for r in rows for i in range(0, min(len(r), -(-2 * count // m)), 16)]
    order = rng.permutation(len(runs))
    return np.concatenate([runs[i] for i in order])


def _prepare_stream(case, seed):
    rng = np.random.default_rng(seed)
    U, slots = case["U"], case["slots"]
    scene = _slide_scene(case, seed, slots, max(U, min(8192, slots)), known=not case["refine"])
    ids = _cycle(scene, case["m"], case["levels"], 2 * slots + 4 * U, rng)
    g = torch.Generator(device="cuda").manual_seed(seed)
    n = max(U, min(8192, slots))
    staged = torch.randint(0, 256, (n * scene.cache.slot_stride,), generator=g, dtype=torch.uint8, device="cuda")
    # a cache much smaller than the volume, full from earlier frames
    at = 0
    while at < min(slots, len(ids)):
        part = ids[at:at + min(n, slots - at)]
        scene.cache.stream_bricks(1 + at // n, part, staged)
        at += len(part)
    scene.tree.update_residency()
    return dict(kind="stream", scene=scene, ids=ids, at=at, U=U, staged=staged, refine=case["refine"], f=1 + at)


def _prepare_exchange(case, seed):
    rng = np.random.default_rng(seed)
    U, slots, m = case["U"], case["slots"], case["m"]
    scene = _slide_scene(case, seed, slots, max(U, min(8192, slots)))
    ids = _cycle(scene, m, case["levels"], slots, rng)[:slots]
    n = max(U, min(8192, slots))
    staged = torch.randint(0, 256, (n * scene.cache.slot_stride,), dtype=torch.uint8, device="cuda",
                           generator=torch.Generator(device="cuda").manual_seed(seed))
    for s in range(0, len(ids), n):
        scene.cache.stream_bricks(1, ids[s:s + n], staged)
    scene.tree.update_residency()
    own = [ids[(ids >> 24) // case["levels"] == c][:U] for c in range(m)]
    ranges = [_u16(_slide_ranges(scene.tree.leaf_grid, seed + 77, c)) for c in range(2)]
    return dict(kind="exchange", scene=scene, own=own, ranges=ranges, staged=staged, f=1)


def _predict_ids(case, seed, scene):
    rng = np.random.default_rng(seed)
    return _cycle(scene, case["m"], case["levels"], case["U"], rng)[:case["U"]]


def _prepare_predict(case, seed):
    scene = _slide_scene(case, seed, case["U"], case["U"])
    ids = _predict_ids(case, seed, scene)
    staged = torch.zeros(len(ids) * scene.cache.slot_stride, dtype=torch.uint8, device="cuda")
    pf = resoct.PrefetchRows(scene.tree)
    scene.cache.stream_bricks(1, ids, staged)
    scene.tree.update_residency()
    pf.record(1)
    cam, chans = _view(dict(case, W=1024, H=1024, view=_predict_view(case), tilt=40.0), seed)
    tf = scene.tf_tensor(chans)
    fd = resoct.frame_desc(2, cam, 1024, 1024, 0.5, chans, tf, case["levels"])
    net = resoct.Mlp()
    net.set_weights(_weights(seed))
    R = pf.rows
    return dict(kind="predict", scene=scene, pf=pf, fd=fd, tf=tf, net=net,
                x=torch.zeros((R, 32), dtype=torch.float16, device="cuda"),
                z=torch.zeros((R, 16), dtype=torch.float32, device="cuda"),
                y=torch.zeros((R, 16), dtype=torch.uint8, device="cuda"),
                m=torch.zeros((R, 16), dtype=torch.uint8, device="cuda"), f=1, **_pairs(1 << 16, np.float32))


def _predict_view(case):
    return 0.5 * _dims(case)[1]


def _weights(seed):
    """He-uniform initial weights, a smaller output layer."""
    rng = np.random.default_rng(seed + 3)
    p, sizes = {}, (24, 64, 64, 9)
    for i in range(3):
        lim = math.sqrt(6.0 / sizes[i]) * (0.25 if i == 2 else 1.0)
        p["W%d" % (i + 1)] = rng.uniform(-lim, lim, (sizes[i], sizes[i + 1])).astype(np.float32)
        p["b%d" % (i + 1)] = rng.uniform(-0.05, 0.05, sizes[i + 1]).astype(np.float32)
    return p


def _train_data(case, seed):
    """Rows as the feature kernel gives them: a few continuous columns, history and residency bits."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    R = case["rows"]
    x = torch.zeros((R, 32), device="cuda")
    x[:, :8] = torch.rand(R, 8, generator=g, device="cuda") * 2 - 1
    x[:, 8:24] = (torch.rand(R, 16, generator=g, device="cuda") < 0.3).float()
    p = torch.sigmoid(3 * x[:, :1] + 2 * x[:, 8:9] - 2 + 0.5 * torch.arange(9, device="cuda") / 9)
    y = torch.zeros((R, 16), dtype=torch.uint8, device="cuda")
    y[:, :9] = (torch.rand(R, 9, generator=g, device="cuda") < p).to(torch.uint8)
    mask = torch.zeros((R, 16), dtype=torch.uint8, device="cuda")
    mask[:, :7] = 1
    return x.half(), y, mask


def _prepare_train(case, seed):
    x, y, mask = _train_data(case, seed)
    net = resoct.Mlp()
    net.set_weights(_weights(seed))
    return dict(kind="train", net=net, x=x, y=y, m=mask, steps=case["steps"])


def _prepare_serve(case, seed):
    scene = _frame_scene(case, seed)
    rng = np.random.default_rng(seed + 4)
    fds, outs, keep = [], [], []
    dims, m = _dims(case), case["m"]
    for r in range(case["requests"]):
        e = r / max(case["requests"] - 1, 1)
        H = int(round(case["small"] * (case["large"] / case["small"]) ** e))
        W = H if r % 2 else (H * 16) // 9
        k = int(rng.integers(min(3, m), m + 1))
        vis = sorted(int(v) for v in rng.permutation(m)[:k]) if r % 3 else list(range(m))
        cam = _camera(dims, (1.0, 1.0, float(case["zs"])), dims[1] * rng.uniform(0.3, 1.1), rng.uniform(20, 55),
                      "persp", W / H, rng)
        chans = _channels(case, m, case["levels"], 16, rng, vis)
        tf = scene.tf_tensor(chans)
        out = torch.empty(W * H * 4, dtype=torch.float32, device="cuda")
        fds.append(resoct.frame_desc(1 + r, cam, W, H, 0.5, chans, tf, case["levels"]))
        outs.append(out)
        keep.append(tf)
    torch.cuda.synchronize()  # the server has streams of its own
    return dict(kind="serve", scene=scene, server=resoct.Server(scene.tree), fds=fds, outs=outs, tfs=keep,
                mode=case["mode"])


# ------------------------------------------------------------------------ run

def run(state):
    return globals()["_run_" + state["kind"]](state)


def _words(t, n, dtype=torch.int32):
    return t[:n * dtype.itemsize].view(dtype)


def _run_frame(s):
    scene = s["scene"]
    s["f"] += 1
    scene.render(s["f"], s["cam"], s["W"], s["H"], 0.5, s["chans"], tf_dev=s["tf"], out=s["out"], flags=s["flags"])
    res = dict(rgba=s["out"].view(s["H"], s["W"], 4), stamps=_words(scene.cache.t["stamps"], scene.cache.n_slots))
    if s["cap"]:
        ids, cnt, distinct, total = scene.cache.read_requests(s["cap"])
        res.update(_keep(s, ids, cnt), distinct=distinct, total=total)
    return res


def _run_stream(s):
    scene, U = s["scene"], s["U"]
    s["f"] += 1
    at = s["at"]
    if at + U > len(s["ids"]):
        at = 0
    ids = s["ids"][at:at + U]
    s["at"] = at + U
    flags = scene.cache.stream_bricks(s["f"], ids, s["staged"])
    if s["refine"]:
        scene.tree.leaf_metadata_from_bricks(ids[flags == 1])
    scene.tree.update_residency()
    tree, m = scene.tree, scene.vol.n_channels
    res = dict(flags=flags, page_table=_words(scene.cache.t["page_table"], scene.cache.n_bricks),
               seqs=_words(scene.cache.t["seqs"], scene.cache.n_slots),
               mask=_words(tree.t["node_mask"], tree.n_nodes * m, torch.int16))
    if s["refine"]:
        res["meta"] = _words(tree.t["node_meta"], tree.n_nodes * m)
    return res


def _run_exchange(s):
    scene = s["scene"]
    s["f"] += 1
    c = s["f"] % scene.vol.n_channels
    scene.cache.evict_channel(c)
    scene.tree.set_leaf_metadata(c, s["ranges"][s["f"] % 2])
    flags = scene.cache.stream_bricks(s["f"], s["own"][c], s["staged"])
    scene.tree.update_residency()
    tree, m = scene.tree, scene.vol.n_channels
    return dict(flags=flags, page_table=_words(scene.cache.t["page_table"], scene.cache.n_bricks),
                mask=_words(tree.t["node_mask"], tree.n_nodes * m, torch.int16),
                meta=_words(tree.t["node_meta"], tree.n_nodes * m))


def _run_predict(s):
    s["f"] += 1
    pf = s["pf"]
    pf.record(s["f"])
    pf.features(s["fd"], s["x"])
    pf.labels(s["y"], s["m"])
    s["net"].forward(s["x"], s["z"])
    ids, prob = pf.candidates(s["z"], 0.5)
    return dict(x=s["x"], z=s["z"], y=s["y"], m=s["m"], **_keep(s, ids, prob))


def _run_train(s):
    for _ in range(s["steps"]):
        s["net"].train_step(s["x"], s["y"], s["m"], 3e-3)
    return s["net"].get_weights()


def _run_serve(s):
    server = s["server"]
    if s["mode"] == "continuous":
        for fd, out in zip(s["fds"], s["outs"]):
            server.enqueue(fd, out)
        server.drain()
    else:
        server.wait(server.launch(s["fds"], s["outs"], graph=s["mode"] == "graph"))
    return s["outs"]


# ----------------------------------------------------------------------- work

def work(case):
    k = case["kind"]
    if k == "train":
        # rows, labels and masks in, weights and moments in and out; three products of each layer a row
        return dict(bytes=case["steps"] * (case["rows"] * 96 + 6 * 4 * 6217),
                    flops=case["steps"] * case["rows"] * 6 * 6208)
    dims = _dims(case)
    spacing = (1.0, 1.0, float(case["zs"]))
    sch = _schedule(dims, spacing, case["levels"])
    B, m = case.get("brick", 32), case["m"]
    nb = [int(np.prod([-(-d // B) for d in s[0]])) for s in sch]
    brick = (B + 2) ** 3 * (1 if case.get("bits", 16) == 8 else 2)
    leaf = _leaf(B, dims[2])
    leaves = int(np.prod([-(-dims[a] // leaf[a]) for a in range(3)]))
    if k == "predict":
        rows = nb[0] * m
        # node ranges, page-table words, history in; features, logits, labels, masks out
        return dict(bytes=rows * (64 + 36 + 32) + leaves * m * 4 + sum(nb) * m * 6, flops=rows * 2 * 6208)
    if k == "stream":
        return dict(bytes=case["U"] * brick * (3 if case["refine"] else 2) + case["slots"] * 12, flops=0)
    if k == "exchange":
        # the bricks, the channel's leaf ranges, node ranges and levels, its page-table words
        return dict(bytes=case["U"] * brick * 2 + leaves * 10 + case["slots"] * 4, flops=0)
    if k == "cold":
        # the leaves' ranges in view, every counter read, the image
        return dict(bytes=leaves * m * 4 + sum(nb) * m * 4 + case["W"] * case["H"] * 16, flops=0)
    if k == "serve":
        px = 0
        for r in range(case["requests"]):
            H = case["small"] * (case["large"] / case["small"]) ** (r / max(case["requests"] - 1, 1))
            px += H * H * (1 if r % 2 else 16 / 9)
        view, cov = 0.7 * dims[1], 0.6
    else:
        px = case["W"] * case["H"]
        view = case["view"]
        cov = min(1.0, view * view * case["W"] / case["H"] / (dims[0] * dims[1]))
    # bricks in view at the level of one voxel a pixel, each read once; half of a ray's samples lie in tissue
    pix = view / max(px ** 0.5, 1.0)
    l = min(max(0, int(math.log2(max(pix, 1.0)))), case["levels"] - 1)
    reads = px * dims[2] * spacing[2] / 0.5 * 0.5 * m / (1 << l if case["mode"] in ("adaptive", "rates") else 1)
    return dict(bytes=nb[l] * m * brick * 0.5 * cov + px * 16, flops=34 * reads)


# ---------------------------------------------------------------------- exact

def exact(case, seed):
    """64-bit values by plain torch; None where there are none or they would take too long."""
    f = globals().get("_exact_" + case["kind"])
    return f(case, seed) if f else None


def _exact_train(case, seed):
    x, y, mask = _train_data(case, seed)
    x, y, mask = x[:, :24].double(), y[:, :9].double(), mask[:, :9].double()
    w = {k: torch.from_numpy(v).double().cuda().requires_grad_() for k, v in _weights(seed).items()}
    mom = {k: (torch.zeros_like(v), torch.zeros_like(v)) for k, v in w.items()}
    for t in range(1, case["steps"] + 1):
        z = _net(w, x)
        loss = (torch.nn.functional.binary_cross_entropy_with_logits(z, y, reduction="none") * mask).sum() / mask.sum()
        grads = torch.autograd.grad(loss, list(w.values()))
        with torch.no_grad():
            for (k, v), g in zip(w.items(), grads):
                a, b = mom[k]
                a.mul_(0.9).add_(0.1 * g)
                b.mul_(0.999).add_(0.001 * g * g)
                v -= 3e-3 * (a / (1 - 0.9 ** t)) / ((b / (1 - 0.999 ** t)).sqrt() + 1e-8)
    return {k: v.detach() for k, v in w.items()}


def _net(w, x):
    h = torch.relu(x @ w["W1"] + w["b1"])
    h = torch.relu(h @ w["W2"] + w["b2"])
    return h @ w["W3"] + w["b3"]


def _empty(ranges, ch):
    """Whether the channel's table is zero over every entry reachable from each [min, max] (exact integers)."""
    den = ch["W1"] - ch["W0"]
    zero = torch.cat([torch.zeros(1, dtype=torch.int64), torch.cumsum(torch.from_numpy(ch["tf"][:, 3] != 0).long(), 0)])
    zero = zero.cuda()
    r = ranges.long()
    lo = torch.div(255 * (256 * r[:, 0] - ch["W0"]), den, rounding_mode="floor").clamp(0, 255)
    hi = (-torch.div(-255 * (256 * r[:, 1] - ch["W0"]), den, rounding_mode="floor")).clamp(0, 255)
    return zero[hi + 1] == zero[lo]


def _exact_predict(case, seed):
    """Features and logits (their integer outputs are compared as they are)."""
    dims, m, L = _dims(case), case["m"], case["levels"]
    sp = np.array([1.0, 1.0, float(case["zs"])])
    scene = _slide_scene(case, seed, 64, 64)
    ids = _predict_ids(case, seed, scene)
    cam, chans = _view(dict(case, W=1024, H=1024, view=_predict_view(case), tilt=40.0), seed)
    sch = _schedule(dims, sp, L)
    nb = [[-(-d // 32) for d in s[0]] for s in sch]
    nx, ny, nz = nb[0]
    P = nx * ny * nz
    z, y, x = np.meshgrid(np.arange(nz), np.arange(ny), np.arange(nx), indexing="ij")
    pos = np.stack([x, y, z], -1).reshape(-1, 3)
    q = (pos + 0.5) * 32.0 * sp
    v = q - np.array(cam["eye"])
    zf, xr, yu = v @ np.array(cam["F"]), v @ np.array(cam["R"]), v @ np.array(cam["U"])
    t = np.maximum(np.sqrt((v * v).sum(1)), 1e-6)
    zz = np.maximum(zf, 1e-6)
    sx, sy = xr / (zz * cam["tx"]), yu / (zz * cam["ty"])
    pix = 2.0 * cam["ty"] / 1024
    D = [s[1][0] / pix for s in sch]
    f = np.zeros((m, P, 32))
    f[:, :, 0] = np.clip(np.log2(32.0 / (t * pix)), -8, 8) / 8
    f[:, :, 1] = np.clip(np.log2(t / D[1]), -8, 8) / 8 if L > 1 else 0
    f[:, :, 2] = sum((t >= D[l]).astype(float) for l in range(1, L)) / 8
    f[:, :, 3] = (zf > 0) & (np.abs(sx) <= 1) & (np.abs(sy) <= 1)
    f[:, :, 4], f[:, :, 5] = np.clip(sx, -2, 2) / 2, np.clip(sy, -2, 2) / 2
    f[:, :, 6] = (pos[:, 2] + 0.5) / nz
    leaf = _leaf(32, dims[2])
    k = [32 // leaf[a] for a in range(3)]
    g = scene.tree.leaf_grid
    for c in range(m):
        e = ~_empty(_slide_ranges(g, seed, c), chans[c]).view(g[2], g[1], g[0])
        # leaves of a brick past the padded grid do not exist: only whole bricks are used here
        pad = [0, nx * k[0] - g[0], 0, ny * k[1] - g[1], 0, nz * k[2] - g[2]]
        if min(pad) < 0:
            e = e[:nz * k[2], :ny * k[1], :nx * k[0]]
            pad = [0, nx * k[0] - e.shape[2], 0, ny * k[1] - e.shape[1], 0, nz * k[2] - e.shape[0]]
        if max(pad) > 0:
            return None
        e = e.reshape(nz, k[2], ny, k[1], nx, k[0]).double().mean((1, 3, 5))
        f[c, :, 7] = e.reshape(-1).cpu().numpy()
    has = np.isin
    for c in range(m):
        f[c, :, 13] = has(_brick_ids(nb, c, 0, L), ids)  # read one frame before
        for l in range(min(L, 8)):
            b = pos // np.array(sch[l][1])
            b_id = ((c * L + l) << 24) | (b[:, 2] << 16) | (b[:, 1] << 8) | b[:, 0]
            f[c, :, 16 + l] = has(b_id.astype(np.uint32), ids)
    x = torch.from_numpy(f.reshape(m * P, 32)).cuda()
    w = {n: torch.from_numpy(a).double().cuda() for n, a in _weights(seed).items()}
    return dict(x=x, z=torch.nn.functional.pad(_net(w, x[:, :24]), (0, 7)))


def _exact_frame(case, seed):
    """The definition of a frame, sample by sample without traversal."""
    L, m, W, H = case["levels"], case["m"], case["W"], case["H"]
    dims = _dims(case)
    sp = torch.tensor([1.0, 1.0, float(case["zs"])], dtype=torch.float64, device="cuda")
    if case["mode"] in ("homogeneous", "rates"):
        return None
    cam, chans = _view(case, seed, bits=case["bits"])
    if work(case)["flops"] / 34 > 4e9:
        return None
    levels, res, leaf, spacing, nb = _volume_scene(case, seed, case["bits"])
    grid = tuple(1 << max(0, (-(-dims[a] // leaf[a]) - 1).bit_length()) for a in range(3))
    sch = _schedule(dims, spacing, L)
    empty = torch.stack([_empty(_leaf_range(levels[0][c], leaf, grid), chans[c]) for c in range(m)])
    tf = torch.from_numpy(np.stack([c["tf"] for c in chans])).double().cuda()
    B, step, pix = case["brick"], 0.5, 2.0 * cam["ty"] / H
    # rays
    dev = dict(dtype=torch.float64, device="cuda")
    px, py = torch.arange(W, **dev), torch.arange(H, **dev)
    a = ((2 * px + 1 - W) / W)[None, :, None]
    b = ((H - 2 * py - 1) / H)[:, None, None]
    eye, F, R, U = (torch.tensor(cam[k], **dev) for k in ("eye", "F", "R", "U"))
    side = a * cam["tx"] * R + b * cam["ty"] * U
    if cam["proj"] == "ortho":
        o, d = (eye + side).reshape(-1, 3), F.expand(H * W, 3)
    else:
        d = (F + side).reshape(-1, 3)
        d = d / d.pow(2).sum(1, keepdim=True).sqrt()
        o = eye.expand(H * W, 3)
    o, d = o / sp, d / sp
    size = torch.tensor(dims, **dev)
    u0, u1 = -o / d, (size - o) / d
    t0 = torch.minimum(u0, u1).amax(1).clamp(min=0)
    t1 = torch.maximum(u0, u1).amin(1)
    rays = torch.nonzero((t0 <= t1)).view(-1)
    T = torch.ones(H * W, **dev)
    col = torch.zeros(H * W, 3, **dev)
    if len(rays) == 0:
        return dict(rgba=torch.zeros(H, W, 4, **dev))
    k0 = (t0 / step).floor().long()
    k1 = (t1 / step).ceil().long()
    stop = 1.0 - float(np.float32(TERM))
    resident = [[torch.from_numpy(r).cuda() for r in per] for per in res]
    whole = case["resident"] >= 1.0
    w0 = torch.tensor([c["W0"] / 256.0 for c in chans], **dev)
    iw = torch.tensor([256.0 / (c["W1"] - c["W0"]) for c in chans], **dev)
    slo, shi = min(c["lo"] for c in chans), min(c["hi"] for c in chans)
    lod = 0
    for k in range(int(k0[rays].min()), int(k1[rays].max()) + 2):
        t = k * step
        if k % 16 == 0 or k == int(k0[rays].min()):
            live = rays[(T[rays] > stop) & (k1[rays] >= k - 1) & (k0[rays] <= k + 17)]
        if len(live) == 0:
            continue
        lod = sum(1 for l in range(1, L) if (pix if cam["proj"] == "ortho" else t * pix) >= sch[l][1][0])
        r = 1
        if case["mode"] == "adaptive":
            r = sch[min(max(lod, slo), shi)][1][0]
            if k % r:
                continue
        u = o[live] + t * d[live]
        on = ((u >= 0) & (u < size)).all(1) & (T[live] > stop)
        n = live[on]
        if len(n) == 0:
            continue
        u = u[on]
        iu = u.long()
        lf = ((iu[:, 2] // leaf[2]) * grid[1] + iu[:, 1] // leaf[1]) * grid[0] + iu[:, 0] // leaf[0]
        use = ~empty[:, lf]  # [m][n]
        some = use.any(0)
        n, u, iu, use = n[some], u[some], iu[some], use[:, some]
        if len(n) == 0:
            continue
        val = torch.zeros(use.shape, **dev)
        left = use.clone()
        want = [min(max(lod, c["lo"]), c["hi"]) for c in chans]
        for l in range(min(want), L):
            cs = [c for c in range(m) if want[c] == l or (want[c] < l and not whole)]
            if not cs:
                continue
            dl, fl = sch[l]
            q = u / torch.tensor(fl, **dev) - 0.5
            qi = q.floor()
            fr = q - qi
            qi = qi.long()
            bk = [iu[:, x] // (B * fl[x]) for x in range(3)]
            bl = (bk[2] * nb[l][1] + bk[1]) * nb[l][0] + bk[0]
            ix = [[(qi[:, x] + e).clamp(0, dl[x] - 1) for e in (0, 1)] for x in range(3)]
            lin = [[[(ix[2][c] * dl[1] + ix[1][j]) * dl[0] + ix[0][i] for i in (0, 1)] for j in (0, 1)] for c in (0, 1)]
            for c in cs:
                flat = levels[l][c].reshape(-1)
                g = [[[_raw(flat[lin[zz][yy][xx]]).double() for xx in (0, 1)] for yy in (0, 1)] for zz in (0, 1)]
                e = [[g[zz][yy][0] + (g[zz][yy][1] - g[zz][yy][0]) * fr[:, 0] for yy in (0, 1)] for zz in (0, 1)]
                e = [e[zz][0] + (e[zz][1] - e[zz][0]) * fr[:, 1] for zz in (0, 1)]
                v = e[0] + (e[1] - e[0]) * fr[:, 2]
                ok = left[c] & resident[c][l][bl]
                val[c] = torch.where(ok, v, val[c])
                left[c] &= ~ok
        use = use & ~left
        p = ((val - w0[:, None]) * iw[:, None]).clamp(0, 1) * 255
        e = p.long()
        fp = (p - e)[..., None]
        row = torch.arange(m, device="cuda")[:, None]
        ta, tb = tf[row, e], tf[row, (e + 1).clamp(max=255)]
        c4 = ta + (tb - ta) * fp
        al = torch.where(use, c4[..., 3], torch.zeros_like(val))
        sa = al.sum(0)
        tr = (1 - al).prod(0) ** r
        rgb = (al[..., None] * c4[..., :3]).sum(0)
        hit = sa > 0
        scale = torch.where(hit, (1 - tr) / sa.clamp(min=1e-300), torch.zeros_like(sa))
        col[n] += (T[n] * scale)[:, None] * rgb
        T[n] = T[n] * torch.where(hit, tr, torch.ones_like(tr))
    return dict(rgba=torch.cat([col, (1 - T)[:, None]], 1).view(H, W, 4))
