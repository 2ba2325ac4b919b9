"""Performance cases of the raycaster: the work its users have it do, through its public entry points.

Kinds of work (each a path of the package's API):

  frame    one image of an AMR hierarchy with `render`: unlit or gradient-lit, trilinear or nearest
           cell, cell- or vertex-centred, with or without a level-of-detail cut, with a kept tile
           `Schedule` (a viewer that repaints one view) or without (a new view every call)
  learned  one unlit image with segment skipping (analytic bound, then the proposal network)
  light    one image with a point light's secondary rays
  serve    several cameras of mixed sizes in one persistent launch
  fit      one step of a transfer-function fit: checkpointed forward and adjoint (`AMRRender`)
  train    one optimiser step of the proposal network: forward, backward, Adam
  ingest   host data to a renderable scene: `build_tree` and `pack`

Hierarchies are synthetic: log-normal density with patches of 8^3..64^3 cells around its peaks
("cosmology"), nested 16^3 blocks around three collapsing cores over 20 levels ("deep"), and a
root grid with a few refined boxes ("tiny").  Everything is made from the seed: the field, the
patch boxes, the transfer function and the cameras.
"""
import math
import types

import numpy as np
import torch

import paper_1212_3333_amd as amr

DEV = "cuda"

# ---------------------------------------------------------------------------------------------
# Hierarchies: objects with the attributes build_tree and pack read
# ---------------------------------------------------------------------------------------------


def _patch(level, lo, cells, centering="cell"):
    extra = 1 if centering == "vertex" else 0
    dims = np.array(cells.shape[::-1], dtype=np.int64) - extra
    return types.SimpleNamespace(level=int(level), lo=np.asarray(lo, dtype=np.int64), dims=dims, cells=cells)


def _hierarchy(root, nlevels, patches, centering="cell"):
    return types.SimpleNamespace(origin=np.zeros(3), h0=np.full(3, 1.0 / root), refine=2, nlevels=int(nlevels),
                                 patches=patches, centering=centering)


class _LogNormal:
    """exp(2 g - 2) with g a unit-variance field of 64 Fourier modes, flat in log k up to 2 pi 2048."""

    def __init__(self, rng):
        k = 2 * math.pi * np.exp(rng.uniform(0.0, math.log(2048.0), 64))
        d = rng.normal(size=(64, 3))
        k = k[:, None] * d / np.linalg.norm(d, axis=1, keepdims=True)
        self.k = torch.from_numpy(k).to(DEV)
        self.phi = torch.from_numpy(rng.uniform(0, 2 * math.pi, 64)).to(DEV)

    def lattice(self, lo, dims, h, shift):
        """fp32 values [nz, ny, nx] at (lo + i + shift) h."""
        e = []
        for a in range(3):
            x = (torch.arange(int(dims[a]), device=DEV, dtype=torch.float64) + float(lo[a] + shift)) * h
            e.append(torch.exp(1j * (self.k[:, a, None] * x + (self.phi[:, None] if a == 2 else 0.0))).to(torch.complex64))
        m = (e[1][:, :, None] * e[0][:, None, :]).reshape(64, -1)
        g = (e[2].T @ m).real.reshape(tuple(int(d) for d in dims[::-1])) * math.sqrt(2.0 / 64)
        return torch.exp(2.0 * g - 2.0)


def _cosmology(rng, npatches, root, nlevels, centering="cell", values_rng=None):
    """Root root^3 in 2^3 patches; on each finer level the blocks of 64^3 cells (on a grid shifted
    by a random even offset) that hold the densest parent cells and lie at least half inside the
    parents; one block in ten is cut down to 32^3, 16^3 or 8^3.  values_rng: the cells hold another
    field, made from it, on these boxes."""
    f = _LogNormal(rng)
    vertex = centering == "vertex"
    half = root // 2
    boxes = [(0, np.array([i, j, k]) * half, np.full(3, half)) for k in range(2) for j in range(2) for i in range(2)]
    parents = boxes
    values = [f.lattice(lo, d, 1.0 / root, 0.5) for _, lo, d in boxes]
    cells = list(values)
    share = np.array([0.04, 0.12, 0.22, 0.30, 0.32])[:nlevels - 1]
    share = share / share.sum()
    for lev in range(1, nlevels):
        n_l = root * 2 ** lev
        off = rng.integers(0, 32, 3) * 2 - 64
        nb = int((n_l + 128) // 64)
        want = max(1, int(round(npatches * share[lev - 1])))
        score, count, maxima, keys = np.zeros(nb ** 3), np.zeros(nb ** 3), [], []
        for (_, lo, d), v in zip(parents, values):
            cuts = []                   # per axis: (block, slice of the parent's cells in it)
            for a in range(3):
                b = (2 * (lo[a] + np.arange(d[a])) - off[a]) // 64
                cuts.append([(int(k), slice(int(np.argmax(b == k)), int(np.argmax(b == k) + np.sum(b == k)))) for k in np.unique(b)])
            for kz, sz in cuts[2]:
                for ky, sy in cuts[1]:
                    for kx, sx in cuts[0]:
                        part = v[sz, sy, sx]
                        keys.append((kz * nb + ky) * nb + kx)
                        count[keys[-1]] += part.numel()
                        maxima.append(part.amax())
        np.maximum.at(score, keys, torch.stack(maxima).double().cpu().numpy())
        score[count < 0.5 * 32 ** 3] = 0.0
        order = np.argsort(-score, kind="stable")[:min(want, int((score > 0).sum()))]
        parents = []
        for key in order:
            lo = np.array([key % nb, (key // nb) % nb, key // (nb * nb)]) * 64 + off
            side = 64
            if rng.random() < 0.1:
                side = int(rng.choice([8, 16, 32]))
                lo = lo + rng.integers(0, 64 // side, 3) * side
            blo, bhi = np.maximum(lo, 0), np.minimum(lo + side, n_l)
            if np.all(bhi > blo):
                parents.append((lev, blo, bhi - blo))
        values = [f.lattice(lo, d, 1.0 / n_l, 0.5) for _, lo, d in parents]
        boxes = boxes + parents
        cells = cells + values
    sample = torch.cat([v.reshape(-1)[::max(1, v.numel() // 4096)] for v in cells])
    vhi = float(torch.quantile(sample[:1 << 22].double(), 0.999))
    if values_rng is not None:
        f = _LogNormal(values_rng)
        cells = [f.lattice(lo, d, 1.0 / (root * 2 ** lev), 0.5) for lev, lo, d in boxes]
    if vertex:
        cells = [f.lattice(lo, d + 1, 1.0 / (root * 2 ** lev), 0.0) for lev, lo, d in boxes]
    ps = [_patch(lev, lo, v.cpu().numpy(), centering) for (lev, lo, _), v in zip(boxes, cells)]
    return _hierarchy(root, nlevels, ps, centering), 0.0, vhi


def _deep(rng, nlevels=20, root=64, block=16, radius=44.0):
    """Three power-law cores; level l tiles a ball of `radius` cells around each with 16^3 blocks.
    Cells hold log10 of the density."""
    cores = rng.uniform(0.3, 0.7, (3, 3))
    amp = torch.from_numpy(10.0 ** (14.0 + rng.uniform(-0.5, 0.5, 3))).to(DEV)
    ct = torch.from_numpy(cores).to(DEV)

    def field(los, dims, h):
        x = [(torch.from_numpy(los[:, a]).to(DEV)[:, None] + torch.arange(dims, device=DEV)[None, :] + 0.5) * h for a in range(3)]
        rho = 1.0
        for j in range(3):
            r2 = (x[2] - ct[j, 2])[:, :, None, None] ** 2 + (x[1] - ct[j, 1])[:, None, :, None] ** 2 + \
                (x[0] - ct[j, 0])[:, None, None, :] ** 2
            rho = rho + amp[j] / (1.0 + r2 * 2.0 ** 48) * torch.exp(-r2 / (2 * 0.05 ** 2))
        return torch.log10(rho).float().cpu().numpy()

    ps = [_patch(0, [0, 0, 0], field(np.zeros((1, 3), np.int64), root, 1.0 / root)[0])]
    for lev in range(1, nlevels):
        n_l = root * 2 ** lev
        off = rng.integers(0, block // 2, 3) * 2
        keys = set()
        for c in cores * n_l:
            lo, hi = np.floor((c - radius - off) / block).astype(np.int64), np.floor((c + radius - off) / block).astype(np.int64)
            g = np.stack(np.meshgrid(*[np.arange(lo[a], hi[a] + 1) for a in range(3)], indexing="ij"), -1).reshape(-1, 3)
            near = np.clip(c, g * block + off, (g + 1) * block + off)
            keys |= {tuple(k) for k in g[np.sum((near - c) ** 2, axis=1) <= radius ** 2]}
        b0 = np.array(sorted(keys), dtype=np.int64) * block + off
        v = field(b0, block, 1.0 / n_l)
        for i in range(len(b0)):
            lo, hi = np.maximum(b0[i], 0), np.minimum(b0[i] + block, n_l)
            s = tuple(slice(int(lo[a] - b0[i][a]), int(hi[a] - b0[i][a])) for a in (2, 1, 0))
            if np.all(hi > lo):
                ps.append(_patch(lev, lo, np.ascontiguousarray(v[i][s])))
    return _hierarchy(root, nlevels, ps), 0.0, 14.5


def _tiny(rng):
    """Root 32^3 and four level-1 boxes of 8..16 root cells a side: a sum of eight Gaussians."""
    c, s, w = rng.random((8, 3)), rng.uniform(0.02, 0.1, 8), rng.random(8)

    def field(lo, d, h):
        z, y, x = np.meshgrid(*[(np.arange(d[a]) + lo[a] + 0.5) * h for a in (2, 1, 0)], indexing="ij")
        v = np.zeros_like(x)
        for j in range(8):
            v += w[j] * np.exp(-((x - c[j, 0]) ** 2 + (y - c[j, 1]) ** 2 + (z - c[j, 2]) ** 2) / (2 * s[j] ** 2))
        return v.astype(np.float32)

    ps = [_patch(0, [0, 0, 0], field([0, 0, 0], [32, 32, 32], 1.0 / 32))]
    taken = []
    while len(taken) < 4:
        ext = rng.integers(8, 17, 3)
        lo = np.array([rng.integers(0, 33 - e) for e in ext])
        if all(np.any(lo + ext <= a) or np.any(b <= lo) for a, b in taken):
            taken.append((lo, lo + ext))
            ps.append(_patch(1, 2 * lo, field(2 * lo, 2 * ext, 1.0 / 64)))
    return _hierarchy(32, 2, ps), 0.0, float(max(p.cells.max() for p in ps))


def _scene_data(case, rng):
    if case["scene"] == "deep":
        return _deep(rng)
    if case["scene"] == "tiny":
        return _tiny(rng)
    root = 128 if case["patches"] >= 1000 else 64
    if case["kind"] == "ingest":    # the next snapshot of a run on the same grids
        return _cosmology(np.random.default_rng([case["patches"], 9]), case["patches"], root, 6, values_rng=rng)
    return _cosmology(rng, case["patches"], root, 6, case.get("centering", "cell"))


# ---------------------------------------------------------------------------------------------
# Transfer functions and cameras
# ---------------------------------------------------------------------------------------------


def _lut(rng, scene):
    u = np.arange(256) / 255.0
    lut = np.zeros((256, 4))
    for ch in range(3):
        for _ in range(3):
            lut[:, ch] += rng.uniform(0.3, 1.0) * np.exp(-((u - rng.random()) ** 2) / (2 * rng.uniform(0.05, 0.3) ** 2))
    lut[:, :3] = np.clip(lut[:, :3], 0.0, 1.0)
    lut[:, 3] = {"deep": 1e-4 * 10.0 ** (10.0 * u), "tiny": 20.0 * u * u}.get(scene, 0.4 + 60.0 * u)
    return torch.from_numpy(lut.astype(np.float32)).to(DEV)


def _camera(eye, centre, width, height, fov=40.0, half=0.0):
    w = np.asarray(centre) - eye
    w = w / np.linalg.norm(w)
    u = np.cross(w, [0.0, 1.0, 0.0])
    u = u / np.linalg.norm(u)
    return dict(eye=eye, u=u, v=np.cross(u, w), w=w, width=int(width), height=int(height), ortho=half > 0.0,
                tan_half_fov=0.0 if half > 0.0 else math.tan(math.radians(fov) / 2),
                win=(half, half * height / width))


def _orbit(rng, width, height, radius=2.0, half=0.0):
    az, el = rng.uniform(0, 2 * math.pi), rng.uniform(-0.5, 0.5)
    d = np.array([math.cos(el) * math.sin(az), math.sin(el), -math.cos(el) * math.cos(az)])
    return _camera(0.5 + radius * d, (0.5, 0.5, 0.5), width, height, half=half)


def _params(case, lo, hi, t_min=1e-5):
    return dict(v_lo=lo, v_hi=hi, step_frac=0.5, uniform_step=False, t_min=t_min, lighting=int(case.get("lit", False)),
                light=(1.0, 1.0, 1.0), k_a=0.3, k_d=0.7, eps_g=1e-3, clip_lo=(-1e300,) * 3, clip_hi=(1e300,) * 3,
                interp=int(case.get("nearest", False)), lod=float(case.get("lod", 0.0)))


def _load(h):
    return amr.pack(amr.build_tree(h), h, device=DEV)


# ---------------------------------------------------------------------------------------------
# The cases
# ---------------------------------------------------------------------------------------------


def listed():
    return [
        # a thumbnail of a small data set while it is set up: launches and latency count
        dict(name="thumbnail lit", kind="frame", scene="tiny", width=256, height=256, lit=True, ortho=True, schedule=False),
        # the benchmark's frame: a viewer that repaints one view of a large snapshot, gradient-lit
        dict(name="view lit", kind="frame", scene="cosmology", patches=2000, width=1024, height=1024, lit=True, schedule=True),
        # a snapshot of half that size flown through unlit: every call a view not seen before
        dict(name="flight unlit", kind="frame", scene="cosmology", patches=1000, width=1024, height=1024, lit=False, schedule=False),
        # an odd-sized window on a medium snapshot, gradient-lit, each call a new view
        dict(name="window lit", kind="frame", scene="cosmology", patches=250, width=517, height=389, lit=True, schedule=False),
        # cell values shown as they are (nearest cell), gradient-lit
        dict(name="cells lit", kind="frame", scene="cosmology", patches=250, width=901, height=677, lit=True, nearest=True,
             schedule=False),
        # a zoom simulation over 20 levels, the whole domain in view
        dict(name="deep unlit", kind="frame", scene="deep", width=1024, height=1024, lit=False, schedule=False),
        # the same with segments skipped by the bound and the network
        dict(name="deep learned", kind="learned", scene="deep", width=1024, height=1024),
        # global illumination: one secondary ray to the light from every sample
        dict(name="point light", kind="light", scene="cosmology", patches=250, width=384, height=288),
        # a server's batch: cameras of mixed sizes in one persistent launch, gradient-lit
        dict(name="serving batch", kind="serve", scene="cosmology", patches=250, cams=12, lit=True),
        # one step of a transfer-function fit over eight views, gradient-lit, no early termination
        dict(name="fit step", kind="fit", scene="cosmology", patches=250, cams=8, width=384, height=384, lit=True),
        # one step of the network's training on logged segments
        dict(name="train step", kind="train", rows=65536),
        # a snapshot from host memory to a renderable scene
        dict(name="ingest", kind="ingest", scene="cosmology", patches=250),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["frame"] * 5 + ["learned", "light", "serve", "fit", "train", "ingest"])
    if kind == "frame":
        scene = rng.choice(["tiny", "cosmology", "cosmology", "cosmology", "deep"])
        c = dict(kind=kind, scene=scene, width=_log(rng, 64, 1024), height=_log(rng, 64, 1024), lit=rng.random() < 0.6,
                 schedule=rng.random() < 0.3, ortho=rng.random() < 0.25)
        if scene == "deep":
            c["lit"] = c["ortho"] = False
        if scene == "cosmology":
            c["patches"] = _log(rng, 40, 600)
            option = rng.choice(["", "", "nearest", "vertex", "lod"])
            if option == "nearest":
                c["nearest"] = True
            elif option == "vertex":
                c["centering"] = "vertex"
            elif option == "lod":
                c["lod"] = rng.choice([1.0, 2.0, 4.0])
        return c
    if kind == "learned":
        return dict(kind=kind, scene="deep", width=_log(rng, 128, 1024), height=_log(rng, 128, 1024))
    if kind == "light":
        return dict(kind=kind, scene="cosmology", patches=_log(rng, 40, 250), width=_log(rng, 48, 384),
                    height=_log(rng, 48, 288))
    if kind == "serve":
        return dict(kind=kind, scene="cosmology", patches=_log(rng, 60, 250), cams=rng.randint(2, 12), lit=rng.random() < 0.7)
    if kind == "fit":
        return dict(kind=kind, scene="cosmology", patches=_log(rng, 60, 250), cams=rng.randint(1, 6), width=_log(rng, 64, 384),
                    height=_log(rng, 64, 384), lit=rng.random() < 0.7)
    if kind == "train":
        return dict(kind=kind, rows=_log(rng, 512, 65536))
    return dict(kind=kind, scene="cosmology", patches=_log(rng, 40, 250))


def _train_inputs(case, seed):
    """Logged segments' features (each in [0, 1] or a small logarithm), their opacity ratios, and
    the fp32 master weights."""
    rng = np.random.default_rng([seed, 5])
    n = case["rows"]
    x = rng.random((n, 12))
    x[:, 1] = rng.normal(0.2, 0.3, n)
    w = np.concatenate([rng.normal(0, math.sqrt(2 / 12), 768), rng.normal(0, 0.05, 64), rng.normal(0, math.sqrt(2 / 64), 4096),
                        rng.normal(0, 0.05, 64), rng.normal(0, math.sqrt(1 / 64), 128), [0.0, 1.0]])
    return x.astype(np.float32), rng.random(n).astype(np.float32) ** 2, w.astype(np.float32)


def prepare(case, seed):
    kind = case["kind"]
    rng = np.random.default_rng([seed, 1])
    s = dict(case)
    if kind == "train":
        s["x"], s["t"], s["w"] = (torch.from_numpy(v).to(DEV) for v in _train_inputs(case, seed))
        s["m"], s["v"], s["step"] = torch.zeros_like(s["w"]), torch.zeros_like(s["w"]), 0
        return s
    h, lo, hi = _scene_data(case, rng)
    if kind == "ingest":
        s["h"] = h
        return s
    s["scene"] = _load(h)
    s["lut"] = _lut(rng, case["scene"])
    if kind == "fit":
        n = case["cams"]
        s["cam_list"] = [_orbit(rng, case["width"], case["height"]) for _ in range(n)]
        s["lut"].requires_grad_(True)
        s["shading"] = torch.tensor([1.0, 1.0, 1.0, 0.3, 0.7], requires_grad=True)
        s["params"] = _params(case, lo, hi, t_min=0.0)
        s["sched"] = amr.Schedule(s["cam_list"], DEV)
        # the images to match: smooth, of the renders' brightness
        g = torch.Generator(device=DEV).manual_seed(int(seed))
        t = torch.rand((n, 4, 8, 8), device=DEV, generator=g)
        t = torch.nn.functional.interpolate(t, size=(case["height"], case["width"]), mode="bilinear", align_corners=True)
        t = t.permute(0, 2, 3, 1).reshape(-1, 4)
        s["target"] = t.reshape(case["height"], case["width"], 4) if n == 1 else t
        return s
    s["params"] = _params(case, lo, hi)
    if kind == "serve":
        sizes = np.random.default_rng([case["cams"], 9]).choice([256, 512, 768, 1024], case["cams"])
        s["cam_list"] = [_orbit(rng, int(z), int(z), radius=float(rng.uniform(1.8, 2.4))) for z in sizes]
        s["table"] = amr.camera_table(s["cam_list"], device=DEV)
        s["queue"] = amr.queue_buffer(len(s["cam_list"]), device=DEV)
        s["out"] = torch.empty(4 * int(sum(int(z) ** 2 for z in sizes)), device=DEV)
        s["params"].update(persistent=1, tile_w=8, tile_h=8, blocks_per_cu=8, waves_per_simd=3, queue_order=1)
        return s
    s["cam"] = _orbit(rng, case["width"], case["height"], half=0.9 if case.get("ortho") else 0.0)
    s["out"] = torch.empty(4 * case["width"] * case["height"], device=DEV)
    s["extra"] = {}
    if kind == "learned":
        _, _, w = _train_inputs(dict(rows=1), seed)
        w[768 + 64 + 4096 + 64:-2] *= 0.1
        w[-2:] = (-4.0, 1.0)
        s["packed"] = amr.mlp_pack(torch.from_numpy(w).to(DEV))
        s["params"].update(tau_e=5e-4, tau_s=0.0)
        s["extra"] = dict(d_mlp=s["packed"])
    elif kind == "light":
        s["params"].update(lighting=2, light=(0.5, 0.5, 0.5))
    elif case["schedule"]:
        s["sched"] = amr.Schedule(s["cam"], DEV)
        s["extra"] = s["sched"].params()
    return s


def run(s):
    kind = s["kind"]
    if kind == "train":
        s["step"] += 1
        y, hidden = amr.mlp_forward(s["x"], s["w"])
        dw, loss = amr.mlp_backward(s["x"], s["w"], hidden, y, s["t"])
        amr.mlp_adam_step(s["w"], dw, s["m"], s["v"], s["step"], lr=3e-3)
        return dict(y=y, hidden=hidden, dw=dw, loss=loss, w=s["w"])
    if kind == "ingest":
        tree = amr.build_tree(s["h"])
        scene = amr.pack(tree, s["h"], device=DEV)
        info = tree.info()
        # without the 256 spare bytes after the last brick, which hold no data and are not written
        return dict(pool=scene.pool[:-256], nodes=info["nodes"], leaves=info["leaves"], depth=info["depth"])
    if kind == "fit":
        s["lut"].grad = s["shading"].grad = None
        rgba = amr.AMRRender.apply(s["lut"], s["shading"], s["scene"], s["cam_list"], s["params"], 4, 16, False, s["sched"])
        loss = ((rgba - s["target"]) ** 2).mean()
        loss.backward()
        return dict(rgba=rgba.detach(), loss=loss.detach(), lut=s["lut"].grad, shading=s["shading"].grad)
    if kind == "serve":
        return amr.render(s["scene"], s["cam_list"], s["lut"], s["params"], out=s["out"], d_cams=s["table"],
                          d_queue=s["queue"])["rgba"]
    return amr.render(s["scene"], s["cam"], s["lut"], s["params"], out=s["out"], **s["extra"])["rgba"]


def work(case):
    """Estimates from the case's sizes alone: samples per pixel from the scenes' mean ray lengths
    (a unit box seen from radius 2 covers 0.85 of the image), and 4 bytes for each cell that a
    pixel's samples can reach, at most the cells of the scene's blocks in view."""
    kind = case["kind"]
    if kind == "train":
        n, p = case["rows"], 768 + 64 + 4096 + 64 + 130
        # x, t, y, and the activations written and read once; three products forward, five backward
        return dict(bytes=float(n * (48 + 4 + 2 * 8 + 2 * 512) + p * 4 * 8), flops=float(n * 2 * (768 + 4096 + 128) * 3))
    if case["scene"] == "tiny":
        cells, per_pixel = 32768 + 4 * 24 ** 3, 60
    elif case["scene"] == "deep":
        cells, per_pixel = 9600 * 4096, 8 if kind == "learned" else 120
    else:
        cells, per_pixel = 250000 * case["patches"], 370 if case["patches"] >= 1000 else 250
    if kind == "ingest":
        return dict(bytes=float(4 * cells + 8 * 1.2 * cells), flops=float(0.1 * cells * 8))
    pixels = 0.36 * 1024 ** 2 * case["cams"] if kind == "serve" else case["width"] * case["height"] * case.get("cams", 1)
    samples = float(pixels) * per_pixel
    per = {"light": 59 + 100 * 30}.get(kind, 206 if case.get("lit") else 59)
    reach = min(0.7 * cells, samples)
    if kind == "fit":      # each sample's value and gradient kept from the forward for the adjoint
        return dict(bytes=4 * reach + 3 * 16 * pixels + (32 * samples if case.get("lit") else 4 * reach), flops=samples * 2 * per)
    return dict(bytes=4 * reach + 16 * pixels, flops=samples * per)


def exact(case, seed):
    """The training step in 64 bits.  The renders' samples lie on segments of the kD-tree that the
    package builds, which has no plain counterpart here; packed bricks are compared as bytes."""
    if case["kind"] != "train":
        return None
    x, t, w = (torch.from_numpy(v).to(DEV).double() for v in _train_inputs(case, seed))
    parts = torch.split(w, [768, 64, 4096, 64, 128, 2])
    w1, b1, w2, b2, w3, b3 = (p.reshape(sh).clone().requires_grad_(True) for p, sh in
                              zip(parts, [(12, 64), (64,), (64, 64), (64,), (64, 2), (2,)]))
    h1 = torch.relu(x @ w1 + b1)
    h2 = torch.relu(h1 @ w2 + b2)
    y = torch.sigmoid(h2 @ w3 + b3)
    q = torch.tensor([0.01, 0.99], dtype=torch.float64, device=DEV)
    r = t[:, None] - y
    loss = torch.maximum(q * r, (q - 1.0) * r).sum(1).mean()
    loss.backward()
    dw = torch.cat([p.grad.reshape(-1) for p in (w1, b1, w2, b2, w3, b3)])
    # Adam's first step from zero moments: m / c1 = dw, v / c2 = dw^2
    new = w - 3e-3 * dw / (dw.abs() + 1e-8)
    return dict(y=y.detach(), hidden=torch.cat([h1, h2], 1).detach(), dw=dw, loss=loss.detach().reshape(1), w=new)
