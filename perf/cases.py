"""Performance cases of the fragment-history-volume path.

Each case is one pass through the package's public entry points on inputs a
program has in hand: meshes, fragment arrays, splat images, training crops,
workspaces allocated once. The cases cover the smallest calls (bound by launch
latency), the benchmark's own sizes and large scenes, and every stage: pixel
and octant lists with their compaction, arrays straight from the triangles,
novel views (plain and shaded), ray casting, the learned fill, its training
gradient and batches of scenes.
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

from paper_2211_15460_amd import fhv, scenes
from paper_2211_15460_amd import learned_fill as lf

# Octant leaves are two samples wide, so a surface leaves about 3.5 fragments
# in every octant it meets (0.29 occupied octants per fragment on the
# procedural scenes, at every depth).
OCC_PER_FRAG = 0.29


def listed() -> list[dict]:
    return [
        # the smallest pass: 64 large triangles into a 128 x 128 per-pixel
        # capture and three small views; launches and latency count
        dict(name="pixel_lists_128", op="pixel", scene="soup", tris=64, width=128, height=128, views=3),
        # the reference image of a novel view, as training data needs one per
        # view: the scene's triangles captured per pixel at 1080p, the
        # nearest fragment of every pixel kept
        dict(name="reference_image_1080p", op="pixel", scene="objects", tris=200_000, width=1920, height=1080, views=1),
        # the benchmark's scene into per-octant lists and their arrays
        dict(name="octant_lists_200k", op="lists", scene="objects", tris=200_000, levels=9, projection=0),
        # many small triangles at octree depth 10: the large-scene regime
        dict(name="octant_lists_1m", op="lists", scene="small", tris=1_000_000, levels=10, projection=0),
        # arrays without lists (two rasterizations), the benchmark's scene
        dict(name="octant_arrays_200k", op="arrays", scene="objects", tris=200_000, levels=9, projection=0),
        # the benchmark's three 1080p views
        dict(name="views_3x1080p", op="views", scene="objects", tris=200_000, levels=9, width=1920, height=1080,
             views=3, shade=False),
        # a shaded stereo pair of the large scene in 4K
        dict(name="stereo_shaded_4k", op="views", scene="small", tris=1_000_000, levels=10, width=3840, height=2160,
             views=2, shade=True),
        # transparency by ray casting, three 1080p views
        dict(name="rays_blended_3x1080p", op="rays", scene="objects", tris=200_000, levels=9, width=1920,
             height=1080, views=3, blend=True),
        # one interactive 720p view of a small scene by simple ray casting
        dict(name="rays_nearest_720p", op="rays", scene="objects", tris=20_000, levels=8, width=1280, height=720,
             views=1, blend=False),
        # the learned fill of the benchmark's three views
        dict(name="fill_3x1080p", op="fill", levels=4, images=3, width=1920, height=1080),
        # the gradient of one training batch: 8 crops of 256 x 256
        dict(name="train_8x256", op="train", levels=4, images=8, width=256, height=256),
        # a batch of scenes of very different sizes, eight 720p views each,
        # replayed as one graph
        dict(name="batch_16x8x720p", op="batch", scenes=16, levels=9, width=1280, height=720, views=8),
    ]


def _log(rng: random.Random, lo: float, hi: float) -> int:
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng: random.Random) -> dict:
    op = rng.choice(["pixel", "pixel", "lists", "lists", "arrays", "views", "views", "rays", "fill", "train", "batch"])
    if op == "pixel":
        if rng.random() < 0.5:
            return dict(op=op, scene="soup", tris=_log(rng, 16, 1500), width=_log(rng, 48, 300),
                        height=_log(rng, 48, 300), views=rng.randint(1, 4))
        return dict(op=op, scene="objects", tris=_log(rng, 2000, 300_000), width=_log(rng, 320, 2560),
                    height=_log(rng, 200, 1440), views=1)
    if op in ("lists", "arrays"):
        levels = rng.randint(6, 10)
        top = min(900_000, 900_000 * 4 ** (9 - levels))
        return dict(op=op, scene="objects", tris=_log(rng, 1500, top), levels=levels,
                    projection=rng.choice([0, 0, 0, 1, 2, 3]))
    if op == "views":
        levels = rng.randint(7, 10)
        return dict(op=op, scene="objects", tris=_log(rng, 2000, min(400_000, 400_000 * 4 ** (9 - levels))),
                    levels=levels, width=_log(rng, 200, 2560), height=_log(rng, 160, 1440), views=rng.randint(1, 6),
                    shade=rng.random() < 0.5)
    if op == "rays":
        # large views of coarse arrays are mostly holes, whose rays stop
        # nowhere: at most one 1080p view's pixels in all
        levels, w, h = rng.randint(7, 9), _log(rng, 160, 1920), _log(rng, 120, 1080)
        return dict(op=op, scene="objects", tris=_log(rng, 2000, 200_000), levels=levels, width=w, height=h,
                    views=rng.randint(1, max(1, min(3, 2_073_600 // (w * h)))), blend=rng.random() < 0.5)
    if op == "fill":
        levels = rng.choice([2, 3, 4, 4, 4])
        m = 2 ** (levels - 1)
        return dict(op=op, levels=levels, images=rng.randint(1, 3), width=m * (_log(rng, 160, 1920) // m),
                    height=m * (_log(rng, 120, 1080) // m))
    if op == "train":
        levels = rng.choice([3, 4, 4])
        m = 2 ** (levels - 1)
        return dict(op=op, levels=levels, images=rng.randint(1, 8), width=m * (_log(rng, 64, 256) // m),
                    height=m * (_log(rng, 64, 256) // m))
    return dict(op=op, scenes=rng.randint(2, 12), levels=rng.randint(7, 9), width=_log(rng, 160, 1280),
                height=_log(rng, 120, 720), views=rng.randint(1, 8))


# ------------------------------------------------------------------ inputs

def _mesh(case: dict, seed: int) -> scenes.Mesh:
    n = case["tris"]
    if case["scene"] == "soup":
        return scenes.clip_soup(n, seed)
    if case["scene"] == "small":   # the large scene's objects of about 250 triangles each
        return scenes.cube_scene(n, seed, scale_range=(0.012, 0.046), n_objects=max(1, n // 250))
    return scenes.pofl_scene(seed, n)


def _to_clip(mesh: scenes.Mesh, view: scenes.View, levels: int) -> scenes.Mesh:
    """The mesh in the clip space of a novel view of its scene cube."""
    m = view.m.astype(np.float64)
    s = (mesh.pos.astype(np.float64) * float(2 ** (levels + 8))) @ m[:, :3].T + m[:, 3]
    s = (s - np.array([0.0, 0.0, 1.0])) / np.array([view.width, view.height, 1.0]) * 2.0 - 1.0
    return scenes.Mesh(s.astype(np.float32), mesh.rgba, mesh.tri, None)


def _capacity(case: dict) -> int:
    """Pool slots a program sets aside for a case's scenes: about twice the
    fragments expected of the scene family (its members differ), a third
    more where many small objects even the count out."""
    op, n = case["op"], case.get("tris", 0)
    objects = 22.0 * max(0, n - 2048) / 2 ** 20   # surface of the objects and of the ground, cube sides squared
    ground = min(1.0, n / 2048.0)
    if op == "pixel" and case["scene"] == "soup":
        return int(2 * n * 11 / 144 * case["width"] * case["height"]) + 4096
    if op == "pixel":
        return int((objects + 0.2) * (case["height"] / 1.25) ** 2) + 4096
    samples = float(2 ** (case["levels"] + 1)) ** 2
    if op == "batch":
        return int(case["scenes"] * (1.0 + 1.7 + 1.0) * samples * 1.5)
    if case["scene"] == "small":
        return int(1.3 * (n / 250 * 4.57 * 0.00074 + 1.0) * samples)
    share = (1.0, 0.5, 1.6, 1.6)[case.get("projection", 0)]   # projected area
    return int((2.0 * (objects + ground) + 0.5) * samples * share)


def _lists(dm, d, case: dict):
    """Lists for the case's scenes; grown, as after any overflow, where a
    first capture counts more fragments than they hold."""
    cap = _capacity(case)
    lists = fhv.alloc_lists(d, 0)
    fhv.capture(dm, d, lists)
    return fhv.alloc_lists(d, max(cap, int(lists.counter.item())))


def _pofa(cap: int):
    p = fhv.alloc_pofa(cap)
    for t in (p.oct_key, p.oct_off, p.oct_cnt, p.frag):
        t.zero_()
    return p


def _arrays_of(mesh, d, case: dict):
    """Per-octant arrays of a mesh (what novel views are made from)."""
    dm = fhv.to_device(mesh)
    lists = _lists(dm, d, case)
    fhv.capture(dm, d, lists)
    return fhv.compact(lists, d, _pofa(lists.capacity))


def _bytes(n: int) -> torch.Tensor:
    return torch.empty(max(int(n), 1), dtype=torch.uint8, device="cuda")


def _angles(rng: random.Random, n: int) -> list[float]:
    t0 = rng.uniform(0.0, 90.0)
    return [t0 + 30.0 * i for i in range(n)]


def prepare(case: dict, seed: int) -> dict:
    rng = random.Random(seed)
    op = case["op"]
    st = {"case": case}
    if op == "pixel":
        W, H = case["width"], case["height"]
        mesh = _mesh(case, seed)
        if case["scene"] == "soup":
            st["views"] = [scenes.ppfl_view(t, W, H) for t in _angles(rng, case["views"])]
        else:
            mesh = _to_clip(mesh, scenes.cube_view(rng.uniform(0.0, 90.0), 9, W, H), 9)
            st["views"] = [scenes.ppfl_view(0.0, W, H)]
        d = fhv.desc(fhv.FHV_PPFL, W, H)
    elif op in ("lists", "arrays"):
        mesh = _mesh(case, seed)
        d = fhv.desc(fhv.FHV_POFL, levels=case["levels"], projection=case["projection"])
    if op in ("pixel", "lists", "arrays"):
        dm = fhv.to_device(mesh)
        lists = _lists(dm, d, case)
        cap = lists.capacity
        st.update(mesh=dm, d=d, arrays=_pofa(cap))
        if op == "arrays":
            st["ws"] = _bytes(fhv.capture_arrays_workspace(d, dm.n_tri, cap))
        else:
            st.update(lists=lists, ws_a=_bytes(fhv.capture_workspace(d, dm.n_tri)),
                      ws_b=_bytes(fhv.compact_workspace(d, cap)))
        if op == "pixel":
            n = len(st["views"])
            st.update(img=fhv.alloc_images(n, W, H), ws_c=_bytes(fhv.splat_workspace(cap, n, W, H)))
        return st
    if op in ("views", "rays"):
        W, H, L = case["width"], case["height"], case["levels"]
        mesh = _mesh(case, seed)
        d = fhv.desc(fhv.FHV_POFL, levels=L)
        angles = _angles(rng, case["views"])
        if op == "rays":   # a transparency of its own for every vertex
            a = np.random.default_rng(seed).integers(0, 256, mesh.rgba.size, dtype=np.uint32)
            mesh = scenes.Mesh(mesh.pos, (mesh.rgba & np.uint32(0x00FFFFFF)) | (a << np.uint32(24)), mesh.tri, mesh.obj)
            st["views"] = [scenes.cube_view(t, L, W, H, splat_px=1) for t in angles]
        elif case["shade"] and case["views"] == 2:
            st["views"] = scenes.stereo_views(angles[0], L, W, H)
        else:
            st["views"] = [scenes.cube_view(t, L, W, H) for t in angles]
        st.update(d=d, arrays=_arrays_of(mesh, d, case))
        n = len(st["views"])
        if op == "rays":
            st.update(out=torch.zeros((n, H, W, 4), dtype=torch.float32, device="cuda"), ws=_bytes(fhv.raycast_workspace(d)))
        else:
            st.update(img=fhv.alloc_images(n, W, H), ws=_bytes(fhv.splat_workspace(st["arrays"].cap_frag, n, W, H)))
            if case["shade"]:
                st["lights"] = np.stack([fhv.light_vectors(v, (0.3, 0.8, -0.5)) for v in st["views"]])
        return st
    if op in ("fill", "train"):
        st.update(_fill_state(case, seed, rng))
        return st
    # batch
    W, H, V, L = case["width"], case["height"], case["views"], case["levels"]
    meshes = scenes.batched_scenes(seed, case["scenes"])
    b = fhv.to_device_batch(meshes, L)
    views = [[scenes.cube_view(t, L, W, H) for t in _angles(rng, V)] for _ in meshes]
    vm = fhv.batch_view_matrices(views)
    img = fhv.alloc_images(len(meshes) * V, W, H)
    px = views[0][0].splat_px
    small = fhv.alloc_batch_lists(b, 0)   # a first run counts the fragments
    fhv.batch_run(b, vm, W, H, px, small, fhv.alloc_pofa(0), img)
    lists = fhv.alloc_batch_lists(b, max(_capacity(case), int(small.counter.item())))
    vs = fhv.BatchViews_(vm.data_ptr(), V, W, H, px)
    st.update(batch=b, vm=vm, px=px, lists=lists, arrays=_pofa(lists.capacity), img=img,
              ws=_bytes(fhv.batch_workspace(b, vs, lists.capacity)))
    return st


def _params(levels: int, seed: int) -> torch.Tensor:
    """Network weights with the head away from zero, as training leaves it."""
    p = lf.init_params(seed, levels)
    g = np.random.default_rng(seed + 1)
    p[-99:-3] = 0.02 * g.standard_normal(96)
    p[-3:] = 0.005 * g.standard_normal(3)
    return torch.from_numpy(p).to("cuda")


def _fill_state(case: dict, seed: int, rng: random.Random) -> dict:
    """Splat images of the benchmark's scene family (seen at depth 9), and
    for training random crops of them with their reference images."""
    L, N, W, H = case["levels"], case["images"], case["width"], case["height"]
    st = {"params": _params(L, seed)}
    mesh = scenes.pofl_scene(seed)
    if case["op"] == "fill":
        views = [scenes.cube_view(t, 9, W, H) for t in _angles(rng, N)]
        st["img"], _ = lf.render_splats(mesh, 9, views)
    else:
        view = scenes.cube_view(rng.uniform(0.0, 90.0), 9, 1920, 1080)
        img, _ = lf.render_splats(mesh, 9, [view])
        target = lf.gpu_reference(mesh, 9, view)[None]
        g = np.random.default_rng(seed)
        o = np.stack([np.zeros(N, np.int64), g.integers(200, 880 - H, N), g.integers(480, 1440 - W, N)], 1)
        parts = []
        for t in (img.rgba, img.depth, img.cov, target):
            parts.append(torch.stack([t[v, y:y + H, x:x + W] for v, y, x in o.tolist()]).contiguous())
        st["img"], st["target"] = lf.SplatImages(*parts[:3]), parts[3]
        st["grad"] = torch.zeros_like(st["params"])
        st["loss"] = torch.zeros(1, dtype=torch.float32, device="cuda")
    st["ws"] = _bytes(fhv.fill_workspace(L, N, H, W, case["op"] == "train"))
    return st


# ------------------------------------------------------------------ a pass

def _table(p) -> list:
    return [p.oct_key, p.oct_off, p.oct_cnt, p.frag, p.n_occ, p.n_frag]


def _images(img) -> list:
    return [img.zbuf, img.rgba, img.depth, img.cov]


def run(st: dict):
    case = st["case"]
    op = case["op"]
    if op in ("pixel", "lists"):
        fhv.capture(st["mesh"], st["d"], st["lists"], st["ws_a"])
        fhv.compact(st["lists"], st["d"], st["arrays"], st["ws_b"])
        if op == "lists":
            return {"count": st["lists"].counter, "arrays": _table(st["arrays"])}
        img = fhv.splat(st["arrays"], st["d"], st["views"], st["img"], ws=st["ws_c"])
        return {"count": st["lists"].counter, "arrays": _table(st["arrays"]), "images": _images(img)}
    if op == "arrays":
        return {"arrays": _table(fhv.capture_arrays(st["mesh"], st["d"], st["arrays"], st["ws"]))}
    if op == "views":
        img = fhv.splat(st["arrays"], st["d"], st["views"], st["img"], ws=st["ws"])
        out = {"images": _images(img)}
        if case["shade"]:
            out["shaded"] = fhv.shade(st["arrays"], img, st["lights"])
        return out
    if op == "rays":
        mode, tau = (fhv.FHV_RAY_BLEND, 1.0 / 256.0) if case["blend"] else (fhv.FHV_RAY_NEAREST, 0.0)
        return {"image": fhv.raycast(st["arrays"], st["d"], st["views"], mode, tau, st["out"], st["ws"])}
    img = st.get("img")
    if op == "fill":
        rgba, res = fhv.fill(st["params"], img.rgba, img.depth, img.cov, case["levels"], residual=True, ws=st["ws"])
        return {"rgba": rgba, "residual": res}
    if op == "train":
        # the batch's loss and gradient, for a program with an optimizer of
        # its own (step 0 leaves the parameters as they are)
        fhv.fill_train_step(st["params"], None, None, 0, 0.0, img.rgba, img.depth, img.cov, st["target"],
                            case["levels"], loss=st["loss"], grad=st["grad"], ws=st["ws"])
        return {"loss": st["loss"], "grad": st["grad"]}
    fhv.batch_run(st["batch"], st["vm"], case["width"], case["height"], st["px"], st["lists"], st["arrays"], img,
                  st["ws"], fhv.FHV_BATCH_GRAPH)
    return {"count": st["lists"].counter, "arrays": _table(st["arrays"]), "images": _images(img)}


# ------------------------------------------------------------------ least work

def _frags(mesh: scenes.Mesh, levels: int, projection: int) -> float:
    """Fragments of an octant capture: the triangles' area in samples."""
    p = mesh.pos.astype(np.float64)[mesh.tri.astype(np.int64)]
    n = 0.5 * np.cross(p[:, 1] - p[:, 0], p[:, 2] - p[:, 0])
    if projection == 0:
        area = np.linalg.norm(n, axis=1).sum()
    elif projection == 1:
        area = np.abs(n[:, 2]).sum()
    else:
        area = np.abs(n).sum()
    return float(area) * (2 ** (levels + 1)) ** 2


def _pixel_frags(mesh: scenes.Mesh, W: int, H: int) -> float:
    p = mesh.pos.astype(np.float64)[mesh.tri.astype(np.int64)][:, :, :2]
    u, v = p[:, 1] - p[:, 0], p[:, 2] - p[:, 0]
    return float(0.5 * np.abs(u[:, 0] * v[:, 1] - u[:, 1] * v[:, 0]).sum() * 0.25 * W * H)


def _mesh_bytes(mesh: scenes.Mesh) -> float:
    return 16.0 * mesh.n_vert + 13.0 * mesh.n_tri


def fill_flops(levels: int) -> float:
    """Matrix-product operations of the network per pixel."""
    ch = [32 << l for l in range(levels)]
    f, cin = 0.0, 6
    for l in range(levels):
        f += 2.0 * 9 * (cin * ch[l] + ch[l] * ch[l]) / 4 ** l
        cin = ch[l]
    for l in range(levels - 1):
        f += 2.0 * ch[l + 1] * ch[l] / 4 ** l + 2.0 * 9 * (2 * ch[l] * ch[l] + ch[l] * ch[l]) / 4 ** l
    return f + 2.0 * 3 * ch[0]


def work(case: dict) -> dict:
    op = case["op"]
    pix = case.get("width", 0) * case.get("height", 0)
    if op in ("fill", "train"):
        n = case["images"] * pix
        params = 4.0 * lf.init_params(0, case["levels"]).size
        if op == "fill":
            return {"bytes": n * (9.0 + 4.0 + 12.0) + params, "flops": n * fill_flops(case["levels"])}
        return {"bytes": n * 13.0 + 2 * params, "flops": 3.0 * n * fill_flops(case["levels"])}
    if op == "batch":
        meshes = scenes.batched_scenes(0, case["scenes"])
        F = sum(_frags(m, case["levels"], 0) for m in meshes)
        keys = case["scenes"] * 8 ** case["levels"]
        b = sum(_mesh_bytes(m) for m in meshes) + F * (16 + (8 if keys > 2 ** 32 else 4) + 16 + 16 * OCC_PER_FRAG)
        return {"bytes": b + 17.0 * pix * case["views"] * case["scenes"], "flops": 0}
    mesh = _mesh(case, 0)
    if op == "pixel":
        W, H = case["width"], case["height"]
        if case["scene"] != "soup":
            mesh = _to_clip(mesh, scenes.cube_view(30.0, 9, W, H), 9)
        F = _pixel_frags(mesh, W, H)
        return {"bytes": _mesh_bytes(mesh) + 4.0 * pix + 36.0 * F + 16.0 * min(F, pix) + 17.0 * pix * case["views"],
                "flops": 0}
    F = _frags(mesh, case["levels"], case.get("projection", 0))
    table = F * (16 + 16 * OCC_PER_FRAG)   # records and occupied octants
    if op == "lists":
        return {"bytes": _mesh_bytes(mesh) + 4.0 * 8 ** case["levels"] + 20.0 * F + table, "flops": 0}
    if op == "arrays":
        return {"bytes": _mesh_bytes(mesh) + table, "flops": 0}
    if op == "views":
        return {"bytes": table + case["views"] * pix * (17.0 + (24.0 if case["shade"] else 0.0)), "flops": 0}
    return {"bytes": table + 16.0 * case["views"] * pix, "flops": 0}


# ------------------------------------------------------------------ 64 bits

def _conv3(x, w, b):
    """3x3 convolution, zero padding, of x [N, H, W, C] with w [co, 3, 3, C]."""
    N, H, W, C = x.shape
    xp = torch.nn.functional.pad(x, (0, 0, 1, 1, 1, 1))
    o = b.expand(N * H * W, w.shape[0])
    for dy in range(3):
        for dx in range(3):
            o = o + xp[:, dy:dy + H, dx:dx + W, :].reshape(-1, C) @ w[:, dy, dx, :].t()
    return o.view(N, H, W, -1)


def _up2(x, w, b):
    """2x2 stride-2 transposed convolution with w [2, 2, co, C]."""
    N, H, W, C = x.shape
    co = w.shape[2]
    rows = []
    for dy in range(2):
        cols = [(x.reshape(-1, C) @ w[dy, dx].t() + b).view(N, H, W, co) for dx in range(2)]
        rows.append(torch.stack(cols, 3).view(N, H, 2 * W, co))
    return torch.stack(rows, 2).view(N, 2 * H, 2 * W, co)


def _network(p, img, levels: int):
    """The fill network's residual [N, H, W, 3] in 64 bits."""
    at = 0

    def take(*shape):
        nonlocal at
        n = math.prod(shape)
        at += n
        return p[at - n:at].view(shape)

    def conv(x, co):
        w = take(co, 3, 3, x.shape[3])
        return torch.relu(_conv3(x, w, take(co)))

    c = img.rgba
    cov = img.cov != 0
    chans = [((c >> (8 * k)) & 0xFF).double() / 255.0 for k in range(4)]
    chans += [torch.where(cov, img.depth.double() - 1.0, torch.zeros_like(chans[0])), cov.double()]
    x = torch.stack(chans, 3)
    ch = [32 << l for l in range(levels)]
    skips = []
    for l in range(levels):
        x = conv(conv(x, ch[l]), ch[l])
        if l + 1 < levels:
            skips.append(x)
            x = torch.nn.functional.max_pool2d(x.permute(0, 3, 1, 2), 2).permute(0, 2, 3, 1)
    for l in reversed(range(levels - 1)):
        w = take(2, 2, ch[l], ch[l + 1])
        x = torch.cat([_up2(x, w, take(ch[l])), skips[l]], 3)
        x = conv(conv(x, ch[l]), ch[l])
    w = take(3, ch[0])
    return x @ w.t() + take(3)


def exact(case: dict, seed: int):
    """Network outputs in 64 bits. The other cases give integers and their
    float outputs copies or fixed orders of single fp32 operations on them."""
    if case["op"] not in ("fill", "train"):
        return None
    st = prepare(case, seed)
    p = st["params"].double()
    if case["op"] == "fill":
        with torch.no_grad():
            # one image at a time keeps the 64-bit activations small
            img = st["img"]
            res = [_network(p, lf.SplatImages(img.rgba[i:i + 1], img.depth[i:i + 1], img.cov[i:i + 1]), case["levels"])
                   for i in range(case["images"])]
        return {"rgba": None, "residual": torch.cat(res)}
    p.requires_grad_(True)
    res = _network(p, st["img"], case["levels"])
    rgb = lambda t: torch.stack([((t >> (8 * k)) & 0xFF).double() / 255.0 for k in range(3)], 3)
    loss = (rgb(st["img"].rgba) + res - rgb(st["target"])).square().mean()
    loss.backward()
    return {"loss": loss.detach().view(1), "grad": p.grad}
