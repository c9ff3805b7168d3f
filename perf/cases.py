"""The work whose speed is measured: what a program that uses this package has it do.

``listed`` gives the fixed cases, ``draw`` more of the same ranges, ``prepare``
what a program holds before the call (inputs from a seed, device buffers,
image-based-lighting tables, plans), ``run`` one pass through the public entry
points, ``work`` the bytes and operations a pass cannot do without, and
``exact`` the computed outputs in 64 bits by plain torch arithmetic, written
here from the definitions in ``include/epb.h``.

Kinds of case:
  frame    a whole frame (SSAO, shading, bloom and tone mapping) of one view
  batch    many views of several scenes rendered together
  ibl      the image-based-lighting tables of a new environment
  gbuffer  the G-buffer of a sphere field from a new camera
  shadows  the depth maps of every light after the geometry moved
  edl      eye-dome lighting of a point cloud, bloom and tone mapping
"""
import math

import numpy as np
import torch

from paper_2012_03325_amd import epb as E
from paper_2012_03325_amd import frame, synth

_IBL = dict(irr_size=32, irr_src_size=64, pref_size=128, pref_levels=5, pref_samples=1024, lut_size=256,
            lut_samples=1024, pref_fis=0)


def _frame(width, height, spheres=512, plane=True, lights=4, shadow=2048, layout=E.EPB_MAP_TILES, env=512, ssao=64,
           half=False, fused=False, surfel=False, levels=6, tonemap=E.EPB_TONEMAP_ACES):
    return dict(kind="frame", width=width, height=height, spheres=spheres, plane=plane, lights=lights, shadow=shadow,
                layout=layout, env=env, ssao=ssao, half=half, fused=fused, surfel=surfel, levels=levels,
                tonemap=tonemap)


def listed():
    cases = [
        # the smallest interactive view: one light, no depth maps; a frame is a handful of short launches
        dict(_frame(256, 256, spheres=64, plane=False, lights=1, shadow=0, env=64, ssao=16), name="frame-256x256"),
        # the benchmark's frame
        dict(_frame(1920, 1080), name="frame-1080p"),
        # a display-sized frame in half storage through the fused call
        dict(_frame(3840, 2160, half=True, fused=True), name="frame-2160p-half-fused"),
        # a resized window: odd sizes, surfel weights, all eight lights, row-major odd depth maps, Reinhard
        dict(_frame(1003, 667, spheres=200, lights=8, shadow=777, layout=E.EPB_MAP_ROWS, env=256, ssao=31,
                    surfel=True, levels=5, tonemap=E.EPB_TONEMAP_REINHARD), name="frame-1003x667-surfel"),
        # the server's batches: views of mixed sizes over a few scenes, half storage
        dict(kind="batch", views=16, scenes=4, largest=1920, env=256, ssao=16, half=True, fused=False,
             name="batch-16-half"),
        # a new environment at the benchmark's settings
        dict(_IBL, kind="ibl", env=512, name="ibl-512"),
        # a thumbnail sky with small tables, filtered sampling
        dict(_IBL, kind="ibl", env=64, irr_size=16, pref_size=64, pref_levels=4, pref_samples=256, lut_size=64,
             lut_samples=256, pref_fis=1, name="ibl-64-filtered"),
        # the frame's geometry pass when the camera moves
        dict(kind="gbuffer", width=1920, height=1080, spheres=512, plane=True, half=False, name="gbuffer-1080p"),
        # a particle field: many small spheres, half storage
        dict(kind="gbuffer", width=1280, height=720, spheres=16384, plane=True, half=True,
             name="gbuffer-720p-particles"),
        # an object moved: the four lights' depth maps are rendered and tiled again
        dict(kind="shadows", size=2048, lights=4, spheres=512, plane=True, name="shadows-4x2048"),
        # a point cloud at the benchmark's size
        dict(kind="edl", width=1920, height=1080, radius=2, dirs=8, half=False, ao=True, env=64, name="edl-1080p"),
        # a point cloud in a small odd window with wide outlines, half storage
        dict(kind="edl", width=801, height=599, radius=7, dirs=16, half=True, ao=False, env=32,
             name="edl-801x599-half"),
    ]
    return cases


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["frame", "frame", "frame", "batch", "ibl", "gbuffer", "shadows", "edl"])
    if kind in ("frame", "gbuffer", "edl"):
        width, height = _log_int(rng, 64, 2560), _log_int(rng, 64, 1600)
    if kind == "frame":
        lights = rng.choice([0, 1, 2, 4, 8])
        return _frame(width, height, spheres=_log_int(rng, 64, 1024), plane=rng.random() < 0.75, lights=lights,
                      shadow=rng.choice([0, _log_int(rng, 256, 2048)]) if lights else 0,
                      layout=rng.choice([E.EPB_MAP_TILES, E.EPB_MAP_TILES, E.EPB_MAP_ROWS]),
                      env=rng.choice([32, 64, 128, 256, 512]), ssao=_log_int(rng, 8, 64), half=rng.random() < 0.5,
                      fused=rng.random() < 0.5, surfel=width * height < 1000000 and rng.random() < 0.25,
                      levels=rng.choice([4, 5, 6, 6]), tonemap=rng.choice([E.EPB_TONEMAP_ACES, E.EPB_TONEMAP_REINHARD]))
    if kind == "batch":
        return dict(kind="batch", views=rng.randint(2, 16), scenes=rng.randint(1, 4),
                    largest=rng.choice([320, 640, 1280, 1920]), env=rng.choice([64, 128, 256]),
                    ssao=rng.choice([16, 32]), half=rng.random() < 0.6, fused=rng.random() < 0.4)
    if kind == "ibl":
        env = rng.choice([32, 64, 128, 256, 512])
        base = rng.choice([s for s in (32, 64, 128) if s <= env])
        return dict(_IBL, kind="ibl", env=env, irr_size=rng.choice([16, 24, 32]), irr_src_size=rng.choice([32, 64]),
                    pref_size=base, pref_levels=rng.randint(3, min(5, base.bit_length() - 1)),
                    pref_samples=_log_int(rng, 128, 1024), lut_size=rng.choice([64, 100, 128, 256]),
                    lut_samples=_log_int(rng, 128, 1024), pref_fis=rng.choice([0, 0, 1]))
    if kind == "gbuffer":
        return dict(kind="gbuffer", width=width, height=height, spheres=_log_int(rng, 32, 16384),
                    plane=rng.random() < 0.75, half=rng.random() < 0.5)
    if kind == "shadows":
        return dict(kind="shadows", size=_log_int(rng, 256, 2048), lights=rng.randint(1, 4),
                    spheres=_log_int(rng, 64, 1024), plane=rng.random() < 0.75)
    return dict(kind="edl", width=width, height=height, radius=rng.randint(1, 8), dirs=rng.choice([4, 8, 12, 16]),
                half=rng.random() < 0.5, ao=rng.random() < 0.6, env=rng.choice([32, 64, 128]))


# ---------------------------------------------------------------------------
# inputs (host), from the seed alone
# ---------------------------------------------------------------------------
def _field(rng, n, plane):
    """A sphere field; beyond 1024 spheres (a particle field) the radii shrink so that the covered area stays."""
    scene = synth.make_spheres(rng, n, plane)
    if n > 1024:
        scene.radii = scene.radii * math.sqrt(1024.0 / n)
        scene.centers[:, 1] = rng.uniform(0.0, 1.0, n)
    return scene


def _sky(rng, size):
    """A sky with a sun at the benchmark's radiances, or (small cubes) the plain gradient under a seeded tint."""
    if size <= 64:
        env = synth.env_sky_gradient(size)
        env[..., :3] *= rng.uniform(0.6, 1.0, 3).astype(np.float32)
        return env, 40.0, 1.0
    az, el = rng.uniform(0.0, 2.0 * math.pi), math.radians(rng.uniform(20.0, 70.0))
    sun = (math.cos(el) * math.cos(az), math.sin(el), math.cos(el) * math.sin(az))
    return synth.env_sky_sun(size, sun_dir=sun, sky_tint=tuple(rng.uniform(0.6, 1.0, 3))), 1500.0, 0.012


def _light_cams(rng, n, size):
    """Positions on a seeded ring around the origin and, for size > 0, the depth maps' cameras."""
    turn, out = rng.uniform(0.0, 2.0 * math.pi), []
    for k in range(n):
        a = turn + 2.0 * math.pi * k / n
        pos = np.array([6.0 * math.cos(a), 6.0 - 0.4 * (k % 4), 6.0 * math.sin(a)])
        pos = pos.astype(np.float32).astype(np.float64)
        cam = synth.look_at(pos, (0.0, 0.0, 0.0), (0.0, 1.0, 0.0), 90.0, size, size) if size else None
        out.append((pos, cam))
    return out


def _frame_view(case, seed):
    rng = np.random.default_rng(seed)
    scene = _field(rng, case["spheres"], case["plane"])
    cam = synth.orbit_camera(rng, case["width"], case["height"])
    env, intensity, exposure = _sky(rng, case["env"])
    lights = []
    for k, (pos, lcam) in enumerate(_light_cams(rng, case["lights"], case["shadow"])):
        colour = np.ones(3) if k < 4 else rng.uniform(0.3, 1.0, 3)
        light = synth.Light(pos, colour, intensity)
        if lcam is not None:
            light.shadow_cam = lcam
            light.shadow_map = synth.raycast(scene, lcam, depth_only=True)["depth"]
        lights.append(light)
    view = synth.ViewInputs("view", cam, synth.raycast(scene, cam), lights, env,
                            synth.ssao_kernel(rng, case["ssao"]), synth.ssao_noise(rng))
    view.exposure = exposure
    view.tonemap = case["tonemap"]
    base = min(128, case["env"])
    view.ibl = dict(_IBL, pref_size=base, irr_src_size=min(64, case["env"]),
                    pref_levels=min(5, base.bit_length() - 1))
    if case["surfel"]:
        view = synth.surfel_accumulate(view, seed + 1)
    return view


_BATCH_SIZES = ((1920, 1080), (1280, 720), (640, 480), (320, 240))


def _batch_views(case, seed):
    """Views of every size up to the largest one in turn, scenes and cameras from the seed."""
    rng = np.random.default_rng(seed)
    sizes = [s for s in _BATCH_SIZES if s[0] <= case["largest"]]
    scenes = [synth.make_scene(int(rng.integers(0, 1 << 30)), case["env"], case["ssao"]) for _ in range(case["scenes"])]
    views = []
    for k in range(case["views"]):
        w, h = sizes[k % len(sizes)]
        s = k % len(scenes)
        views.append(synth.scene_view(scenes[s], synth.orbit_camera(rng, w, h), f"view{k}", index=s))
    return views


def _gbuffer_scene(case, seed):
    rng = np.random.default_rng(seed)
    scene = _field(rng, case["spheres"], case["plane"])
    return scene, synth.orbit_camera(rng, case["width"], case["height"])


def _shadow_scene(case, seed):
    rng = np.random.default_rng(seed)
    scene = _field(rng, case["spheres"], case["plane"])
    return scene, [c for _, c in _light_cams(rng, case["lights"], case["size"])]


def _cloud(case, seed):
    """The depth and colour planes of a one-pixel point cloud: the surface under about 40 % of the pixels."""
    rng = np.random.default_rng(seed)
    W, H = case["width"], case["height"]
    cam = synth.orbit_camera(rng, W, H)
    g = synth.raycast(_field(rng, 512, True), cam)
    keep = (rng.random((H, W), np.float32) < 0.4) & np.isfinite(g["depth"])
    depth = np.where(keep, g["depth"], np.float32(np.inf))
    color = np.where(keep, g["albedo"], np.float32(0.0))
    ao = (0.3 + 0.7 * rng.random(((H + 1) // 2, (W + 1) // 2), np.float32)).astype(np.float32)
    env = synth.env_sky_gradient(case["env"])
    env[..., :3] *= rng.uniform(0.6, 1.0, 3).astype(np.float32)
    pc = synth.PointCloudView("cloud", cam, depth, color, env, ao)
    pc.edl_radius, pc.edl_dirs = case["radius"], case["dirs"]
    return pc


def _types(case):
    t = E.EPB_F16 if case["half"] else E.EPB_F32
    return dict(gdtype=t, ao_dtype=t, hdr_dtype=t)


# ---------------------------------------------------------------------------
# what a program holds before the call
# ---------------------------------------------------------------------------
def prepare(case, seed):
    kind = case["kind"]
    if kind == "frame":
        view = _frame_view(case, seed)
        ibl = frame.DeviceIBL(view.env, **view.ibl)
        ibl.precompute()
        dv = frame.DeviceView(view, ibl, bloom_levels=case["levels"], shadow_layout=case["layout"], **_types(case))
        return dict(kind=kind, view=dv, fused=case["fused"])
    if kind == "batch":
        views = _batch_views(case, seed)
        ibls = {}
        for v in views:
            if v.scene not in ibls:
                ibls[v.scene] = frame.DeviceIBL(v.env, **v.ibl)
                ibls[v.scene].precompute()
        dvs = [frame.DeviceView(v, ibls[v.scene], solo_scratch=False, **_types(case)) for v in views]
        schedule = frame.make_schedule(fuse_bloom=1 if case["fused"] else 0)
        return dict(kind=kind, batch=frame.DeviceBatch(dvs, schedule), views=dvs)
    if kind == "ibl":
        env, _, _ = _sky(np.random.default_rng(seed), case["env"])
        return dict(kind=kind, ibl=frame.DeviceIBL(env, **{k: case[k] for k in _IBL}))
    if kind == "gbuffer":
        scene, cam = _gbuffer_scene(case, seed)
        return dict(kind=kind, scene=frame.DeviceScene(scene), cam=cam,
                    dtype=E.EPB_F16 if case["half"] else E.EPB_F32)
    if kind == "shadows":
        scene, cams = _shadow_scene(case, seed)
        ds = frame.DeviceScene(scene)
        return dict(kind=kind, scene=ds, cams=cams, cache=frame.ShadowCache(ds, tiles=True))
    pc = _cloud(case, seed)
    t = E.EPB_F16 if case["half"] else E.EPB_F32
    edl = frame.DeviceEDL(pc, color_dtype=t, ao_dtype=t, hdr_dtype=t, use_ao=case["ao"])
    return dict(kind=kind, edl=edl, post=frame.DevicePost(pc.cam.width, pc.cam.height, pyr_dtype=t))


def run(state):
    kind = state["kind"]
    if kind == "frame":
        dv = state["view"]
        dv.render(fused=state["fused"])
        return dict(ao=dv.ao, hdr=dv.hdr, ldr=dv.ldr)
    if kind == "batch":
        state["batch"].render()
        return [dict(ao=dv.ao, hdr=dv.hdr, ldr=dv.ldr) for dv in state["views"]]
    if kind == "ibl":
        ibl = state["ibl"]
        ibl.precompute()
        return dict(irradiance=ibl.irr, prefiltered=ibl.pref, lut=ibl.lut)
    if kind == "gbuffer":
        return state["scene"].render_gbuffer(state["cam"], state["dtype"])
    if kind == "shadows":
        state["scene"].move()  # the geometry changed: every depth map is stale
        return state["cache"].maps(state["cams"])
    state["edl"].run()
    state["post"].run(state["edl"].hdr)
    return dict(hdr=state["edl"].hdr, ldr=state["post"].ldr)


# ---------------------------------------------------------------------------
# bytes and operations of one pass
# ---------------------------------------------------------------------------
def _view_work(W, H, half, lights, shadow, ssao, surfel=False, env=0):
    px = W * H
    e = 2 if half else 4
    b = px * (4 + 8 * e + (e if surfel else 0)) + px // 4 * e + px * 3 * e + px * 4  # G-buffer, AO, HDR, LDR
    b += lights * min(shadow * shadow, 9 * px) * 4 + 6 * env * env * 16
    return b, px * (ssao / 4 * 30 + lights * 90 + 350)


def work(case):
    kind = case["kind"]
    if kind == "frame":
        b, f = _view_work(case["width"], case["height"], case["half"], case["lights"], case["shadow"], case["ssao"],
                          case["surfel"], 32)
    elif kind == "batch":
        sizes = [s for s in _BATCH_SIZES if s[0] <= case["largest"]]
        each = [_view_work(*sizes[k % len(sizes)], case["half"], 1, 0, case["ssao"]) for k in range(case["views"])]
        b, f = sum(x[0] for x in each), sum(x[1] for x in each)
    elif kind == "ibl":
        S, irr = case["env"], 6 * case["irr_size"] ** 2
        base = min(S, case["pref_size"])
        texels = [6 * (base >> m) ** 2 for m in range(case["pref_levels"])]
        b = 6 * S * S * 16 + irr * 16 + sum(texels) * 16 + case["lut_size"] ** 2 * 8
        f = (irr * 6 * min(S, case["irr_src_size"]) ** 2 * 14 + sum(texels[1:]) * case["pref_samples"] * 60 +
             case["lut_size"] ** 2 * case["lut_samples"] * 25)
    elif kind == "gbuffer":
        px = case["width"] * case["height"]
        b = px * (4 + 8 * (2 if case["half"] else 4)) + case["spheres"] * 52
        f = px * 60
    elif kind == "shadows":
        px = case["size"] ** 2 * case["lights"]
        b = px * 4 + px * 64 / 36 * 4 + case["spheres"] * 32  # the map, and its tiled copy of 64 floats to 36 texels
        f = px * 60
    else:
        px = case["width"] * case["height"]
        e = 2 if case["half"] else 4
        b = px * (4 + 3 * e + 3 * e + 4) + (px // 4 * e if case["ao"] else 0) + 6 * case["env"] ** 2 * 16
        f = px * (case["dirs"] * 3 + 120)
    return dict(bytes=float(b), flops=float(f))


# ---------------------------------------------------------------------------
# 64-bit values of the computed outputs
# ---------------------------------------------------------------------------
def _dev(a, half=False):
    t = torch.from_numpy(np.ascontiguousarray(a)).cuda()
    return (t.half() if half else t).double()


def _grid(W, H):
    y, x = torch.meshgrid(torch.arange(H, device="cuda"), torch.arange(W, device="cuda"), indexing="ij")
    return x, y


def _unit(v):
    return v / v.pow(2).sum(0, keepdim=True).sqrt()


def _dot(a, b):
    return (a * b).sum(0)


def _texel_dirs(S):
    """Unit directions [3][6 S S] of the texels of a cube of face size S."""
    c = (2.0 * torch.arange(S, device="cuda", dtype=torch.float64) + 1.0) / S - 1.0
    t, s = torch.meshgrid(c, c, indexing="ij")
    o = torch.ones_like(s)
    f = [(o, -t, -s), (-o, -t, s), (s, o, t), (s, -o, -t), (s, -t, o), (-s, -t, -o)]
    return _unit(torch.stack([torch.stack([x.reshape(-1) for x in v]) for v in f], 1).reshape(3, -1))


def _solid_angles(S):
    """Solid angles [6 S S] of the texels of a cube of face size S."""
    e = 2.0 * torch.arange(S + 1, device="cuda", dtype=torch.float64) / S - 1.0
    y, x = torch.meshgrid(e, e, indexing="ij")
    a = torch.atan2(x * y, (x * x + y * y + 1.0).sqrt())
    return (a[1:, 1:] - a[1:, :-1] - a[:-1, 1:] + a[:-1, :-1]).reshape(-1).repeat(6)


def _faces(d):
    """Face index and in-face coordinates of directions [3][n] (major axis, ties z, then y, then x)."""
    x, y, z = d[0], d[1], d[2]
    ax, ay, az = x.abs(), y.abs(), z.abs()
    on_z = (az >= ax) & (az >= ay)
    on_y = ~on_z & (ay >= ax)
    face = torch.where(on_z, 4 + (z < 0).long(), torch.where(on_y, 2 + (y < 0).long(), (x < 0).long()))
    m = torch.where(on_z, az, torch.where(on_y, ay, ax))
    sx, sz = torch.where(x < 0, z, -z), torch.where(z < 0, -x, x)
    s = torch.where(on_z, sz, torch.where(on_y, x, sx)) / m
    t = torch.where(on_y & (y >= 0), z, torch.where(on_y, -z, -y)) / m
    return face, s, t


def _bilinear(cube, face, s, t):
    """Bilinear lookup [n][3] of cube [6][S][S][3], clamped to the face."""
    S = cube.shape[1]
    x = ((s * 0.5 + 0.5) * S - 0.5).clamp(0, S - 1)
    y = ((t * 0.5 + 0.5) * S - 0.5).clamp(0, S - 1)
    x0, y0 = x.long().clamp(max=S - 2), y.long().clamp(max=S - 2)
    wx, wy = (x - x0)[:, None], (y - y0)[:, None]
    q = (face * S + y0) * S + x0
    c = cube.reshape(-1, 3)
    top = c[q] + wx * (c[q + 1] - c[q])
    bot = c[q + S] + wx * (c[q + S + 1] - c[q + S])
    return top + wy * (bot - top)


def _halve(cube):
    S = cube.shape[1]
    w = _solid_angles(S).reshape(6, S, S, 1)
    n = lambda a: a.reshape(6, S // 2, 2, S // 2, 2, -1).sum((2, 4))  # noqa: E731
    return n(cube * w) / n(w)


def _hammersley(n):
    k = torch.arange(n, device="cuda", dtype=torch.int64)
    r, v = torch.zeros(n, dtype=torch.float64, device="cuda"), k.clone()
    for b in range(20):
        r += (v & 1).double() * 0.5 ** (b + 1)
        v >>= 1
    return k.double() / n, r


def _ggx(n, alpha):
    """Tangent-frame half vectors [n] (x, y, z) of the sample set."""
    u1, u2 = _hammersley(n)
    a2 = alpha * alpha
    den = (1.0 - u2) + a2 * u2
    ct, st = ((1.0 - u2) / den).sqrt(), (a2 * u2 / den).sqrt()
    return st * (2.0 * math.pi * u1).cos(), st * (2.0 * math.pi * u1).sin(), ct, den


def _tables(env, p):
    """(irradiance [6][s][s][3], prefiltered levels, table [n][n][2]) of an environment [6][S][S][3]."""
    S = env.shape[1]
    src = env
    while src.shape[1] > p["irr_src_size"]:
        src = _halve(src)
    w = _texel_dirs(src.shape[1])
    dw = _solid_angles(src.shape[1])
    L = torch.cat([src.reshape(-1, 3), torch.ones_like(src.reshape(-1, 3)[:, :1])], 1) * dw[:, None]
    n = _texel_dirs(p["irr_size"])
    e = torch.cat([(n[:, k:k + 512].T @ w).clamp(min=0) @ L for k in range(0, n.shape[1], 512)])
    irr = (e[:, :3] / e[:, 3:]).reshape(6, p["irr_size"], p["irr_size"], 3)
    base, M = min(S, p["pref_size"]), p["pref_levels"]
    chain = [env]
    while p["pref_fis"] and chain[-1].shape[1] > 2:
        chain.append(_halve(chain[-1]))
    pref = []
    for m in range(M):
        sm = base >> m
        n = _texel_dirs(sm)
        alpha = (m / (M - 1)) ** 2 if M > 1 else 0.0
        if alpha == 0.0:
            pref.append(_bilinear(env, *_faces(n)).reshape(6, sm, sm, 3))
            continue
        up = torch.zeros_like(n)
        steep = n[2].abs() >= 0.999
        up[2], up[0] = (~steep).double(), steep.double()
        T = _unit(torch.cross(up, n, dim=0))
        B = torch.cross(n, T, dim=0)
        hx, hy, hz, den = _ggx(p["pref_samples"], alpha)
        lod = torch.zeros_like(den)
        if p["pref_fis"]:
            lod = 0.5 * math.log2(6.0 * S * S * alpha * alpha / p["pref_samples"]) + 1.0 - den.log2()
        lod = lod.clamp(0, len(chain) - 1).tolist()
        acc, wt = torch.zeros(n.shape[1], 3, dtype=torch.float64, device="cuda"), 0.0
        for k, (x, y, z) in enumerate(zip(hx.tolist(), hy.tolist(), hz.tolist())):
            h = T * x + B * y + n * z
            l = h * (2.0 * _dot(n, h)) - n
            nl = _dot(n, l).clamp(min=0)
            f = _faces(l)
            l0 = int(lod[k])
            c = _bilinear(chain[l0], *f)
            if lod[k] > l0:
                c = c + (lod[k] - l0) * (_bilinear(chain[l0 + 1], *f) - c)
            acc, wt = acc + c * nl[:, None], wt + nl
        pref.append((acc / wt[:, None]).reshape(6, sm, sm, 3))
    size = p["lut_size"]
    nov = ((torch.arange(size, device="cuda", dtype=torch.float64) + 0.5) / size)[:, None]
    rows = []
    for j in range(size):
        alpha = ((j + 0.5) / size) ** 2
        _, hy, hz, _ = (v[None, :] for v in _ggx(p["lut_samples"], alpha))
        vh = (1.0 - nov * nov).sqrt() * hy + nov * hz  # (the frame of +z has B = +x)
        nl = (2.0 * vh * hz - nov).clamp(min=0)
        k = alpha / 2.0
        g = nl * vh / (hz * (nl * (1.0 - k) + k) * (nov * (1.0 - k) + k))
        fc = (1.0 - vh) ** 5
        rows.append(torch.stack([((1.0 - fc) * g).mean(1), (fc * g).mean(1)], 1))
    return irr, pref, torch.stack(rows)


def _rgb0(t):
    return torch.cat([t, torch.zeros_like(t[..., :1])], -1)


def _slopes(cam, W, H):
    x, y = (v.double() for v in _grid(W, H))
    return (x + 0.5 - cam.cx) / cam.fx, -(y + 0.5 - cam.cy) / cam.fy


def _ssao(view, depth, normal):
    cam = view.cam
    W, H = cam.width, cam.height
    R = torch.from_numpy(cam.R.copy()).cuda()
    ax, ay = _slopes(cam, W, H)
    d, ax, ay = (v[::2, ::2] for v in (depth, ax, ay))
    Hh, Wh = d.shape
    nv = _unit((R @ normal[:, ::2, ::2].reshape(3, -1)).reshape(3, Hh, Wh))
    i, j = _grid(Wh, Hh)
    nz = _dev(view.ssao_noise)[j % 4, i % 4]
    r = torch.stack([nz[..., 0], nz[..., 1], torch.zeros_like(d)])
    t = _unit(r - nv * _dot(nv, r))
    b = torch.cross(nv, t, dim=0)
    dd = torch.where(torch.isinf(d), torch.ones_like(d), d)
    P = torch.stack([ax * dd, ay * dd, -dd])
    rad, bias = float(np.float32(view.ssao_radius)), float(np.float32(view.ssao_bias))
    occ = torch.zeros_like(d)
    for s in view.ssao_kernel.astype(np.float64).tolist():
        Q = P + rad * (t * s[0] + b * s[1] + nv * s[2])
        zq = -Q[2]
        u = cam.cx + cam.fx * Q[0] / zq
        v = cam.cy - cam.fy * Q[1] / zq
        qi, qj = ((u - 0.5) / 2 + 0.5).floor(), ((v - 0.5) / 2 + 0.5).floor()
        ok = (zq > 0) & (qi >= 0) & (qi < Wh) & (qj >= 0) & (qj < Hh)
        ds = d[qj.clamp(0, Hh - 1).nan_to_num().long(), qi.clamp(0, Wh - 1).nan_to_num().long()]
        w = (rad / (dd - ds).abs()).clamp(0, 1)
        occ += torch.where(ok & (ds <= zq - bias), w * w * (3 - 2 * w), torch.zeros_like(w))
    raw = torch.where(torch.isinf(d), torch.ones_like(d), 1 - occ / len(view.ssao_kernel))
    pad = lambda a, fill: torch.nn.functional.pad(a, (2, 1, 2, 1), value=fill)  # noqa: E731
    dp, ap = pad(d, math.inf), pad(raw, 0.0)
    s = sw = 0.0
    tau = float(np.float32(view.blur_tau))
    for y in range(4):
        for x in range(4):
            q = dp[y:y + Hh, x:x + Wh]
            w = (1 - (q - dd).abs() / (tau * dd)).clamp(min=0)
            s, sw = s + w * ap[y:y + Hh, x:x + Wh], sw + w
    return torch.where(torch.isinf(d), torch.ones_like(d), s / sw)


def _upsampled(ao, W, H):
    x, y = _grid(W, H)
    Hh, Wh = ao.shape
    x0, y0 = x // 2, y // 2
    x1, y1 = (x0 + x % 2).clamp(max=Wh - 1), (y0 + y % 2).clamp(max=Hh - 1)
    wx, wy = (x % 2) * 0.5, (y % 2) * 0.5
    top = ao[y0, x0] + wx * (ao[y0, x1] - ao[y0, x0])
    bot = ao[y1, x0] + wx * (ao[y1, x1] - ao[y1, x0])
    return top + wy * (bot - top)


def _lit(light, Pw):
    """Lit fraction of the 3x3 patch of the light's depth map at world points [3][n]."""
    c = light.shadow_cam
    m = _dev(light.shadow_map)
    h, w = m.shape
    R, t = torch.from_numpy(c.R.copy()).cuda(), torch.from_numpy(c.t.copy()).cuda()
    P = R @ Pw + t[:, None]
    dl = -P[2]
    u, v = c.cx + c.fx * P[0] / dl, c.cy - c.fy * P[1] / dl
    inside = (dl > 0) & (u >= 0) & (u < w) & (v >= 0) & (v < h)
    i, j = (torch.where(inside, q, torch.zeros_like(q)).floor().long() for q in (u, v))
    ref, lit = dl - float(np.float32(light.shadow_bias)), 0.0
    for y in (-1, 0, 1):
        for x in (-1, 0, 1):
            a, b = i + x, j + y
            out = (a < 0) | (a >= w) | (b < 0) | (b >= h)
            lit = lit + (out | (ref <= m[b.clamp(0, h - 1), a.clamp(0, w - 1)])).double()
    return torch.where(inside, lit / 9.0, torch.ones_like(dl))


def _view_exact(view, half, tables):
    """(AO, HDR) of one view."""
    cam, g = view.cam, view.gbuf
    W, H = cam.width, cam.height
    depth = _dev(g["depth"])
    normal, albedo = _dev(g["normal"], half), _dev(g["albedo"], half)
    rough, metal = _dev(g["roughness"], half), _dev(g["metalness"], half)
    ao = _ssao(view, depth, normal)
    R = torch.from_numpy(cam.R.copy()).cuda()
    pos = torch.from_numpy(cam.position.copy()).cuda()[:, None]
    env = _dev(view.env)[..., :3]
    ax, ay = _slopes(cam, W, H)
    hdr = torch.empty(3, H, W, dtype=torch.float64, device="cuda")
    bg = torch.isinf(depth)
    ray = lambda m: R.T @ torch.stack([ax[m], ay[m], -torch.ones_like(ax[m])])  # noqa: E731
    hdr[:, bg] = _bilinear(env, *_faces(ray(bg))).T
    fg = ~bg
    Pr = ray(fg) * depth[fg]
    V, n = _unit(-Pr), _unit(normal[:, fg])
    a, r, mt = albedo[:, fg], rough[fg], metal[fg]
    if g.get("weight") is not None:
        w = _dev(g["weight"], half)[fg]
        w = torch.where(w > 0, w, torch.ones_like(w))
        a, r, mt = a / w, r / w, mt / w
    nvr = _dot(n, V)
    nov = nvr.clamp(1e-4, 1.0)
    F0, cd = 0.04 + mt * (a - 0.04), a * (1 - mt)
    al2, k = r.pow(4), (r + 1).pow(2) / 8
    Lo = torch.zeros_like(a)
    for light in view.lights:
        lv = torch.from_numpy(np.asarray(light.pos, np.float64)).cuda()[:, None] - (Pr + pos)
        d2 = _dot(lv, lv)
        l = lv / d2.sqrt()
        nol = _dot(n, l).clamp(min=0)
        sh = _lit(light, Pr + pos) if light.shadow_map is not None else 1.0
        h = _unit(V + l)
        nh, vh = _dot(n, h), _dot(V, h)
        off = h - n * nh
        D = al2 / (math.pi * (nh * nh * al2 + _dot(off, off)).pow(2))
        vis = 0.25 / ((nol * (1 - k) + k) * (nov * (1 - k) + k))
        F = F0 + (1 - F0) * (1 - vh).pow(5)
        rad = torch.from_numpy(np.asarray(light.color, np.float32).astype(np.float64)).cuda()[:, None]
        Lo += (cd / math.pi + D * vis * F) * rad * float(light.intensity) * (nol * sh / d2)
    irr, pref, lut = tables
    size = lut.shape[0]
    x, y = (nov * size - 0.5).clamp(0, size - 1), (r * size - 0.5).clamp(0, size - 1)
    x0, y0 = x.long().clamp(max=size - 2), y.long().clamp(max=size - 2)
    wx, wy = (x - x0)[:, None], (y - y0)[:, None]
    top = lut[y0, x0] + wx * (lut[y0, x0 + 1] - lut[y0, x0])
    bot = lut[y0 + 1, x0] + wx * (lut[y0 + 1, x0 + 1] - lut[y0 + 1, x0])
    A, B = (top + wy * (bot - top)).T
    Em = _bilinear(irr, *_faces(n)).T
    f = _faces(n * (2 * nvr) - V)
    lod = (r * (len(pref) - 1)).clamp(0, len(pref) - 1)
    P = torch.zeros_like(Em)
    for m, level in enumerate(pref):
        P += _bilinear(level, *f).T * (1 - (lod - m).abs()).clamp(min=0)
    Ems = 1 - (A + B)
    kS = F0 + (torch.maximum(1 - r, F0) - F0) * (1 - nov).pow(5)
    ss = kS * A + B
    Fa = F0 + (1 - F0) / 21
    ms = ss * Fa / (1 - Ems * Fa) * Ems
    up = _upsampled(ao, W, H)[fg]
    hdr[:, fg] = Lo + up * (ss * P + (ms + cd * (1 - ss - ms)) * Em)
    return ao, hdr.clamp(max=65504.0) if half else hdr  # half storage saturates


def _cast(scene, cam, attributes):
    """Nearest hits of a sphere field; depth and, with `attributes`, normal, albedo, roughness and metalness."""
    W, H, n = cam.width, cam.height, len(scene.radii)
    R, o = torch.from_numpy(cam.R.copy()).cuda(), torch.from_numpy(cam.position.copy()).cuda()
    ax, ay = _slopes(cam, W, H)
    d = (R.T @ torch.stack([ax, ay, -torch.ones_like(ax)]).reshape(3, -1)).reshape(3, H, W)
    aa = _dot(d, d)
    depth = torch.full((H, W), math.inf, dtype=torch.float64, device="cuda")
    who = torch.full((H, W), -1, dtype=torch.long, device="cuda")
    vc = scene.centers @ cam.R.T + cam.t
    for q in range(n):
        c, r = scene.centers[q], float(scene.radii[q])
        z = -vc[q, 2] - r
        if z + 2 * r <= 1e-3:
            continue
        x0, x1, y0, y1 = 0, W, 0, H
        if z > 1e-3:  # the sphere's bounding cube lies in front of the camera
            corner = vc[q] + r * np.array([[a, b, e] for a in (-1, 1) for b in (-1, 1) for e in (-1, 1)], np.float64)
            px = cam.cx + cam.fx * corner[:, 0] / -corner[:, 2]
            py = cam.cy - cam.fy * corner[:, 1] / -corner[:, 2]
            x0, x1 = max(int(px.min()) - 2, 0), min(int(px.max()) + 3, W)
            y0, y1 = max(int(py.min()) - 2, 0), min(int(py.max()) + 3, H)
            if x0 >= x1 or y0 >= y1:
                continue
        oc = cam.position - c
        dw, aw = d[:, y0:y1, x0:x1], aa[y0:y1, x0:x1]
        b = dw[0] * oc[0] + dw[1] * oc[1] + dw[2] * oc[2]
        disc = b * b - aw * float(oc @ oc - r * r)
        t = (-b - disc.clamp(min=0).sqrt()) / aw
        near = (disc >= 0) & (t > 0) & (t < depth[y0:y1, x0:x1])
        depth[y0:y1, x0:x1][near] = t[near]
        who[y0:y1, x0:x1][near] = q
    if scene.plane:
        t = -o[1] / d[1]
        near = (d[1] < 0) & (t > 0) & (t < depth)
        depth[near] = t[near]
        who[near] = n
    if not attributes:
        return depth
    pad = lambda a, e: torch.cat([_dev(np.asarray(a, np.float32)), torch.tensor([e], dtype=torch.float64, device="cuda")])  # noqa: E731,E501
    on, hit = (who >= 0) & (who < n), who >= 0
    centre = _dev(scene.centers)[who.clamp(0, n - 1)].permute(2, 0, 1)
    at = torch.where(on, depth, torch.ones_like(depth)) * d + o[:, None, None]
    up = torch.tensor([0.0, 1.0, 0.0], dtype=torch.float64, device="cuda")[:, None, None]
    normal = torch.where(on, _unit(at - centre), torch.where(hit, up, torch.zeros_like(up)))
    k = who.clamp(min=0)
    z = torch.zeros_like(depth)
    albedo = torch.stack([torch.where(hit, pad(np.asarray(scene.albedo)[:, c], scene.plane_albedo[c])[k], z)
                          for c in range(3)])
    rough = torch.where(hit, pad(scene.roughness, float(np.float32(scene.plane_roughness)))[k], z)
    metal = torch.where(hit, pad(scene.metalness, scene.plane_metalness)[k], z)
    return dict(depth=depth, normal=normal, albedo=albedo, roughness=rough, metalness=metal)


def _tiled(m):
    """The tiled form of a depth map [h][w], flat."""
    h, w = m.shape
    ny, nx = -(-h // 6), -(-w // 6)
    full = torch.full((6 * ny + 2, 6 * nx + 2), math.inf, dtype=m.dtype, device=m.device)
    full[1:h + 1, 1:w + 1] = m
    blocks = full.unfold(0, 8, 6).unfold(1, 8, 6).reshape(-1)
    return torch.cat([blocks, torch.full((64,), math.inf, dtype=m.dtype, device=m.device)])


def _edl(pc, half, use_ao):
    W, H = pc.cam.width, pc.cam.height
    d = _dev(pc.depth)
    z = d.clamp(max=float(np.float32(pc.edl_far))).log2()
    r = pc.edl_radius
    zp = torch.nn.functional.pad(z, (r, r, r, r), value=math.inf)
    acc = torch.zeros_like(z)
    away = lambda v: int(math.copysign(math.floor(abs(v) + 0.5 + 1e-9), v))  # noqa: E731
    for k in range(pc.edl_dirs):
        a = 2.0 * math.pi * k / pc.edl_dirs
        x, y = r + away(r * math.cos(a)), r + away(r * math.sin(a))
        acc += (z - zp[y:y + H, x:x + W]).clamp(min=0)
    shade = (-pc.edl_strength / pc.edl_dirs * acc).exp2()
    ax, ay = _slopes(pc.cam, W, H)
    R = torch.from_numpy(pc.cam.R.copy()).cuda()
    bg = torch.isinf(d)
    hdr = _dev(pc.color, half) * shade * (_upsampled(_dev(pc.ao, half), W, H) if use_ao else 1.0)
    ray = R.T @ torch.stack([ax[bg], ay[bg], -torch.ones_like(ax[bg])])
    hdr[:, bg] = _bilinear(_dev(pc.env)[..., :3], *_faces(ray)).T * shade[bg]
    return hdr


def exact(case, seed):
    kind = case["kind"]
    if kind == "frame":
        view = _frame_view(case, seed)
        ao, hdr = _view_exact(view, case["half"], _tables(_dev(view.env)[..., :3], view.ibl))
        return dict(ao=ao, hdr=hdr, ldr=None)
    if kind == "batch":
        tables, out = {}, []
        for v in _batch_views(case, seed):
            if v.scene not in tables:
                tables[v.scene] = _tables(_dev(v.env)[..., :3], dict(v.ibl, pref_fis=0))
            ao, hdr = _view_exact(v, case["half"], tables[v.scene])
            out.append(dict(ao=ao, hdr=hdr, ldr=None))
        return out
    if kind == "ibl":
        env, _, _ = _sky(np.random.default_rng(seed), case["env"])
        irr, pref, lut = _tables(_dev(env)[..., :3], case)
        return dict(irradiance=_rgb0(irr), prefiltered=torch.cat([_rgb0(m).reshape(-1) for m in pref]), lut=lut)
    if kind == "gbuffer":
        scene, cam = _gbuffer_scene(case, seed)
        return _cast(scene, cam, True)
    if kind == "shadows":
        scene, cams = _shadow_scene(case, seed)
        return [_tiled(_cast(scene, c, False)) for c in cams]
    return dict(hdr=_edl(_cloud(case, seed), case["half"], case["ao"]), ldr=None)
