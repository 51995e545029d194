"""Workloads of the volume ray caster whose speed is followed from change to change.

Each case is one call (or one short chain of calls) of the public interface on
inputs of the shapes the scenes, tests and bench.py of this repository use:
`prepare` makes what a program holds before the call, `run` makes the call,
`work` says what the call cannot do without, and `exact` renders the same scene
in 64-bit torch from the definition of the method, without the library.

A case names its contents:
  kind     render | bricks | batch | serve | frame
  content  blob (one FP32 scalar without guard layers), blob1 (one, with a guard
           layer), pic3 (density, |E|, sqrt(2|B|)), pair (pic3 with E switched
           off), four (a scalar and vectors of 2, 3 and 4 components)
  tuned    false: a context as isaac_init leaves it; true: the tile shape the
           tuner's cache holds for these workloads, set for every image size
"""

from __future__ import annotations

import math
import random

import numpy as np
import torch

import paper_1611_09048_amd as isaac

STORAGE = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
# what the tuner's cache holds for three-source frames and for batches of scalars
TUNED_FRAME = (4, 1, 1, 16, 4, 0)
TUNED_BATCH = {7: (8, 4, 1, 4, 0, 1), 8: (8, 2, 1, 4, 0, 1), 9: (16, 1, 1, 4, 0, 1), 10: (8, 1, 1, 4, 0, 1)}
RESOLUTIONS = ((512, 512), (1280, 720), (1920, 1080))
FOVY = 60.0


# ---------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------

def _render(name, dims, content, dtype, width, height, clips=0, interp=1, mode="volume", tuned=True, call="async",
            layout="aos", persistent=True, step=0.5):
    return dict(name=name, kind="render", nx=dims[0], ny=dims[1], nz=dims[2], content=content, dtype=dtype,
                width=width, height=height, clips=clips, interp=interp, mode=mode, tuned=tuned, call=call,
                layout=layout, persistent=persistent, step=step)


def listed():
    return [
        # the first picture: one small scalar, nearest cell, a context nobody tuned, the call waits for its image
        _render("scalar_256", (64, 64, 64), "blob", "f32", 256, 256, interp=0, tuned=False, call="sync"),
        # a program that calls render() as the README does, three fields, no tuning step
        _render("untuned_720p", (128, 128, 128), "pic3", "f32", 1280, 720, tuned=False, call="sync"),
        # the benchmark's frame: a simulation's three fields in place, new every frame
        _render("pic3_1080p", (256, 256, 256), "pic3", "f32", 1920, 1080, clips=2),
        # half-precision fields of a ragged local volume, separate component arrays, ragged window
        _render("half_ragged", (213, 187, 241), "pic3", "f16", 1279, 717, clips=1, layout="soa"),
        # a client has switched one of the three fields off
        _render("pair_720p", (192, 160, 224), "pair", "f32", 1280, 720, clips=1),
        # iso-surfaces of density and |E|
        _render("iso_1080p", (256, 256, 256), "pic3", "f32", 1920, 1080, clips=2, mode="iso"),
        # a caller that may not allocate device memory; fields read in place at every corner
        _render("noalloc_768p", (192, 192, 192), "pic3", "f32", 1024, 768, call="noalloc"),
        # coupled to a running simulation: one field is a scratch buffer copied at every frame
        _render("insitu_1080p", (128, 128, 128), "pic3", "f32", 1920, 1080, call="sync", persistent=False),
        # one node's share of sort-last rendering: eight bricks and their depth-ordered composite
        dict(name="bricks_1080p", kind="bricks", edge=128, width=1920, height=1080, clips=2, step=0.5),
        # many small sub-volumes, each with its own camera, in one call
        dict(name="batch_64", kind="batch", jobs=64, lo=32, hi=192, picks=4),
        # a resident data set explored by several clients, one admitted batch of requests
        dict(name="serve_6", kind="serve", nx=512, ny=512, nz=256, requests=6),
        # the finished frame on its way to the viewer: 8 bits over white, then JPEG
        dict(name="frame_1080p", kind="frame", width=1920, height=1080, quality=90),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    pick = rng.random()
    if pick < 0.10:
        return dict(kind="frame", width=_log_int(rng, 64, 1920), height=_log_int(rng, 48, 1080),
                    quality=rng.randint(50, 95))
    if pick < 0.20:
        return dict(kind="batch", jobs=_log_int(rng, 2, 40), lo=24, hi=rng.randint(60, 180), picks=rng.randint(1, 4))
    if pick < 0.30:
        return dict(kind="serve", nx=_log_int(rng, 96, 512), ny=_log_int(rng, 96, 512), nz=_log_int(rng, 64, 256),
                    requests=rng.randint(1, 6))
    if pick < 0.38:
        return dict(kind="bricks", edge=_log_int(rng, 24, 128), width=_log_int(rng, 256, 1920),
                    height=_log_int(rng, 200, 1080), clips=rng.randint(0, 2), step=0.5)
    dims = tuple(_log_int(rng, 33, 256) for _ in range(3))
    width, height = _log_int(rng, 160, 1920), _log_int(rng, 120, 1080)
    content = rng.choice(("pic3", "pic3", "pic3", "blob", "blob1", "pair", "four"))
    mode = "iso" if content == "pic3" and rng.random() < 0.2 else "volume"
    call = rng.choice(("async", "async", "sync", "noalloc"))
    if call == "noalloc":                    # the calls that fit the static scratch whatever the view
        width, height = min(width, 1024), min(height, 768)
    case = _render("", dims, content, rng.choice(("f32", "f32", "f16", "bf16")), width, height,
                   clips=rng.randint(0, 2), interp=0 if rng.random() < 0.2 else 1, mode=mode,
                   tuned=rng.random() < 0.6, call=call, layout=rng.choice(("aos", "aos", "soa")),
                   persistent=rng.random() < 0.85, step=rng.choice((0.5, 0.5, 0.3, 1.0)))
    del case["name"]
    return case


# ---------------------------------------------------------------------------
# inputs: seeded fields on the device, transfer functions, cameras, planes
# ---------------------------------------------------------------------------

def _centres(n, g):
    return torch.arange(-g, n + g, dtype=torch.float64, device="cuda") + 0.5


def _blobs(rng, gen, dims, g):
    scale = sum(dims) / 3.0 / 64.0
    ax = [_centres(n, g) for n in dims]
    out = torch.zeros([a.numel() for a in reversed(ax)], dtype=torch.float64, device="cuda")
    for _ in range(8):
        sig, amp = rng.uniform(4.0, 12.0) * scale, rng.uniform(0.2, 1.0)
        gx, gy, gz = (torch.exp(-0.5 * ((a - rng.uniform(0, n)) / sig) ** 2) for a, n in zip(ax, dims))
        out += amp * gz[:, None, None] * gy[None, :, None] * gx[None, None, :]
    return (out + 0.01 * torch.rand(out.shape, generator=gen, device="cuda", dtype=torch.float64)).float()[..., None]


def _density(rng, gen, dims, g):
    x, y, z = (_centres(n, g) for n in dims)
    r2 = (x - dims[0] / 2)[None, :] ** 2 + (z - dims[2] / 2)[:, None] ** 2
    R, lam, y0 = rng.uniform(16, 48), rng.uniform(32, 96), rng.uniform(0, dims[1])
    wave = 0.5 * (1 + torch.cos(2 * math.pi * (y - y0) / lam))
    m = 1 - 0.8 * torch.exp(-r2 / (2 * R * R))[:, None, :] * wave[None, :, None]
    noise = torch.randn(m.shape, generator=gen, device="cuda")
    return (torch.exp(noise) * m.float())[..., None]


def _waves(rng, dims, g, comps=3):
    x, y, z = (_centres(n, g) for n in dims)
    out = torch.zeros((z.numel(), y.numel(), x.numel(), comps), dtype=torch.float32, device="cuda")
    for _ in range(4):
        k = np.array([rng.gauss(0, 1) for _ in range(3)])
        k /= np.linalg.norm(k)
        e = np.array([rng.gauss(0, 1) for _ in range(3)])
        e -= (e @ k) * k
        e = np.resize(e / np.linalg.norm(e), comps)
        k *= 2 * math.pi / rng.uniform(16, 128)
        ph = (k[0] * x)[None, None, :] + (k[1] * y)[None, :, None] + (k[2] * z)[:, None, None] + rng.uniform(0, 6.3)
        s = (rng.uniform(0.05, 0.25) * torch.sin(ph)).float()
        for c in range(comps):
            out[..., c] += float(e[c]) * s
    return out


def _tf(rng, points):
    xs = [0] + sorted(rng.sample(range(1, 255), points - 2)) + [255]
    return [(x / 255, rng.random(), rng.random(), rng.random(), rng.uniform(0, 0.03)) for x in xs]


def _direction(rng):
    d = np.array([rng.gauss(0, 1) for _ in range(3)])
    return d / np.linalg.norm(d)


def _camera(dims, direction):
    c = np.array(dims, dtype=np.float64) / 2
    return dict(eye=tuple(c + 2 * math.sqrt(sum(n * n for n in dims)) * direction), center=tuple(c), up=(0.0, 0.0, 1.0))


def _plane(rng, dims):
    n = _direction(rng)
    q = [s / 4 + rng.random() * s / 2 for s in dims]
    d = -float(n @ q)
    if float(n @ (np.array(dims) / 2)) + d < 0:
        n, d = -n, -d
    return (float(n[0]), float(n[1]), float(n[2]), d)


def _sources(rng, gen, content, dims, dtype):
    """One dict per source: stored values [z][y][x][c], guard layers, chain, table points, weight, iso value."""
    nan = float("nan")
    if content in ("blob", "blob1"):
        g = 0 if content == "blob" else 1
        fields = [(_blobs(rng, gen, dims, g), g, "", nan)]
    elif content == "four":
        fields = [(_density(rng, gen, dims, 1), 1, "mul(0.5)", nan),
                  (_waves(rng, dims, 1, 2), 1, "add(0.2) | sum", nan),
                  (_waves(rng, dims, 1, 3), 1, "length", nan),
                  (_waves(rng, dims, 1, 4), 1, "mul(1.5,1,1,0.5) | length | pow(0.5)", nan)]
    else:
        fields = [(_density(rng, gen, dims, 1), 1, "", 1.0),
                  (_waves(rng, dims, 1), 1, "length", 0.2),
                  (_waves(rng, dims, 1), 1, "length | mul(2) | pow(0.5)", nan)]
    n = 4 if content in ("blob", "blob1") else 8
    return [dict(values=v.to(STORAGE[dtype]), guard=g, chain=ch, iso=iso, tf=_tf(rng, n),
                 weight=1.0 if n == 4 else float(np.float32(rng.uniform(0.3, 1.0))),
                 enabled=not (content == "pair" and k == 1))
            for k, (v, g, ch, iso) in enumerate(fields)]


def _scene(case, seed):
    """A render case's inputs: dims, sources, camera, clipping planes."""
    rng = random.Random(seed)
    gen = torch.Generator(device="cuda").manual_seed(seed)
    dims = (case["nx"], case["ny"], case["nz"])
    src = _sources(rng, gen, case["content"], dims, case["dtype"])
    return dict(dims=dims, src=src, cam=_camera(dims, _direction(rng)),
                clip=[_plane(rng, dims) for _ in range(case["clips"])])


def _store(values, layout):
    """The field as a simulation holds it: rows padded to 256 bytes; (buffers, component addresses of array
    element (0,0,0), byte strides along x, y, z)."""
    nz, ny, nx, c = values.shape
    es = values.element_size()
    parts = [values] if layout == "aos" else [values[..., k:k + 1] for k in range(c)]
    bufs, comp, per = [], [], parts[0].shape[3]
    row = -(-nx * per * es // 256) * 256 // es
    for p in parts:
        b = torch.zeros((nz, ny, row), dtype=values.dtype, device="cuda")
        b[:, :, :nx * per] = p.reshape(nz, ny, nx * per)
        bufs.append(b)
        comp += [b.data_ptr() + k * es for k in range(per)]
    return bufs, comp, (per * es, row * es, row * es * ny)


def _define(ctx, vid, dims, src, layout="aos", persistent=True):
    """Register a volume's sources and transfer functions; returns the buffers to keep."""
    keep, descs = [], []
    for k, s in enumerate(src):
        dtype = next(n for n, t in STORAGE.items() if t == s["values"].dtype)
        bufs, comp, stride = _store(s["values"], layout)
        keep += bufs
        o = s["guard"] * sum(stride)
        descs.append(isaac.source_desc(name=f"s{k}", f_dim=s["values"].shape[3], dtype=dtype,
                                       comp=[c + o for c in comp], stride=stride, guard=s["guard"],
                                       chain=s["chain"], weight=s["weight"], enabled=s["enabled"],
                                       persistent=persistent or k != len(src) - 1))
    torch.cuda.synchronize()
    ctx.set_sources(vid, dims, descs)
    for k, s in enumerate(src):
        ctx.set_transfer(vid, k, s["tf"])
    return keep


def _context(tuned, **kw):
    ctx = isaac.Context(device=0, **kw)
    if tuned:
        for cls in range(16):
            ctx.set_tile_shape(cls, *(tuned.get(cls, TUNED_BATCH[8]) if isinstance(tuned, dict) else TUNED_FRAME))
    return ctx


def _image(width, height):
    return torch.zeros((height, width, 4), device="cuda")


def _batch_jobs(case):
    """Sizes of a batch's sub-volumes and images (part of the case, the same for every seed)."""
    rng = random.Random(case["jobs"])
    sizes = (128, 256, 512, 1024)[:case["picks"]]
    return [(tuple(rng.randint(case["lo"], case["hi"]) for _ in range(3)), rng.choice(sizes))
            for _ in range(case["jobs"])]


def _batch_scenes(case, seed):
    rng = random.Random(seed)
    gen = torch.Generator(device="cuda").manual_seed(seed)
    return [dict(dims=dims, src=_sources(rng, gen, "blob1", dims, "f32"), cam=_camera(dims, _direction(rng)), size=size)
            for dims, size in _batch_jobs(case)]


def _serve_scene(case, seed):
    rng = random.Random(seed)
    gen = torch.Generator(device="cuda").manual_seed(seed)
    dims = (case["nx"], case["ny"], case["nz"])
    src = _sources(rng, gen, "pic3", dims, "f32")
    reqs = [dict(size=RESOLUTIONS[k % 3], cam=_camera(dims, _direction(rng)),
                 clip=[_plane(rng, dims)] if k % 2 else []) for k in range(case["requests"])]
    return dims, src, reqs


def _brick_scene(case, seed):
    n = 2 * case["edge"]
    return _scene(dict(nx=n, ny=n, nz=n, content="pic3", dtype="f32", clips=case["clips"]), seed)


# ---------------------------------------------------------------------------
# prepare and run
# ---------------------------------------------------------------------------

def prepare(case, seed):
    kind = case["kind"]
    if kind == "frame":
        # a rendered frame: a shaded body over transparent black, premultiplied
        w, h = case["width"], case["height"]
        rng = random.Random(seed)
        y, x = torch.meshgrid(torch.linspace(-1, 1, h, device="cuda"), torch.linspace(-w / h, w / h, w, device="cuda"),
                              indexing="ij")
        a = (1.2 - 2.2 * torch.sqrt(x * x + y * y) + 0.15 * torch.sin(9 * x + rng.uniform(0, 6)) *
             torch.cos(7 * y)).clamp(0, 1)
        rgb = [0.5 + 0.5 * torch.sin(rng.uniform(3, 40) * x + rng.uniform(3, 40) * y + rng.uniform(0, 6))
               for _ in range(3)]
        img = torch.stack([a * c for c in rgb] + [a], dim=-1).contiguous()
        out = torch.zeros((h, w, 4), dtype=torch.uint8, device="cuda")
        message = np.zeros(2 * w * h + 4096, dtype=np.uint8)      # longer than any such stream
        torch.cuda.synchronize()
        return dict(kind=kind, ctx=_context(False), img=img, rgba8=out, message=message, size=(w, h),
                    quality=case["quality"])
    if kind == "batch":
        ctx, keep, jobs, imgs = _context(TUNED_BATCH), [], [], []
        for vid, s in enumerate(_batch_scenes(case, seed)):
            keep += _define(ctx, vid, s["dims"], s["src"])
            imgs.append(_image(s["size"], s["size"]))
            jobs.append(isaac.render_desc(volume_id=vid, width=s["size"], height=s["size"], fovy_deg=FOVY, step=0.5,
                                          interpolation=isaac.TRILINEAR, out_rgba=imgs[-1].data_ptr(), **s["cam"]))
        return dict(kind=kind, ctx=ctx, keep=keep, jobs=jobs, out=imgs)
    if kind == "serve":
        dims, src, reqs = _serve_scene(case, seed)
        ctx = _context(True, mem_budget=256 << 20)
        keep = _define(ctx, 0, dims, src)
        ctx.freeze_volume(0)
        jobs = [isaac.render_desc(volume_id=0, width=r["size"][0], height=r["size"][1], fovy_deg=FOVY, step=0.5,
                                  interpolation=isaac.TRILINEAR, clip=r["clip"], **r["cam"]) for r in reqs]
        return dict(kind=kind, ctx=ctx, keep=keep, jobs=jobs, out=[_image(*r["size"]) for r in reqs])
    if kind == "bricks":
        s, e, w, h = _brick_scene(case, seed), case["edge"], case["width"], case["height"]
        ctx, keep, jobs, imgs, depths = _context(True), [], [], [], []
        for vid, org in enumerate([(x, y, z) for x in (0, e) for y in (0, e) for z in (0, e)]):
            part = [dict(f, values=f["values"][org[2]:org[2] + e + 2, org[1]:org[1] + e + 2, org[0]:org[0] + e + 2])
                    for f in s["src"]]
            keep += _define(ctx, vid, (e, e, e), part)
            imgs.append(_image(w, h))
            depths.append(torch.zeros((h, w), device="cuda"))
            jobs.append(isaac.render_desc(volume_id=vid, width=w, height=h, fovy_deg=FOVY, step=case["step"],
                                          interpolation=isaac.TRILINEAR, clip=s["clip"], ert_threshold=2.0,
                                          out_rgba=imgs[-1].data_ptr(), out_depth=depths[-1].data_ptr(),
                                          brick_origin=org, global_dims=s["dims"], **s["cam"]))
        return dict(kind=kind, ctx=ctx, keep=keep, jobs=jobs, imgs=imgs, depths=depths, out=_image(w, h), size=(w, h))
    s = _scene(case, seed)
    ctx = _context(case["tuned"])
    keep = _define(ctx, 0, s["dims"], s["src"], case["layout"], case["persistent"])
    img = _image(case["width"], case["height"])
    iso = dict(mode=isaac.ISO, iso_values=[f["iso"] for f in s["src"]]) if case["mode"] == "iso" else {}
    job = isaac.render_desc(volume_id=0, width=case["width"], height=case["height"], fovy_deg=FOVY, step=case["step"],
                            interpolation=case["interp"], clip=s["clip"], out_rgba=img.data_ptr(), **s["cam"], **iso)
    torch.cuda.synchronize()
    return dict(kind=kind, ctx=ctx, keep=keep, job=job, out=img, call=case["call"])


class _Owned:
    """A library-owned image, for torch.as_tensor (valid until its ticket is released)."""

    def __init__(self, ptr, shape):
        self.__cuda_array_interface__ = dict(shape=tuple(shape), typestr="<f4", data=(ptr, False), version=2)


def run(state):
    ctx, kind = state["ctx"], state["kind"]
    if kind == "render":
        if state["call"] == "noalloc":
            ctx.render_noalloc([state["job"]], isaac.ASYNC)
        else:
            ctx.render([state["job"]], isaac.ASYNC if state["call"] == "async" else 0)
        return state["out"]
    if kind == "batch":
        ctx.render(state["jobs"], isaac.ASYNC)
        return state["out"]
    if kind == "bricks":
        for job in state["jobs"]:
            ctx.render([job], isaac.ASYNC)
        ctx.composite([t.data_ptr() for t in state["imgs"]], [t.data_ptr() for t in state["depths"]], *state["size"],
                      state["out"].data_ptr(), isaac.ASYNC)
        return state["out"]
    if kind == "serve":
        # admit the requests, take each image when it is complete, give the library its memory back
        tickets = ctx.submit_batch(state["jobs"])
        for t, out in zip(tickets, state["out"]):
            done, ptr = ctx.poll(t)
            while not done:
                done, ptr = ctx.poll(t)
            out.copy_(torch.as_tensor(_Owned(ptr, out.shape), device="cuda"))
        torch.cuda.current_stream().synchronize()      # the copies read the library's images
        for t in tickets:
            ctx.release(t)
        return state["out"]
    w, h = state["size"]
    ctx.encode_rgba8(state["img"].data_ptr(), w, h, state["rgba8"].data_ptr(), (1.0, 1.0, 1.0), isaac.ASYNC)
    data = ctx.encode_jpeg(state["rgba8"].data_ptr(), w, h, state["quality"])
    state["message"][:len(data)] = np.frombuffer(data, dtype=np.uint8)
    return [state["rgba8"], state["message"], len(data)]


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------

def _points(dims, width, height, step, clips):
    """Scan points: cells over the step, times rays per cell cross-section from two diagonals away; a plane
    through the middle half keeps about 0.62 of them."""
    r = 2 * math.sqrt(sum(n * n for n in dims))
    px = height / (2 * r * math.tan(math.radians(FOVY) / 2))
    return dims[0] * dims[1] * dims[2] / step * px * px * 0.62 ** clips


def _voxels(dims, g=1):
    return (dims[0] + 2 * g) * (dims[1] + 2 * g) * (dims[2] + 2 * g)


def work(case):
    kind = case["kind"]
    point = {1: 27 + 41, 2: 27 + 82, 3: 27 + 123, 4: 27 + 164}     # FP32 operations per scan point, trilinear
    if kind == "frame":
        n = case["width"] * case["height"]
        # 16 bytes in, 4 out and in again; colour conversion and two 8-point passes of three components
        return dict(bytes=24 * n, flops=n * (15 + 3 * 2 * 16))
    if kind == "batch":
        b = f = 0
        for dims, size in _batch_jobs(case):
            b += 4 * _voxels(dims) + 16 * size * size
            f += point[1] * _points(dims, size, size, 0.5, 0)
        return dict(bytes=b, flops=f)
    if kind == "serve":
        dims = (case["nx"], case["ny"], case["nz"])
        reqs = [(RESOLUTIONS[k % 3], k % 2) for k in range(case["requests"])]
        return dict(bytes=12 * _voxels(dims) + sum(16 * w * h for (w, h), _ in reqs),
                    flops=sum(point[3] * _points(dims, w, h, 0.5, c) for (w, h), c in reqs))
    if kind == "bricks":
        n = 2 * case["edge"]
        keep = 0.62 ** case["clips"]
        return dict(bytes=28 * _voxels((n, n, n)) * keep + 16 * case["width"] * case["height"],
                    flops=point[3] * _points((n, n, n), case["width"], case["height"], case["step"], case["clips"]))
    dims = (case["nx"], case["ny"], case["nz"])
    comps = {"blob": [1], "blob1": [1], "pic3": [1, 3, 3], "pair": [1, 3], "four": [1, 2, 3, 4]}[case["content"]]
    if case["mode"] == "iso":
        comps = comps[:2]
    es = 4 if case["dtype"] == "f32" else 2
    voxels = _voxels(dims, 0 if case["content"] == "blob" else 1) * 0.62 ** case["clips"]
    pts = _points(dims, case["width"], case["height"], case["step"], case["clips"])
    if case["mode"] == "iso":
        pts /= 20                                                  # a ray ends at its first surface
    return dict(bytes=voxels * sum(comps) * es + 16 * case["width"] * case["height"],
                flops=pts * (point[len(comps)] if case["interp"] else point[len(comps)] - 21 * len(comps)))


# ---------------------------------------------------------------------------
# the method in 64 bits
# ---------------------------------------------------------------------------

def _chain(values, text):
    v = values.double()
    for op in filter(None, (t.strip() for t in text.split("|"))):
        name, _, rest = op.partition("(")
        a = torch.tensor([float(x) for x in rest.rstrip(")").split(",")] if rest else [0.0], dtype=torch.float64,
                         device=v.device)
        if name == "add":
            v = v + a
        elif name == "mul":
            v = v * a
        elif name == "pow":
            v = v ** a
        elif name == "length":
            v = torch.sqrt((v * v).sum(-1, keepdim=True))
        elif name == "sum":
            v = v.sum(-1, keepdim=True)
    return v[..., 0].contiguous()


def _table(points):
    xs, cols = [p[0] for p in points], np.array([p[1:] for p in points])
    t = np.stack([np.interp(np.arange(256) / 255, xs, cols[:, c]) for c in range(4)], axis=1)
    return torch.from_numpy(np.concatenate([t, t[-1:]])).cuda()


def _rays(dims, cam, clip, width, height, step):
    """Rays that keep scan points: pixel, origin, direction, entry, first and end index."""
    eye, centre, up = (np.array(cam[k]) for k in ("eye", "center", "up"))
    fwd = (centre - eye) / np.linalg.norm(centre - eye)
    right = np.cross(fwd, up)
    right /= np.linalg.norm(right)
    upp = np.cross(right, fwd)
    h = math.tan(math.radians(FOVY) / 2)
    f64 = dict(dtype=torch.float64, device="cuda")
    x = (2 * (torch.arange(width, **f64) + 0.5) / width - 1) * h * (width / height)
    y = (1 - 2 * (torch.arange(height, **f64) + 0.5) / height) * h
    vec = [torch.as_tensor(v, **f64) for v in (fwd, right, upp)]
    d = (vec[0] + x[None, :, None] * vec[1] + y[:, None, None] * vec[2]).reshape(-1, 3)
    d = d / d.norm(dim=1, keepdim=True)
    o, hi = torch.as_tensor(eye, **f64), torch.tensor([float(n) for n in dims], **f64)
    ta, tb = -o / d, (hi - o) / d
    t0 = torch.minimum(ta, tb).amax(1).clamp(min=0)
    t1 = torch.maximum(ta, tb).amin(1)
    kb = torch.zeros_like(t0)
    ke = torch.where(t1 > t0, torch.ceil((t1 - t0) / step - 0.5), kb)
    for p in clip:
        n = torch.tensor(p[:3], **f64)
        nd, no = d @ n, float(o @ n) + p[3]
        kc = ((-no / nd - t0) / step - 0.5).clamp(-1, 2e9)
        kb = torch.where(nd > 0, torch.maximum(kb, torch.ceil(kc)), kb)
        ke = torch.where(nd > 0, ke, torch.minimum(ke, torch.floor(kc) + 1))
    pix = torch.nonzero(ke > kb)[:, 0]
    return pix, o, d[pix], t0[pix], kb[pix].long(), ke[pix].long()


def _sample(vol, g, dims, p, interp):
    """Interpolated (or nearest) values of a padded volume [z][y][x] at positions [..., 3]."""
    sz, sy = vol.shape[1] * vol.shape[2], vol.shape[2]
    flat = vol.reshape(-1)

    def at(i):
        return flat[(i[2] + g) * sz + (i[1] + g) * sy + i[0] + g]

    if not interp:
        return at([torch.floor(p[..., a]).long().clamp(0, dims[a] - 1) for a in range(3)])
    lo, hi, w = [], [], []
    for a in range(3):
        u = p[..., a] - 0.5
        f = torch.floor(u)
        w.append(u - f)
        i = f.long()
        b = (0, dims[a] - 1) if g == 0 else (-1, dims[a])
        lo.append(i.clamp(*b))
        hi.append((i + 1).clamp(*b))
    v = 0
    for c in range(8):
        idx = [(hi if c >> a & 1 else lo)[a] for a in range(3)]
        wt = 1
        for a in range(3):
            wt = wt * (w[a] if c >> a & 1 else 1 - w[a])
        v = v + wt * at(idx)
    return v


def _lookup(table, x):
    u = 255 * torch.nan_to_num(x, nan=0.0).clamp(0, 1)
    j = u.long().clamp(max=254)
    f = (u - j)[..., None]
    return table[j] + f * (table[j + 1] - table[j])


def _reference(dims, src, cam, clip, width, height, step, interp=1, mode="volume", ert=0.999):
    src = [s for s in src if s["enabled"] and (mode == "volume" or not math.isnan(s["iso"]))]
    vols = [(_chain(s["values"], s["chain"]), s["guard"], _table(s["tf"]), s) for s in src]
    out = torch.zeros((height * width, 4), dtype=torch.float64, device="cuda")
    pix, o, d, t0, kb, ke = _rays(dims, cam, clip, width, height, step)
    state = torch.zeros((pix.numel(), 4), dtype=torch.float64, device="cuda")
    prev = [torch.zeros(pix.numel(), dtype=torch.float64, device="cuda") for _ in vols]
    live = torch.arange(pix.numel(), device="cuda")
    box = torch.tensor([float(x) for x in dims], dtype=torch.float64, device="cuda")
    k0, n = 0, 8
    while live.numel():
        k = kb[live][:, None] + k0 + torch.arange(n, device="cuda")
        kept = k < ke[live][:, None]
        t = t0[live][:, None] + (k.double() + 0.5) * step
        p = o + t[..., None] * d[live][:, None, :]
        p = torch.minimum(p.clamp(min=0), box)   # points past a ray's end are not used: their reads stay inside
        x = [_sample(v, g, dims, p, interp) for v, g, _, _ in vols]
        done = torch.zeros(live.numel(), dtype=torch.bool, device="cuda")
        st = state[live]
        if mode == "volume":
            S = torch.zeros_like(t)
            E = torch.zeros(t.shape + (3,), dtype=torch.float64, device="cuda")
            for (_, _, table, s), xs in zip(vols, x):
                c = _lookup(table, xs)
                S = S + s["weight"] * c[..., 3]
                E = E + (s["weight"] * c[..., 3])[..., None] * c[..., :3]
            over = S > 1
            E = torch.where(over[..., None], E / S.clamp(min=1)[..., None], E)
            ES = torch.cat([E, S.clamp(max=1)[..., None]], -1)
            for j in range(n):
                use = kept[:, j] & ~done
                st = torch.where(use[:, None], st + (1 - st[:, 3:]) * ES[:, j], st)
                done |= use & (st[:, 3] >= ert)
        else:
            for j in range(n):
                for (v, g, table, s), xs, pr in zip(vols, x, prev):
                    a, b, iso = pr[live] if j == 0 else xs[:, j - 1], xs[:, j], s["iso"]
                    hit = kept[:, j] & ~done & (k[:, j] > kb[live]) & ((a >= iso) != (b >= iso))
                    i = torch.nonzero(hit)[:, 0]
                    if i.numel() == 0:
                        continue
                    ts = t[i, j] - step + (iso - a[i]) / (b[i] - a[i]) * step
                    di = d[live][i]
                    q = o + ts[:, None] * di
                    grad = torch.stack([_sample(v, g, dims, q + e, interp) - _sample(v, g, dims, q - e, interp)
                                        for e in 0.5 * torch.eye(3, dtype=torch.float64, device="cuda")], -1)
                    gl = grad.norm(dim=1)
                    cos = torch.where(gl > 0, (grad * di).sum(1).abs() / gl, torch.ones_like(gl))
                    rgb = _lookup(table, torch.full_like(gl, iso))[:, :3] * (0.3 + 0.7 * cos.clamp(max=1))[:, None]
                    st[i] = torch.cat([rgb, torch.ones_like(gl)[:, None]], 1)
                    done |= hit
            for pr, xs in zip(prev, x):
                pr[live] = xs[:, -1]
        state[live] = st
        k0 += n
        live = live[~done & (kb[live] + k0 < ke[live])]
    out[pix] = state
    return out.reshape(height, width, 4)


def exact(case, seed):
    kind = case["kind"]
    if kind == "frame":
        return None                              # bytes
    if kind == "batch":
        return [_reference(s["dims"], s["src"], s["cam"], [], s["size"], s["size"], 0.5)
                for s in _batch_scenes(case, seed)]
    if kind == "serve":
        dims, src, reqs = _serve_scene(case, seed)
        return [_reference(dims, src, r["cam"], r["clip"], *r["size"], 0.5) for r in reqs]
    if kind == "bricks":
        s = _brick_scene(case, seed)             # the bricks split every ray's scan points without overlap
        return _reference(s["dims"], s["src"], s["cam"], s["clip"], case["width"], case["height"], case["step"],
                          ert=2.0)
    s = _scene(case, seed)
    return _reference(s["dims"], s["src"], s["cam"], s["clip"], case["width"], case["height"], case["step"],
                      case["interp"], case["mode"])
