"""The workloads this library's speed is measured on.

Each case is one call (or one short sequence of calls) a renderer, a server or a
trainer makes through the public binding, over the range such programs use:

* ``query``: one object, one batch of rays (``lsnif_query``).
* ``scene``: world rays against instances (``lsnif_query_scene``), with ``bounces``
  diffuse bounces after it (``lsnif_bounce`` and another scene query each).
* ``serve``: concurrent pair requests through the serving loop.
* ``train``: a training step on an object and reading its parameters and gradients back.

Objects have the shapes of this repository's workloads: ``c1`` (V = 32, 8 levels
of 2**14 x 2), ``c2`` (V = 128, 16 levels of 2**19 x 2), ``paper`` (V = 32, 2
face-aligned levels of 2**17 x 3, width 128, albedo head), ``paper_lq`` (its
low-quality variant) and, in scenes, V 32-256, 8-16 levels, 2**14-2**19 entries.
Occupancy is that of seeded bumpy spheres and tori, tables are uniform in
[-1e-2, 1e-2] and weights Kaiming-normal.
"""

import math
from types import SimpleNamespace

import numpy as np
import torch

from paper_2504_21627_amd import lsnif as L
from paper_2504_21627_amd.serving import RequestSet

DEV = "cuda"
LR = 1e-4   # a late stage's learning rate (the first steps of a fresh Adam move every entry by about this much)
FP8_ACT_SCALE = [2.5e-5, 5e-5, 6.5e-5, 5.5e-5, 5.5e-5]   # as calibrated for these weights, with headroom


def listed():
    return [
        # a picking or visibility probe: the smallest call, all latency
        {"name": "probe_fp16_256", "kind": "query", "shape": "c2", "feat": "fp16", "mlp": "fp16",
         "mix": "primary", "n": 256},
        # the plain FP32 object at its latency batch
        {"name": "latency_fp32_4096", "kind": "query", "shape": "c1", "feat": "fp32", "mlp": "fp32",
         "mix": "sphere", "n": 4096},
        # one 199 x 201 tile of a tiled renderer
        {"name": "tile_fp16_39999", "kind": "query", "shape": "c2", "feat": "fp16", "mlp": "fp16",
         "mix": "primary", "n": 39999},
        # a frame: 1024 x 1024 primary rays and as many shadow rays, with the tuning the
        # autotuner keeps for it
        {"name": "frame_fp16_2m", "kind": "query", "shape": "c2", "feat": "fp16", "mlp": "fp16",
         "mix": "frame", "n": 2097152, "sort_bits": 7, "persistent": 1},
        # half a megapixel at reference precision
        {"name": "frame_fp32_524288", "kind": "query", "shape": "c2", "feat": "fp32", "mlp": "fp32",
         "mix": "frame", "n": 524288},
        # incoherent diffuse bounces at the lowest precision
        {"name": "bounce_fp8_1000003", "kind": "query", "shape": "c2", "feat": "fp16", "mlp": "fp8",
         "mix": "bounce", "n": 1000003, "sort_bits": 7},
        # the paper's default object, a megapixel
        {"name": "paper_fp16_1m", "kind": "query", "shape": "paper", "feat": "fp16", "mlp": "fp16",
         "mix": "sphere", "n": 1048576},
        # the same object as the trainer holds it, for a preview between steps
        {"name": "paper_fp32_262144", "kind": "query", "shape": "paper", "feat": "fp32", "mlp": "fp32",
         "mix": "sphere", "n": 262144},
        # a small request against a scene: a few image rows
        {"name": "scene_2500", "kind": "scene", "objects": 8, "instances": 64, "feat": "fp16", "mlp": "fp16",
         "n": 2500, "bounces": 0},
        # a wavefront path tracer's depth: primary image, then one diffuse bounce
        {"name": "wavefront_512x512", "kind": "scene", "objects": 8, "instances": 64, "feat": "fp16", "mlp": "fp16",
         "n": 262144, "bounces": 1},
        # requests of many sizes in flight at once
        {"name": "serve_24_requests", "kind": "serve", "objects": 8, "instances": 64, "feat": "fp16", "mlp": "fp16",
         "requests": 24, "lo": 256, "hi": 262144},
        # training the paper's default object
        {"name": "train_paper_262144", "kind": "train", "shape": "paper", "n": 262144, "steps": 1},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["query"] * 6 + ["scene"] * 2 + ["serve", "train"])
    if kind == "query":
        shape = rng.choice(["c1", "c2", "c2", "paper", "paper_lq"])
        mlp = rng.choice(["fp32", "fp16", "fp16", "bf16", "fp8"])
        feat = "fp32" if mlp == "fp32" and rng.random() < 0.7 else rng.choice(["fp16", "fp16", "bf16"])
        top = 524288 if mlp == "fp32" else 2097152
        c = {"kind": "query", "shape": shape, "feat": feat, "mlp": mlp,
             "mix": rng.choice(["primary", "frame", "bounce", "sphere"]), "n": _log_int(rng, 200, top)}
        if rng.random() < 0.3:
            c["sort_bits"] = rng.choice([0, 4, 6, 7])
            c["persistent"] = rng.choice([0, 1])
        return c
    if kind == "scene":
        objects = rng.randint(1, 8)
        return {"kind": "scene", "objects": objects, "instances": rng.randint(objects, 64), "feat": "fp16",
                "mlp": rng.choice(["fp16", "bf16"]), "n": _log_int(rng, 500, 262144), "bounces": rng.randint(0, 1)}
    if kind == "serve":
        return {"kind": "serve", "objects": rng.randint(2, 8), "instances": rng.randint(16, 64), "feat": "fp16",
                "mlp": "fp16", "requests": rng.choice([8, 10, 13, 16, 20, 24]), "lo": 256, "hi": _log_int(rng, 4096, 262144)}
    return {"kind": "train", "shape": rng.choice(["paper", "paper", "paper_lq", "c1"]),
            "n": _log_int(rng, 2048, 262144), "steps": 1}


# ------------------------------------------------------------------- objects
_SHAPES = {
    "c1": dict(V=32, half=1.1, L=8, r_min=4, r_max=64, F=2, log2_T=14, H=18, n_hidden=3, width=64, act=0, albedo=0,
               amp=0.0),
    "c2": dict(V=128, half=1.2, L=16, r_min=16, r_max=2048, F=2, log2_T=19, H=18, n_hidden=3, width=64, act=0,
               albedo=0, amp=0.1),
    "paper": dict(V=32, half=1.1, L=2, r_min=64, r_max=128, F=3, log2_T=17, H=18, n_hidden=2, width=128, act=1,
                  albedo=1, amp=0.0),
    "paper_lq": dict(V=32, half=1.1, L=2, r_min=64, r_max=128, F=3, log2_T=17, H=10, n_hidden=2, width=64, act=1,
                     albedo=1, amp=0.0),
}


def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _bumps(g, amp):
    """Amplitudes, frequencies and phases of the sphere's radius 1 + sum a sin(w . u + phi)."""
    k = 8
    return (amp / k * (2 * torch.rand(k, generator=g, device=DEV, dtype=torch.float64) - 1) * 2,
            6 * torch.randn(k, 3, generator=g, device=DEV, dtype=torch.float64),
            6.2831853 * torch.rand(k, generator=g, device=DEV, dtype=torch.float64))


def _surface(kind, bumps, p):
    """Signed function of points p (..., 3): negative inside."""
    if kind == "torus":
        return (torch.sqrt(p[..., 0] ** 2 + p[..., 1] ** 2) - 0.7) ** 2 + p[..., 2] ** 2 - 0.0625
    r = p.norm(dim=-1)
    u = p / r.clamp_min(1e-9)[..., None]
    a, w, ph = bumps
    rad = torch.ones_like(r)
    for i in range(len(a)):
        rad = rad + a[i] * torch.sin(u @ w[i] + ph[i])
    return r - rad


def _occupancy(kind, bumps, V, half):
    """Bits of the voxels the surface passes through: its function changes sign over the corners."""
    t = torch.linspace(-half, half, V + 1, device=DEV, dtype=torch.float64)
    inside = torch.empty((V + 1,) * 3, dtype=torch.bool, device=DEV)
    for z0 in range(0, V + 1, 32):
        zz, yy, xx = torch.meshgrid(t[z0:z0 + 32], t, t, indexing="ij")
        inside[z0:z0 + 32] = _surface(kind, bumps, torch.stack([xx, yy, zz], -1)) < 0
    c = [inside[a:V + a, b:V + b, d:V + d] for a in (0, 1) for b in (0, 1) for d in (0, 1)]
    some, every = c[0].clone(), c[0].clone()
    for q in c[1:]:
        some |= q
        every &= q
    occ = (some & ~every).reshape(-1)
    bits = np.packbits(occ.cpu().numpy(), bitorder="little")
    return np.ascontiguousarray(np.pad(bits, (0, -len(bits) % 4))).view(np.uint32)


def _object(g, V, half, L, r_min, r_max, F, log2_T, H, n_hidden, width, act, albedo, amp, kind="sphere"):
    bumps = _bumps(g, amp)
    b = (r_max / r_min) ** (1.0 / (L - 1))
    R = np.array([int(math.floor(r_min * b ** l + 0.5)) for l in range(L)], np.int32)
    dims = [H * L * F] + [width] * n_hidden + [5 + 3 * albedo + 4]
    tables = (2 * torch.rand(L, 1 << log2_T, F, generator=g, device=DEV) - 1) * 1e-2
    W = [torch.randn(dims[i + 1], dims[i], generator=g, device=DEV) * math.sqrt(2.0 / dims[i])
         for i in range(len(dims) - 1)]
    return SimpleNamespace(bmin=np.full(3, -half, np.float32), bmax=np.full(3, half, np.float32), V=V,
                           occ=_occupancy(kind, bumps, V, half), L=L, F=F, log2_T=log2_T, R=R,
                           tables=tables.cpu().numpy(), H=H, weights=[w.cpu().numpy() for w in W], act=act,
                           leaky_slope=0.01, n_mat=4, has_albedo=albedo, kind=kind, bumps=bumps, half=half)


def _scene_object(g, i):
    """Object i of a scene: the sizes of the many-object workload."""
    r = np.random.Generator(np.random.PCG64(int(torch.randint(1 << 30, (1,), generator=g, device=DEV).item())))
    V = [32, 64, 128, 256][i % 4]
    return _object(g, V=V, half=1.15, L=int(r.integers(8, 17)), r_min=16, r_max=16 * V, F=2,
                   log2_T=int(r.integers(14, 20)), H=18, n_hidden=3, width=64, act=0, albedo=0, amp=0.1,
                   kind="torus" if i % 3 == 0 else "sphere")


# ---------------------------------------------------------------------- rays
def _unit(v):
    return v / v.norm(dim=-1, keepdim=True)


def _rays(o, d, tmax=None):
    n = len(o)
    r = torch.empty(n, 8, dtype=torch.float32, device=DEV)
    r[:, 0:3], r[:, 3:6], r[:, 6] = o.float(), d.float(), 0.0
    r[:, 7] = math.inf if tmax is None else tmax.float()
    return r


def _randn(g, n):
    return torch.randn(n, 3, generator=g, device=DEV, dtype=torch.float64)


def _rand(g, *s):
    return torch.rand(*s, generator=g, device=DEV, dtype=torch.float64)


def _sphere_rays(g, n):
    o = 2.0 * _unit(_randn(g, n))
    return _rays(o, _unit(2 * _rand(g, n, 3) - 1 - o))


def _pinhole(n, width, row0, height, eye, target, vfov):
    eye = torch.tensor(eye, dtype=torch.float64, device=DEV)
    fwd = _unit(torch.tensor(target, dtype=torch.float64, device=DEV) - eye)
    up = torch.tensor([0.0, 1.0, 0.0], dtype=torch.float64, device=DEV)
    right = _unit(torch.linalg.cross(fwd, up))
    up = torch.linalg.cross(right, fwd)
    th = math.tan(math.radians(vfov) / 2)
    k = torch.arange(n, device=DEV)
    i, j = k % width, row0 + k // width
    sx = ((i + 0.5) / width * 2 - 1) * th * (width / height)
    sy = (1 - (j + 0.5) / height * 2) * th
    d = _unit(fwd + sx[:, None] * right + sy[:, None] * up)
    return _rays(eye.expand(n, 3), d)


def _primary(g, n):
    """A square image of n pixels (the last row cut short) of the object at the origin."""
    side = math.isqrt(max(n - 1, 0)) + 1
    r = _pinhole(n, side, 0, side, (0.0, 0.0, 3.0), (0.0, 0.0, 0.0), 50.0)
    # the camera turns with the seed
    a = 6.2831853 * float(_rand(g, 1).item())
    m = torch.tensor([[math.cos(a), 0, math.sin(a)], [0, 1, 0], [-math.sin(a), 0, math.cos(a)]], device=DEV)
    r[:, 0:3], r[:, 3:6] = r[:, 0:3] @ m.T, r[:, 3:6] @ m.T
    return r


def _surface_points(g, obj, n):
    """Points of a bumpy sphere, uniform in direction, and their outward normals."""
    u = _unit(_randn(g, n))
    a, w, ph = obj.bumps
    rad = torch.ones(n, dtype=torch.float64, device=DEV)
    grad = torch.zeros(n, 3, dtype=torch.float64, device=DEV)
    for i in range(len(a)):
        x = u @ w[i] + ph[i]
        rad = rad + a[i] * torch.sin(x)
        grad = grad + (a[i] * torch.cos(x))[:, None] * w[i]
    grad = grad - (grad * u).sum(1, keepdim=True) * u
    return rad[:, None] * u, _unit(u - grad / rad[:, None])


def _cosine(g, nrm):
    n = len(nrm)
    r, phi = _rand(g, n).sqrt(), 6.283185307179586 * _rand(g, n)
    x = torch.tensor([1.0, 0, 0], dtype=torch.float64, device=DEV)
    y = torch.tensor([0, 1.0, 0], dtype=torch.float64, device=DEV)
    t = _unit(torch.linalg.cross(torch.where(nrm[:, :1].abs() > 0.9, y, x), nrm))
    b = torch.linalg.cross(nrm, t)
    return _unit((r * phi.cos())[:, None] * t + (r * phi.sin())[:, None] * b + (1 - r * r).clamp_min(0).sqrt()[:, None] * nrm)


def _bounce(g, obj, n):
    p, nrm = _surface_points(g, obj, n)
    return _rays(p + 1e-4 * nrm, _cosine(g, nrm))


def _shadow(g, obj, n):
    p, nrm = _surface_points(g, obj, n)
    o = p + 1e-4 * nrm
    to = torch.tensor([2.0, 3.0, 4.0], dtype=torch.float64, device=DEV) - o
    dist = to.norm(dim=1)
    return _rays(o, to / dist[:, None], dist)


def _mix(g, obj, mix, n):
    if mix == "sphere":
        return _sphere_rays(g, n)
    if mix == "primary":
        return _primary(g, n)
    if mix == "bounce":
        return _bounce(g, obj, n)
    return torch.cat([_primary(g, n - n // 2), _shadow(g, obj, n // 2)])


def _train_batch(g, n):
    """Half from the box's enclosing sphere toward its centre, half leaving the surface; the
    references are the unit sphere's nearest intersections."""
    rad = 1.1 * math.sqrt(3.0)
    u = _unit(_randn(g, n // 2))
    s = _unit(_randn(g, n - n // 2))
    o = torch.cat([rad * u, (1 + 1e-4) * s])
    d = torch.cat([_cosine(g, -u), _cosine(g, s)])
    rays = _rays(o, d)
    o, d = rays[:, 0:3].double(), rays[:, 3:6].double()
    b, c = (o * d).sum(1), (o * o).sum(1) - 1.0
    disc = b * b - c
    t = -b - disc.clamp_min(0).sqrt()
    hit = (disc > 0) & (t > 0)
    p = _unit(o + t[:, None] * d)
    mat = (p[:, 0] > 0).int() + 2 * (p[:, 1] > 0).int()
    colours = 0.05 + 0.9 * _rand(g, 4, 3)
    gt = torch.zeros(n, 9, dtype=torch.float32, device=DEV)
    gt[:, 0] = hit.int().view(torch.float32)
    gt[:, 1] = torch.where(hit, t, 0.0).float()
    gt[:, 2:5] = torch.where(hit[:, None], p, 0.0).float()
    gt[:, 5:8] = torch.where(hit[:, None], colours[mat.long()], 0.0).float()
    gt[:, 8] = torch.where(hit, mat, 0).int().view(torch.float32)
    return rays, gt


def _instances(g, objects, instances):
    """Instances on a square grid (spacing 3) with a seeded yaw and a scale in [0.8, 1.2]."""
    side = math.isqrt(max(instances - 1, 0)) + 1
    u = _rand(g, instances, 2).cpu().numpy()
    out = []
    for k in range(instances):
        c = np.array([3.0 * (k % side) - 1.5 * (side - 1), 0.0, 3.0 * (k // side) - 1.5 * (side - 1)])
        th, s = 2 * math.pi * u[k, 0], 0.8 + 0.4 * u[k, 1]
        A = np.array([[math.cos(th), 0, math.sin(th)], [0, 1, 0], [-math.sin(th), 0, math.cos(th)]]).T / s
        out.append((k % objects, np.concatenate([A, (-A @ c)[:, None]], 1).astype(np.float32)))
    return out


def _scene_rays(g, n):
    """n pixels of a 1024-wide image of the grid: a window of rows in its middle."""
    width = 1024 if n < 262144 else math.isqrt(n)
    rows = -(-n // width)
    height = max(width, rows)
    row0 = min(height - rows, height // 3 + int(_rand(g, 1).item() * height / 4)) if rows < height else 0
    return _pinhole(n, width, row0, height, (0.0, 18.0, -22.0), (0.0, 0.0, 0.0), 50.0)


# --------------------------------------------------------- the state of a case
class _Program(SimpleNamespace):
    """What a program keeps: its context (destroyed with it), objects and buffers."""

    def __del__(self):
        try:
            if getattr(self, "trainer", None) is not None:
                L.lsnif_trainer_destroy(self.trainer)
            L.lsnif_destroy(self.ctx)   # stops a serving loop first
        except Exception:
            pass


def _inputs(case, seed):
    """Objects, instances and rays of a case, made from the seed alone."""
    g = _gen(seed)
    if case["kind"] in ("query", "train"):
        objs = [_object(g, **_SHAPES[case["shape"]])]
        if case["kind"] == "query":
            return objs, None, _mix(g, objs[0], case["mix"], case["n"])
        return objs, None, [_train_batch(g, case["n"]) for _ in range(case["steps"])]
    objs = [_scene_object(g, i) for i in range(case["objects"])]
    insts = _instances(g, case["objects"], case["instances"])
    if case["kind"] == "scene":
        return objs, insts, _scene_rays(g, case["n"])
    pool = _pinhole(1 << 18, 512, 0, 512, (0.0, 18.0, -22.0), (0.0, 0.0, 0.0), 50.0)
    return objs, insts, (pool, [(int(u * (len(pool) - n)), n, 1) for n, u in
                                zip(_request_sizes(case), _rand(g, case["requests"]).tolist())])


def _request_sizes(case):
    """Sizes spread evenly over the logarithm of [lo, hi], small and large ones interleaved."""
    k = case["requests"]
    return [int(round(case["lo"] * (case["hi"] / case["lo"]) ** (((7 * j) % k + 0.5) / k))) for j in range(k)]


def prepare(case, seed):
    objs, insts, rays = _inputs(case, seed)
    s = _Program(ctx=L.lsnif_create(0), kind=case["kind"], case=case)
    feat, mlp = case.get("feat", "fp32"), case.get("mlp", "fp32")
    ids = [L.lsnif_build(s.ctx, L.ObjectDesc(o, feat, mlp,
                                             FP8_ACT_SCALE[:len(o.weights)] if mlp == "fp8" else None)) for o in objs]
    if case["kind"] == "query":
        s.oid, s.rays = ids[0], rays
        s.out = torch.empty(len(rays), 6, dtype=torch.float32, device=DEV)
        if "sort_bits" in case:
            t = L.lsnif_get_tuning(s.ctx, s.oid)
            t.update(sort_bits=case["sort_bits"], persistent=case.get("persistent", 0))
            L.lsnif_set_tuning(s.ctx, s.oid, **t)
    elif case["kind"] == "train":
        s.obj, s.batches = objs[0], rays
        s.trainer = L.lsnif_trainer_create(s.ctx, ids[0], lr=LR)
        s.loss = torch.zeros(case["steps"], dtype=torch.float32, device=DEV)
    else:
        insts = [(ids[k], m) for k, m in insts]
        if case["kind"] == "scene":
            n = len(rays)
            s.rays, s.inst = rays, torch.from_numpy(L.instances_array(insts)).to(DEV)
            s.out = [torch.zeros(n, 6, dtype=torch.float32, device=DEV) for _ in range(1 + case["bounces"])]
            s.next = torch.zeros(n, 8, dtype=torch.float32, device=DEV)
            s.parent = torch.zeros(n, dtype=torch.int32, device=DEV)
        else:
            pool, windows = rays
            inst = torch.from_numpy(L.instances_array(insts)).to(DEV)
            pr = torch.empty(8 * len(pool), dtype=torch.int32, device=DEV)
            pi = torch.empty_like(pr)
            k = L.lsnif_broad_phase(s.ctx, pool, inst, pr, pi)
            s.set = RequestSet(L, pool.cpu().numpy(), pr[:k].cpu().numpy(), pi[:k].cpu().numpy(), insts, windows)
            L.lsnif_serve_start(s.ctx, max_inflight=8, n_streams=4)
    return s


def _hits(out):
    return dict(L.hits_from(out))


def run(s):
    if s.kind == "query":
        L.lsnif_query(s.ctx, s.oid, s.rays, s.out)
        return _hits(s.out)
    if s.kind == "scene":
        L.lsnif_query_scene(s.ctx, s.rays, s.inst, s.out[0])
        got, rays = [_hits(s.out[0])], s.rays
        for b in range(s.case["bounces"]):
            m = L.lsnif_bounce(s.ctx, rays, s.out[b], 17, b, 1e-4, s.next, s.parent)
            rays = s.next[:m]
            L.lsnif_query_scene(s.ctx, rays, s.inst, s.out[b + 1])
            got.append(dict(_hits(s.out[b + 1]), parent=s.parent, rays=s.next))   # the first m rows
        return got
    if s.kind == "serve":
        tickets = [L.lsnif_serve_submit(s.ctx, s.set.request(j)) for j in range(len(s.set.windows))]
        for t in tickets:
            st = L.lsnif_serve_wait(s.ctx, t)
            if st != L.LSNIF_OK:
                raise RuntimeError(f"request ended with status {st}")
        return [_hits(o) for o in s.set.outs[:16]]
    for k, (rays, gt) in enumerate(s.batches):
        L.lsnif_train_step(s.trainer, rays, gt, s.loss[k:k + 1])
    tab, W, gtab, gW, _ = L.lsnif_trainer_read(s.trainer, s.obj)
    return {"loss": s.loss, "tables": tab, "weights": W, "grad_tables": gtab, "grad_weights": gW}


# ------------------------------------------------------------------------ work
# Rays that meet an occupied voxel, and the boundary points of such a ray, as these mixes have them.
_CAND = {"primary": 0.5, "frame": 0.75, "bounce": 1.0, "sphere": 0.75, "train": 0.6}
_POINTS = {"primary": 12.0, "frame": 9.0, "bounce": 6.0, "sphere": 8.0, "train": 7.0}


def _object_work(shape, mix, n, feat, mlp):
    z = _SHAPES[shape] if isinstance(shape, str) else shape
    cand, pts = n * _CAND[mix], min(_POINTS[mix], z["H"])
    fb, mb = {"fp32": 4, "fp16": 2, "bf16": 2, "fp8": 1}[feat], {"fp32": 4, "fp16": 2, "bf16": 2, "fp8": 1}[mlp]
    LF, w, out = z["L"] * z["F"], z["width"], 9 + 3 * z["albedo"]
    macs = pts * LF * w + (z["n_hidden"] - 1) * w * w + w * out
    table = z["L"] * 2 ** z["log2_T"] * z["F"] * fb
    weights = (z["H"] * LF * w + (z["n_hidden"] - 1) * w * w + w * out) * mb
    gathered = min(table, cand * pts * 8 * LF * fb)   # each entry once, or fewer where few rays ask
    return {"bytes": n * 56 + gathered + min(weights, cand * weights), "flops": 2 * macs * cand}


def work(case):
    if case["kind"] == "query":
        return _object_work(case["shape"], case["mix"], case["n"], case["feat"], case["mlp"])
    if case["kind"] == "train":
        w = _object_work(case["shape"], "train", case["n"], "fp32", "fp32")
        z = _SHAPES[case["shape"]]
        params = z["L"] * 2 ** z["log2_T"] * z["F"] * 4
        # per step: forward, both backward products, the target, and Adam's three arrays read and written;
        # then four arrays of parameters read back
        return {"bytes": case["steps"] * (w["bytes"] + case["n"] * 12 + 6 * params) + 2 * params,
                "flops": case["steps"] * 3 * w["flops"]}
    z = dict(_SHAPES["c2"], L=12, log2_T=17, V=128)
    if case["kind"] == "scene":
        n = case["n"] * (1 + 0.25 * case["bounces"])
    else:
        n = sum(_request_sizes(case))
    return _object_work(z, "primary", n, case["feat"], case["mlp"])


# ----------------------------------------------------------------------- exact
def _span(o, inv, up, k):
    lo, hi = (k - o) * inv, ((k + 1.0) - o) * inv
    return torch.where(up, lo, hi), torch.where(up, hi, lo)


def _setup(obj, rays):
    """Voxel-space rays and their interval in float32, as the format defines the walk."""
    f = torch.float32
    bmin = torch.from_numpy(obj.bmin).to(DEV)
    sc = torch.from_numpy(np.float32(obj.V) / (obj.bmax - obj.bmin)).to(DEV)
    o, d = (rays[:, 0:3] - bmin) * sc, rays[:, 3:6] * sc
    inv = torch.ones((), dtype=f, device=DEV) / d
    mov = (d != 0) & inv.isfinite()
    inv = torch.where(mov, inv, 0.0)
    V = float(obj.V)
    a, b = (0.0 - o) * inv, (V - o) * inv
    inf = torch.tensor(math.inf, device=DEV)
    t0 = torch.where(mov, torch.minimum(a, b), -inf).amax(1)
    t1 = torch.where(mov, torch.maximum(a, b), inf).amin(1)
    inside = (mov | ((o >= 0) & (o <= V))).all(1)
    ta, tb = torch.maximum(t0, rays[:, 6]), t1
    return o, d, inv, mov, ta, tb, inside & mov.any(1) & (ta < tb)


def _walk(obj, o, d, inv, mov, ta, tb):
    """The first H/2 occupied voxels of each (candidate) ray, cell by cell in float32."""
    V, cap, n = obj.V, obj.H // 2, len(o)
    occ = np.unpackbits(obj.occ.view(np.uint8), bitorder="little")[:V ** 3]
    occ = torch.from_numpy(occ).to(DEV).bool()
    up = d > 0
    inf = torch.tensor(math.inf, device=DEV)
    step = torch.where(up, 1.0, -1.0)
    x = (o + ta[:, None] * d).clamp(0.0, V - 1.0)
    c = torch.where(mov, x.floor(), o.floor().clamp_max(V - 1.0))
    for _ in range(4):   # a floor guess, corrected by at most a few cells
        en, ex = _span(o, inv, up, c)
        back, on = mov & (en > ta[:, None]), mov & (ex <= ta[:, None])
        nk = torch.where(back, c - step, torch.where(on & ~back, c + step, c))
        c = torch.where((nk < 0) | (nk >= V), c, nk)
    cells = torch.full((n, cap, 3), -1.0, device=DEV)
    count = torch.zeros(n, dtype=torch.long, device=DEV)
    alive = torch.arange(n, device=DEV)
    for _ in range(3 * V):
        if not len(alive):
            break
        oa, ia, ua, ca, ma = o[alive], inv[alive], up[alive], c[alive], mov[alive]
        en, ex = _span(oa, ia, ua, ca)
        en, ex = torch.where(ma, en, -inf), torch.where(ma, ex, inf)
        tin, tout = en.amax(1), ex.amin(1)
        axis = torch.where(ex[:, 0] == tout, 0, torch.where(ex[:, 1] == tout, 1, 2))
        keep = torch.minimum(tout, tb[alive]) > torch.maximum(tin, ta[alive])
        idx = (ca[:, 0] + V * (ca[:, 1] + V * ca[:, 2])).long() if V <= 128 else \
            ca[:, 0].long() + V * (ca[:, 1].long() + V * ca[:, 2].long())
        sel = (keep & occ[idx]).nonzero()[:, 0]
        r = alive[sel]
        cells[r, count[r]] = ca[sel]
        count[r] += 1
        ca = ca.scatter_add(1, axis[:, None], step[alive].gather(1, axis[:, None]))
        c[alive] = ca
        moved = ca.gather(1, axis[:, None])[:, 0]
        on = (count[alive] < cap) & (tout < tb[alive]) & (moved >= 0) & (moved < V)
        alive = alive[on]
    return cells, count


def _points(obj, o, d, inv, mov, cells, count):
    """Boundary points (n, H, 3) in float32 and which of them exist."""
    n, cap = cells.shape[:2]
    inf = torch.tensor(math.inf, device=DEV)
    up = (d > 0)[:, None]
    en, ex = _span(o[:, None], inv[:, None], up, cells)
    m = mov[:, None]
    en, ex = torch.where(m, en, -inf), torch.where(m, ex, inf)
    out = []
    for t3, best, is_exit in ((en, en.amax(2), False), (ex, ex.amin(2), True)):
        eq = t3 == best[..., None]
        face = torch.where(eq[..., 0], 0, torch.where(eq[..., 1], 1, 2))
        v = o[:, None] + best[..., None] * d[:, None]
        v = torch.minimum(torch.maximum(v, cells), cells + 1.0)
        plane = torch.where(up == is_exit, cells + 1.0, cells)
        on = torch.arange(3, device=DEV) == face[..., None]
        out.append(torch.where(on, plane, v))
    p = torch.stack(out, 2).reshape(n, 2 * cap, 3)
    has = torch.arange(2 * cap, device=DEV)[None] < 2 * count[:, None]
    return p, has


def _features(obj, tables, p, has):
    """Trilinear hash-grid features (n, H L F) of float32 points, in the tables' 64 bits."""
    n, H = p.shape[:2]
    T = 1 << obj.log2_T
    feats = []
    for l in range(obj.L):
        R = int(obj.R[l])
        x = (p * torch.tensor(np.float32(R) / np.float32(obj.V), device=DEV)).clamp(0.0, float(R))
        k = x.floor().clamp_max(R - 1.0)
        w, i = (x - k).double(), k.long()
        acc = 0
        for c in range(8):
            b = [c & 1, (c >> 1) & 1, c >> 2]
            v = [i[..., a] + b[a] for a in range(3)]
            if (R + 1) ** 3 <= T:
                slot = v[0] + (R + 1) * (v[1] + (R + 1) * v[2])
            else:
                slot = (v[0] ^ (v[1] * 2654435761) ^ (v[2] * 805459861)) & (T - 1)
            wc = 1.0
            for a in range(3):
                wc = wc * (w[..., a] if b[a] else 1.0 - w[..., a])
            acc = acc + torch.where(has, wc, 0.0)[..., None] * tables[l][torch.where(has, slot, 0)]
        feats.append(acc)
    return torch.stack(feats, 2).reshape(n, H * obj.L * obj.F)


def _act(obj, x):
    return torch.where(x > 0, x, x * (obj.leaky_slope if obj.act else 0.0))


def _mlp(obj, W, x):
    for w in W[:-1]:
        x = _act(obj, x @ w.T)
    return x @ W[-1].T


def _as(x, dtype):
    """Values as the object stores them, in 64 bits."""
    t = torch.from_numpy(np.asarray(x)).to(DEV)
    return t.to({"fp32": torch.float32, "fp16": torch.float16, "bf16": torch.bfloat16}[dtype]).double()


def _answer(obj, rays, feat, mlp):
    """(hit, t, normal, material) of object-space rays in 64 bits; t is +inf and the rest 0 on a miss."""
    n = len(rays)
    t = torch.full((n,), math.inf, dtype=torch.float64, device=DEV)
    nrm = torch.zeros(n, 3, dtype=torch.float64, device=DEV)
    hit = torch.zeros(n, dtype=torch.bool, device=DEV)
    tables, W = _as(obj.tables, feat), [_as(w, mlp) for w in obj.weights]
    o, d, inv, mov, ta, tb, cand = _setup(obj, rays)
    who = cand.nonzero()[:, 0]
    if not len(who):
        return hit, t, nrm
    cells, count = _walk(obj, o[who], d[who], inv[who], mov[who], ta[who], tb[who])
    some = (count > 0).nonzero()[:, 0]
    for part in some.split(65536):
        r = who[part]
        p, has = _points(obj, o[r], d[r], inv[r], mov[r], cells[part], count[part])
        z = _mlp(obj, W, _features(obj, tables, p, has))
        th = ta[r].double() + torch.sigmoid(z[:, 1]) * (tb[r] - ta[r]).double()
        h = (z[:, 0] > 0) & (th <= rays[r, 7].double())
        hit[r] = h
        t[r] = torch.where(h, th, math.inf)
        nrm[r] = torch.where(h[:, None], _unit(z[:, 2:5]), 0.0)
    return hit, t, nrm


def _answer_scene(objs, insts, rays, feat, mlp):
    n = len(rays)
    t = torch.full((n,), math.inf, dtype=torch.float64, device=DEV)
    nrm = torch.zeros(n, 3, dtype=torch.float64, device=DEV)
    by_object = {}
    for k, m in insts:
        by_object.setdefault(k, []).append(torch.from_numpy(m).to(DEV))
    for k, ms in by_object.items():
        local, owner, mats = [], [], []
        for j, m in enumerate(ms):
            r = rays.clone()
            for a in range(3):
                r[:, a] = ((m[a, 0] * rays[:, 0] + m[a, 1] * rays[:, 1]) + m[a, 2] * rays[:, 2]) + m[a, 3]
                r[:, 3 + a] = (m[a, 0] * rays[:, 3] + m[a, 1] * rays[:, 4]) + m[a, 2] * rays[:, 5]
            ta, cand = _setup(objs[k], r)[4::2]
            who = (cand & (ta <= r[:, 7])).nonzero()[:, 0]
            local.append(r[who])
            owner.append(who)
            mats.append(torch.full((len(who),), j, dtype=torch.long, device=DEV))
        local, owner, mats = torch.cat(local), torch.cat(owner), torch.cat(mats)
        if not len(local):
            continue
        _, th, nh = _answer(objs[k], local, feat, mlp)
        A = torch.stack(ms).double()[:, :, :3]
        for j in range(len(ms)):
            sel = (mats == j).nonzero()[:, 0]
            r = owner[sel]
            near = th[sel] < t[r]
            w = nh[sel] @ A[j]
            w = torch.where(near[:, None], w / w.norm(dim=1, keepdim=True).clamp_min(1e-300), nrm[r])
            t[r], nrm[r] = torch.where(near, th[sel], t[r]), w
    return t, nrm


def _loss(obj, z, gt, ta, tb, n):
    y = gt[:, 0].contiguous().view(torch.int32) != 0
    yh = y.double()
    per = torch.nn.functional.softplus(z[:, 0]) - yh * z[:, 0]
    tau = ((gt[:, 1].double() - ta.double()) / (tb - ta).double()).clamp(0, 1)
    more = (torch.sigmoid(z[:, 1]) - tau).abs()
    v = z[:, 2:5]
    more = more + 1 - (v * gt[:, 2:5].double()).sum(1) / v.norm(dim=1).clamp_min(1e-8)
    m0 = 5
    if obj.has_albedo:
        a = torch.sigmoid(z[:, 5:8])
        more = more + ((a - gt[:, 5:8].double()) ** 2 / (a.detach() + 0.01) ** 2).sum(1) / 3
        m0 = 8
    mat = gt[:, 8].contiguous().view(torch.int32).long()
    more = more + torch.nn.functional.cross_entropy(z[:, m0:m0 + obj.n_mat], mat, reduction="none")
    return (per + torch.where(y, more, 0.0)).sum() / n


def _exact_train(case, seed):
    objs, _, batches = _inputs(case, seed)
    obj = objs[0]
    P = [_as(obj.tables, "fp32")] + [_as(w, "fp32") for w in obj.weights]
    M, S = [torch.zeros_like(p) for p in P], [torch.zeros_like(p) for p in P]
    losses, G = [], None
    for k, (rays, gt) in enumerate(batches):
        for p in P:
            p.requires_grad_(True)
            p.grad = None
        o, d, inv, mov, ta, tb, cand = _setup(obj, rays)
        who = cand.nonzero()[:, 0]
        cells, count = _walk(obj, o[who], d[who], inv[who], mov[who], ta[who], tb[who])
        total = 0.0
        for part in (count > 0).nonzero()[:, 0].split(32768):
            r = who[part]
            p, has = _points(obj, o[r], d[r], inv[r], mov[r], cells[part], count[part])
            z = _mlp(obj, P[1:], _features(obj, P[0], p, has))
            loss = _loss(obj, z, gt[r], ta[r], tb[r], len(rays))
            loss.backward()
            total += float(loss.detach())
        losses.append(total)
        G = [p.grad for p in P]
        with torch.no_grad():
            for i, p in enumerate(P):
                M[i] = 0.9 * M[i] + 0.1 * G[i]
                S[i] = 0.999 * S[i] + 0.001 * G[i] ** 2
                P[i] = p - LR * (M[i] / (1 - 0.9 ** (k + 1))) / ((S[i] / (1 - 0.999 ** (k + 1))).sqrt() + 1e-8)
    num = lambda v: v.detach().cpu().numpy()   # noqa: E731
    return {"loss": np.array(losses), "tables": num(P[0]), "weights": [num(w) for w in P[1:]],
            "grad_tables": num(G[0]), "grad_weights": [num(w) for w in G[1:]]}


def exact(case, seed):
    if case["kind"] == "train":
        return _exact_train(case, seed)
    if case["mlp"] == "fp8":   # the 8-bit values are the definition: no 64-bit answer stands behind them
        return None
    objs, insts, rays = _inputs(case, seed)
    if case["kind"] == "query":
        _, t, nrm = _answer(objs[0], rays, case["feat"], case["mlp"])
        return {"hit": None, "t": t, "normal": nrm, "material": None}
    if case["kind"] == "scene":
        t, nrm = _answer_scene(objs, insts, rays, case["feat"], case["mlp"])
        first = {"hit": None, "t": t, "normal": nrm, "material": None}
        return [first] + [None] * case["bounces"]   # bounce rays follow from rounded hits
    pool, windows = rays
    t, nrm = _answer_scene(objs, insts, pool, case["feat"], case["mlp"])
    return [{"hit": None, "t": t[s:s + n], "normal": nrm[s:s + n], "material": None} for s, n, _ in windows[:16]]
