"""The work whose speed is measured: calls of this framework's public entry points over
the sizes, options and directions that its users run.

A case is a dict of plain values; ``op`` says which entry point it goes through:

* ``render``: ``Renderer.render`` into destinations allocated once (a training loop);
* ``graph``:  ``Graph.replay`` of one captured render of an uneven batch;
* ``shade``:  ``autograd.shade`` forward and backward (gradients of the randomized
  parameters for a given image gradient);
* ``serve``:  ``Server.run`` on a burst of requests.

``exact`` renders the same inputs in 64 bits with plain torch operations (projection,
rasterization, visibility, shadow maps, textures, shading, and the gradients by torch's own
differentiation); 8-bit, integer and tracker outputs have no value there.
"""
import math

import numpy as np
import torch

from paper_1906_11633_amd import scenes as S

CHANNELS = ("rgb", "depth", "normal", "seg")
PIXEL_BYTES = dict(rgb=12, depth=4, normal=12, seg=4, tri_id=4, alpha=4, rgb8=3)
SERVE_RES = (64, 128, 200)
SERVE_POOL = 64


def _case(name, op, scene, scenes, cams, width, height, outputs="rgb,depth,normal,seg", spot=0, materials=False,
          post=False):
    c = dict(op=op, scene=scene, scenes=scenes, cams=cams, width=width, height=height, outputs=outputs, spot=spot,
             materials=materials, post=post)
    return c if name is None else dict(name=name, **c)


def listed():
    every = "rgb,depth,normal,seg,tri_id,alpha,rgb8,track"
    return [
        # the smallest batch: four plain scenes at 64 x 64 (a unit-test or debugging call)
        _case("plain_4x64", "render", "plain", 4, 1, 64, 64),
        # one small policy request: two scenes, three cameras
        _case("hand_2x3_128", "render", "hand", 2, 3, 128, 128),
        # a request of the average size that the server meets, alone
        _case("hand_16x3_200", "render", "hand", 16, 3, 200, 200),
        # the training batch: 256 randomized scenes, three cameras, four channels
        _case("hand_256x3_200", "render", "hand", 256, 3, 200, 200),
        # the paper's benchmark batch: 64 scenes, 3 cameras, spot lights with soft shadows,
        # randomized materials and post-processing, 3 x 8-bit RGB only
        _case("paper_64x3_200_rgb8", "render", "hand", 64, 3, 200, 200, "rgb8", 3, True, True),
        # shadowed and textured scenes with the float channels
        _case("spot_48x3_128", "render", "hand", 48, 3, 128, 128, spot=3, materials=True),
        # every output at a ragged size (no row is a multiple of four pixels)
        _case("every_40x3_177x131", "render", "hand", 40, 3, 177, 131, every, post=True),
        # the uneven batch (mixed resolutions and 2 k to 50 k triangles a scene), graph replay
        _case("uneven_256x3", "graph", "mixed", 256, 3, 256, 256),
        # single large images (beyond the persistent kernel's 256 x 256)
        _case("large_2x1_1024x768", "render", "hand", 2, 1, 1024, 768),
        # differentiable shading: forward and backward of the gradient workload
        _case("shade_64x3_200", "shade", "hand", 64, 3, 200, 200, "rgb"),
        # a small gradient step, as in fitting one scene's materials
        _case("shade_2x3_96", "shade", "hand", 2, 3, 96, 96, "rgb"),
        # a burst of eight requests through the server's queue
        _case("serve_8", "serve", "hand", 8, 3, 200, 200),
    ]


def _log(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["render"] * 6 + ["graph"] * 2 + ["shade"] * 3 + ["serve"] * 1 + ["large"] * 2)
    if kind == "graph":
        return _case(None, "graph", "mixed", _log(rng, 8, 256), rng.randint(1, 3), 256, 256)
    if kind == "shade":
        side = rng.randint(48, 200)
        return _case(None, "shade", "hand", _log(rng, 1, 64), rng.randint(1, 3), side, rng.randint(48, 200), "rgb")
    if kind == "serve":
        return _case(None, "serve", "hand", rng.randint(2, 12), 3, 200, 200)
    if kind == "large":
        return _case(None, "render", "hand", rng.randint(1, 4), 1, rng.randint(257, 1024), rng.randint(200, 1024))
    if rng.random() < 0.15:
        return _case(None, "render", "plain", _log(rng, 1, 256), 1, 64, 64)
    outs = rng.choice(["rgb,depth,normal,seg"] * 4 + ["rgb8"] * 2 + ["depth,seg", "rgb,depth,normal,seg,tri_id,alpha,rgb8,track"])
    square = rng.random() < 0.6
    w = rng.choice((64, 128, 200, 256)) if square else rng.randint(48, 256)
    h = w if square else rng.randint(48, 256)
    n = _log(rng, 1, 256 if w * h <= 200 * 200 else 128)
    spot = rng.choice((0, 0, 3)) if n <= 128 and outs != "depth,seg" else 0
    return _case(None, "render", "hand", n, rng.randint(1, 3), w, h, outs, spot, rng.random() < 0.3 and n <= 128,
                 "rgb8" in outs)


# --------------------------------------------------------------------------------------
# inputs
# --------------------------------------------------------------------------------------


def _resized(batch, width, height):
    """The batch with frames of width x height (same vertical field of view)."""
    F = batch.n_frames
    intr = np.tile(S.intrinsics(width, height), (F, 1)).astype(np.float32)
    return batch.replace(width=np.full(F, width, np.int32), height=np.full(F, height, np.int32), intr=intr)


def _point_lights(batch, seed):
    """The batch with 1, 2, 3, 4, 1, ... point lights in its scenes, drawn like the generator's
    (whose counts are random): the arrays have the same sizes for every seed."""
    n = 1 + np.arange(batch.n_scenes) % 4
    L = int(n.sum())
    rng = np.random.default_rng([seed, 0x116])
    az, rho, height = rng.uniform(0, 2 * np.pi, L), rng.uniform(0.4, 0.8, L), rng.uniform(0.3, 0.8, L)
    pos = S.HAND_TARGET + np.stack([rho * np.cos(az), rho * np.sin(az), height], 1)
    return batch.replace(scene_light_begin=np.concatenate([[0], np.cumsum(n)]).astype(np.int32),
                         light_type=np.zeros(L, np.int32), light_vec=pos.astype(np.float32),
                         light_intensity=rng.uniform(0.5, 2.0, L).astype(np.float32))


def _restated(batch, seed):
    """The uneven batch's structure (meshes, triangle counts, resolutions, lights) with another
    randomized state: poses, materials, lights and exposures."""
    rng = np.random.default_rng([seed, 0x57A7])
    O, L = batch.n_objects, batch.n_lights
    q = rng.normal(size=(O, 4))
    w, x, y, z = (q / np.linalg.norm(q, axis=1, keepdims=True)).T
    R = np.stack([1 - 2 * (y * y + z * z), 2 * (x * y - z * w), 2 * (x * z + y * w),
                  2 * (x * y + z * w), 1 - 2 * (x * x + z * z), 2 * (y * z - x * w),
                  2 * (x * z - y * w), 2 * (y * z + x * w), 1 - 2 * (x * x + y * y)], 1).reshape(O, 3, 3)
    scale = np.linalg.norm(batch.object_pose[:, :, 0].astype(np.float64), axis=1)
    pose = np.zeros((O, 3, 4))
    pose[:, :, :3] = scale[:, None, None] * R
    pose[:, :, 3] = S.HAND_TARGET + rng.uniform(-0.15, 0.15, (O, 3))
    f32 = lambda a: np.asarray(a).astype(np.float32)
    return batch.replace(object_pose=f32(pose), albedo=f32(rng.uniform(0, 1, (O, 3))),
                         roughness=f32(rng.uniform(0.05, 1.0, O)), specular=f32(rng.uniform(0, 1, O)),
                         light_intensity=f32(rng.uniform(0.5, 2.0, L)),
                         exposure=f32(rng.uniform(0.7, 1.3, batch.n_frames)))


def _batch(case, seed):
    n, cams = case["scenes"], case["cams"]
    if case["scene"] == "plain":
        return S.config1(seed, n, case["width"], materials=True)
    if case["scene"] == "mixed":
        return _restated(S.config3(3, n, cams), seed)
    b = _point_lights(S.config2(seed, n, case["height"], cams), seed)
    if case["width"] != case["height"]:
        b = _resized(b, case["width"], case["height"])
    if case["materials"]:
        b = S.with_materials(b, seed)
    if case["spot"]:
        b = S.with_spot_lights(b, seed, case["spot"])
    if case["post"]:
        b = S.with_postprocessing(b, seed)
    return b


def _image_gradient(batch, seed):
    """dL/d(rgb) as a learner hands it back: dense, a bias per channel and noise."""
    g = torch.Generator().manual_seed(seed)
    P = batch.total_pixels
    return (torch.randn(3 * P, generator=g) * 0.5 + 0.25) * 1e-3


def _requests(case, seed):
    """(pool scene ids, resolution) of each request of the burst."""
    size, pick = np.random.default_rng(0x5E4E), np.random.default_rng([seed, 0x5E4E])
    return [(pick.integers(0, SERVE_POOL, int(size.integers(1, 33))), int(size.choice(SERVE_RES)))
            for _ in range(case["scenes"])]


def prepare(case, seed):
    from paper_1906_11633_amd import autograd, renderer, serving
    r = renderer.Renderer(0)
    if case["op"] == "serve":
        pool = serving.ScenePool(r.ctx, SERVE_POOL, seed)
        server = serving.Server(r.ctx, pool, keep_results=True)
        return dict(op="serve", server=server, request=serving.Request, requests=_requests(case, seed))
    batch = _batch(case, seed)
    job = r.prepare(batch)
    if case["op"] == "shade":
        params = [job.state[k].clone().requires_grad_() for k in autograd.PARAMS]
        job.extra["grad_workspace"] = torch.empty(max(int(job.layout.info.grad_workspace_bytes), 256),
                                                  dtype=torch.uint8, device="cuda")
        return dict(op="shade", r=r, job=job, shade=autograd.shade, names=autograd.PARAMS, params=params,
                    grad=_image_gradient(batch, seed).cuda())
    names = case["outputs"].split(",")
    out = r.alloc_outputs(job, base=tuple(k for k in CHANNELS if k in names),
                          **{k: True for k in names if k not in CHANNELS})
    if case["op"] == "graph":
        job.layout.set_tuning(path=2)
        stream = torch.cuda.Stream()
        graph = renderer.Graph(r.ctx, job.layout, job.state, out, job.workspace, stream)
        return dict(op="graph", r=r, job=job, out=out, graph=graph)
    return dict(op="render", r=r, job=job, out=out)


def run(state):
    op = state["op"]
    if op == "render":
        return state["r"].render(state["job"], state["out"])
    if op == "graph":
        state["graph"].replay()
        return state["out"]
    if op == "shade":
        rgb = state["shade"](state["r"], state["job"], *state["params"])
        grads = torch.autograd.grad(rgb, state["params"], state["grad"])
        return dict(zip(state["names"], grads), rgb=rgb.detach())
    server = state["server"]
    reqs = [state["request"](k, ids, res, 0.0) for k, (ids, res) in enumerate(state["requests"])]
    server.run(reqs)
    server.done.clear()
    return [r.result for r in reqs]


# --------------------------------------------------------------------------------------
# what a pass cannot do without
# --------------------------------------------------------------------------------------


def _tracked(batch):
    return int(np.diff(batch.scene_object_begin)[batch.frame_scene].sum())


def work(case):
    """Every output written once, the scene state and meshes read once.  Operations: each
    vertex and triangle instance transformed and set up once, and the covered pixels' shade
    (a fifth of the pixels, four lights)."""
    if case["op"] == "serve":
        reqs = _requests(case, 1)
        pixels = sum(3 * len(ids) * res * res for ids, res in reqs)
        n = sum(len(ids) for ids, _ in reqs)
        verts, tris = 3 * n * 6936, 3 * n * 13568
        return dict(bytes=32 * pixels + n * 2600, flops=60 * verts + 30 * tris + 60 * pixels)
    batch = _batch(case, 1)
    names = case["outputs"].split(",")
    pixels = batch.total_pixels
    out = sum(PIXEL_BYTES.get(k, 0) for k in names) * pixels + (48 * _tracked(batch) if "track" in names else 0)
    mesh = sum(32 * m.n_verts + 16 * m.n_tris for m in batch.meshes)
    state = 73 * batch.n_objects + 16 * batch.n_lights + 72 * batch.n_frames
    if case["materials"]:
        mesh += sum(8 * m.n_verts for m in batch.meshes) + sum(16 * t.shape[0] * t.shape[1] for t in batch.textures)
        state += 28 * batch.n_objects
    if case["spot"]:
        state += 84 * batch.n_lights
    if case["post"]:
        state += 48 * batch.n_frames + batch.grain.nbytes
    tris = int(batch.frame_triangles().sum())
    flops = 60 * (tris // 2) + 30 * tris + 60 * pixels
    if case["op"] == "shade":  # forward writes rgb; backward reads the image gradient
        return dict(bytes=24 * pixels + mesh + 2 * state, flops=2 * flops)
    return dict(bytes=out + mesh + state, flops=flops)


# --------------------------------------------------------------------------------------
# the same results in 64 bits
# --------------------------------------------------------------------------------------


class _Scene:
    """One scene's geometry as flat tensors: vertices, triangles and their objects."""

    def __init__(self, b, s, dev):
        o0, o1 = int(b.scene_object_begin[s]), int(b.scene_object_begin[s + 1])
        ms = [b.meshes[m] for m in b.object_mesh[o0:o1]]
        vb = np.concatenate([[0], np.cumsum([m.n_verts for m in ms])]).astype(np.int64)
        d = lambda a: torch.as_tensor(np.asarray(a), dtype=torch.float64, device=dev)
        i = lambda a: torch.as_tensor(np.asarray(a), dtype=torch.int64, device=dev)
        self.o0, self.o1 = o0, o1
        self.pos = d(np.concatenate([m.pos for m in ms]))
        nrm = d(np.concatenate([m.nrm for m in ms]))
        self.nrm = nrm / nrm.norm(dim=1, keepdim=True)
        self.uv = d(np.concatenate([m.uv for m in ms]))
        self.tri = i(np.concatenate([m.idx + v for m, v in zip(ms, vb)]))
        self.vert_obj = i(np.repeat(np.arange(o1 - o0), [m.n_verts for m in ms]))
        self.tri_obj = i(np.repeat(np.arange(o1 - o0), [m.n_tris for m in ms]))


def _matrix(view, pose):
    """view o pose for poses [O, 3, 4], as 3 x 4 matrices."""
    R = view[:, :3] @ pose[:, :, :3]
    t = (view[:, :3] @ pose[:, :, 3:])[:, :, 0] + view[:, 3]
    return R, t


def _visible(sc, view, intr, near, pose, shown, W, H):
    """Nearest fragment of each pixel: (pixel, triangle, edge weights over w, depth) of the
    covered pixels, in pixel order."""
    R, t = _matrix(view, pose)
    e = (R[sc.vert_obj] @ sc.pos[:, :, None])[:, :, 0] + t[sc.vert_obj]
    w = -e[:, 2]
    X = torch.round(256 * (intr[0] * (e[:, 0] / w) + intr[2]))
    Y = torch.round(256 * (-intr[1] * (e[:, 1] / w) + intr[3]))
    ok = (w >= near) & shown[sc.vert_obj] & (X.abs() <= 2 ** 24) & (Y.abs() <= 2 ** 24)
    X, Y = torch.where(ok, X, torch.zeros_like(X)).long(), torch.where(ok, Y, torch.zeros_like(Y)).long()
    a, b, c = sc.tri[:, 0], sc.tri[:, 2], sc.tri[:, 1]  # positive area for front faces
    area = (X[b] - X[a]) * (Y[c] - Y[a]) - (Y[b] - Y[a]) * (X[c] - X[a])
    xs, ys = torch.stack([X[a], X[b], X[c]]), torch.stack([Y[a], Y[b], Y[c]])
    up = lambda v: -torch.div(128 - v, 256, rounding_mode="floor")
    dn = lambda v: torch.div(v - 128, 256, rounding_mode="floor")
    i0, i1 = up(xs.amin(0)).clamp(min=0), dn(xs.amax(0)).clamp(max=W - 1)
    j0, j1 = up(ys.amin(0)).clamp(min=0), dn(ys.amax(0)).clamp(max=H - 1)
    keep = (ok[a] & ok[b] & ok[c] & (area > 0) & (i0 <= i1) & (j0 <= j1)).nonzero()[:, 0]
    nx, n = (i1 - i0 + 1)[keep], ((i1 - i0 + 1) * (j1 - j0 + 1))[keep]
    T = torch.repeat_interleave(keep, n)
    k = torch.arange(T.numel(), device=T.device) - torch.repeat_interleave(n.cumsum(0) - n, n)
    nx = torch.repeat_interleave(nx, n)
    px, py = i0[T] + k % nx, j0[T] + torch.div(k, nx, rounding_mode="floor")
    PX, PY = 256 * px + 128, 256 * py + 128
    E, inside = [], None
    for p, q in ((b, c), (c, a), (a, b)):
        p, q = p[T], q[T]
        dx, dy = X[q] - X[p], Y[q] - Y[p]
        v = dx * (PY - Y[p]) - dy * (PX - X[p])
        top_left = (dy < 0) | ((dy == 0) & (dx > 0))
        good = (v > 0) | ((v == 0) & top_left)
        inside = good if inside is None else inside & good
        E.append(v)
    m = inside.nonzero()[:, 0]
    T, pix = T[m], (py * W + px)[m]
    E = torch.stack([v[m] for v in E], 1).double()
    q = E / torch.stack([w[a[T]], w[b[T]], w[c[T]]], 1)
    z = area[T].double() / q.sum(1)
    best = torch.full((W * H,), math.inf, dtype=torch.float64, device=T.device)
    best = best.scatter_reduce(0, pix, z, "amin")
    m = (z == best[pix]).nonzero()[:, 0]
    first = torch.full((W * H,), 2 ** 62, dtype=torch.int64, device=T.device).scatter_reduce(0, pix[m], T[m], "amin")
    m = m[T[m] == first[pix[m]]]
    m = m[torch.argsort(pix[m])]
    return pix[m], T[m], q[m], z[m], R


def _sample(tex, uv):
    """Bilinear, repeating, texel centres at (i + 1/2) / size."""
    Ht, Wt = tex.shape[0], tex.shape[1]
    x, y = uv[:, 0] * Wt - 0.5, uv[:, 1] * Ht - 0.5
    fx, fy = x.floor(), y.floor()
    ax, ay = (x - fx)[:, None], (y - fy)[:, None]
    i0, j0 = fx.long() % Wt, fy.long() % Ht
    i1, j1 = (i0 + 1) % Wt, (j0 + 1) % Ht
    return (1 - ay) * ((1 - ax) * tex[j0, i0] + ax * tex[j0, i1]) + ay * ((1 - ax) * tex[j1, i0] + ax * tex[j1, i1])


def _unit(v):
    return v / v.norm(dim=-1, keepdim=True)


def _bumped(sc, tex, uv, T, R, n):
    """Normals n replaced by a normal texture's direction in the triangles' tangent frames."""
    a, b, c = sc.tri[T, 0], sc.tri[T, 2], sc.tri[T, 1]
    e1, e2 = sc.pos[b] - sc.pos[a], sc.pos[c] - sc.pos[a]
    d1, d2 = sc.uv[b] - sc.uv[a], sc.uv[c] - sc.uv[a]
    det = d1[:, :1] * d2[:, 1:] - d2[:, :1] * d1[:, 1:]
    safe = torch.where(det == 0, torch.ones_like(det), det)
    rot = lambda v: (R @ v[:, :, None])[:, :, 0]
    tan = rot((e1 * d2[:, 1:] - e2 * d1[:, 1:]) / safe)
    bit = rot((e2 * d1[:, :1] - e1 * d2[:, :1]) / safe)
    tan = tan - (n * tan).sum(1, keepdim=True) * n
    t = 2 * _sample(tex, uv) - 1
    flat = (det[:, 0] == 0) | ((tan * tan).sum(1) == 0) | ((t * t).sum(1) == 0)
    tan = _unit(torch.where(flat[:, None], torch.ones_like(tan), tan))
    co = torch.linalg.cross(n, tan)
    co = torch.where((co * bit).sum(1, keepdim=True) < 0, -co, co)
    t = torch.where(flat[:, None], torch.ones_like(t), t)
    s = _unit(t[:, :1] * tan + t[:, 1:2] * co + t[:, 2:] * n)
    return torch.where(flat[:, None], n, s)


class _Truth:
    """A batch rendered in 64 bits."""

    def __init__(self, b):
        self.b = b
        self.dev = dev = "cuda" if torch.cuda.is_available() else "cpu"
        d = lambda a: None if a is None else torch.as_tensor(np.asarray(a), dtype=torch.float64, device=dev)
        for k in ("object_pose", "albedo", "roughness", "specular", "light_vec", "light_intensity", "view", "intr",
                  "near", "exposure", "light_dir", "light_cone", "shadow_view", "shadow_intr", "tex_xform", "emission"):
            setattr(self, k, d(getattr(b, k)))
        self.shown = torch.as_tensor(b.object_visible != 0, device=dev)
        self.textures = [d(t) for t in b.textures or []]
        self.scenes, self.maps = {}, {}

    def scene(self, s):
        if s not in self.scenes:
            self.scenes = {s: _Scene(self.b, s, self.dev)}  # frames come scene by scene
            self.maps = {}
        return self.scenes[s]

    def shadow_map(self, sc, l):
        if l not in self.maps:
            N = self.b.shadow_res
            pix, _, _, z, _ = _visible(sc, self.shadow_view[l], self.shadow_intr[l], 0.01,
                                       self.object_pose[sc.o0:sc.o1], self.shown[sc.o0:sc.o1], N, N)
            m = torch.zeros(N * N, dtype=torch.float64, device=self.dev)
            m[pix] = z
            self.maps[l] = m.view(N, N)
        return self.maps[l]

    def lit(self, sc, l, view, p):
        """Fraction of the 3 x 3 shadow-map texels around view-space points p that see light l."""
        world = (p - view[:, 3]) @ view[:, :3]
        q = world @ self.shadow_view[l][:, :3].T + self.shadow_view[l][:, 3]
        w = -q[:, 2]
        K, N = self.shadow_intr[l], self.b.shadow_res
        safe = torch.where(w > 0, w, torch.ones_like(w))
        u = torch.floor(K[0] * q[:, 0] / safe + K[2]).clamp(-4, N + 4).long()
        v = torch.floor(-K[1] * q[:, 1] / safe + K[3]).clamp(-4, N + 4).long()
        m = self.shadow_map(sc, l)
        count = torch.zeros_like(w)
        for dj in (-1, 0, 1):
            for di in (-1, 0, 1):
                x, y = u + di, v + dj
                on = (x >= 0) & (y >= 0) & (x < N) & (y < N)
                z = torch.where(on, m[y.clamp(0, N - 1), x.clamp(0, N - 1)], torch.zeros_like(w))
                count = count + ((z == 0) | (0.98 * w <= z)).double()
        return torch.where(w > 0, count / 9, torch.ones_like(w))

    def frame(self, f):
        """(covered pixels, depth, normal, rgb) of frame f."""
        b = self.b
        s, W, H = int(b.frame_scene[f]), int(b.width[f]), int(b.height[f])
        sc, view, K = self.scene(s), self.view[f], self.intr[f]
        pix, T, q, z, R = _visible(sc, view, K, self.near[f], self.object_pose[sc.o0:sc.o1],
                                   self.shown[sc.o0:sc.o1], W, H)
        obj = sc.tri_obj[T]
        corner = sc.tri[T][:, [0, 2, 1]]
        n = _unit((R[obj] @ (q[:, :, None] * sc.nrm[corner]).sum(1)[:, :, None])[:, :, 0])
        i, j = (pix % W).double(), torch.div(pix, W, rounding_mode="floor").double()
        p = torch.stack([z * (i + 0.5 - K[2]) / K[0], -z * (j + 0.5 - K[3]) / K[1], -z], 1)
        v, g = _unit(-p), obj + sc.o0
        albedo, seen = self.albedo[g], n
        total = torch.zeros_like(p)
        if self.textures:
            uv = (q[:, :, None] * sc.uv[corner]).sum(1) / q.sum(1, keepdim=True)
            uv = uv * self.tex_xform[g, :2] + self.tex_xform[g, 2:]
            ids = torch.as_tensor(b.object_texture, device=self.dev)[g]
            bumps = torch.as_tensor(b.object_normal_texture, device=self.dev)[g]
            albedo, seen = albedo.clone(), n.clone()
            for k, tex in enumerate(self.textures):
                m = (ids == k).nonzero()[:, 0]
                albedo[m] = albedo[m] * _sample(tex, uv[m])
                m = (bumps == k).nonzero()[:, 0]
                seen[m] = _bumped(sc, tex, uv[m], T[m], R[obj[m]], n[m])
            total = total + self.emission[g, None] * albedo
        power = 2 / self.roughness[g] ** 2 - 2
        for l in range(int(b.scene_light_begin[s]), int(b.scene_light_begin[s + 1])):
            kind, u = int(b.light_type[l]), self.light_vec[l]
            if kind == 1:
                to = -_unit(view[:, :3] @ u).expand_as(p)
                fall = self.light_intensity[l].expand(len(z))
            else:
                to = view[:, :3] @ u + view[:, 3] - p
                D = (to * to).sum(1)
                to = to / D.sqrt()[:, None]
                fall = self.light_intensity[l] / D.clamp(min=1e-4)
            if kind == 2:
                axis = _unit(view[:, :3] @ self.light_dir[l])
                cin, cout = self.light_cone[l]
                t = ((-(to @ axis) - cout) / (cin - cout)).clamp(0, 1)
                fall = fall * t * t * (3 - 2 * t) * self.lit(sc, l, view, p)
            nl = (seen * to).sum(1).clamp(min=0)
            nh = (seen * _unit(to + v)).sum(1)
            front = nh > 0
            s_ = torch.where(front, torch.where(front, nh, torch.ones_like(nh)) ** power, torch.zeros_like(nh))
            total = total + (fall * nl)[:, None] * (albedo + (self.specular[g] * s_)[:, None])
        return pix, z, n, total * self.exposure[f]


def _exact_images(b, names):
    """The float outputs among `names` of a batch, planar like the framework's."""
    truth = _Truth(b)
    P, po = b.total_pixels, b.pixel_offset
    planes = dict(rgb=3, depth=1, normal=3, alpha=1)
    out = {k: torch.zeros(planes[k] * P, dtype=torch.float64, device=truth.dev) for k in names if k in planes}
    for f in range(b.n_frames):
        pix, z, n, rgb = truth.frame(f)
        o, n_pix = int(po[f]), int(po[f + 1] - po[f])
        if "depth" in out:
            out["depth"][o + pix] = z
        if "alpha" in out:
            out["alpha"][o + pix] = 1.0
        for k, v in (("rgb", rgb), ("normal", n)):
            if k in out:
                for c in range(3):
                    out[k][3 * o + c * n_pix + pix] = v[:, c]
    return {k: out[k].cpu() if k in out else None for k in names}


def _exact_shade(b, grad):
    truth = _Truth(b)
    names = ("albedo", "roughness", "specular", "light_vec", "light_intensity", "exposure")
    leaves = {k: getattr(truth, k).requires_grad_() for k in names}
    rgb = torch.zeros(3 * b.total_pixels, dtype=torch.float64, device=truth.dev)
    grad, po = grad.to(truth.dev, torch.float64), b.pixel_offset
    for f in range(b.n_frames):
        pix, _, _, v = truth.frame(f)
        o, n_pix = int(po[f]), int(po[f + 1] - po[f])
        at = [3 * o + c * n_pix + pix for c in range(3)]
        for c in range(3):
            rgb[at[c]] = v[:, c].detach()
        if len(pix):
            v.backward(torch.stack([grad[a] for a in at], 1))
    out = {k: (torch.zeros_like(t) if t.grad is None else t.grad).cpu() for k, t in leaves.items()}
    return dict(out, rgb=rgb.cpu())


def exact(case, seed):
    if case["op"] == "serve":
        pool = S.config2(seed, SERVE_POOL, 200)
        return [_exact_images(_resized(pool.select_scenes(ids), res, res), CHANNELS)
                for ids, res in _requests(case, seed)]
    names = case["outputs"].split(",")
    if not {"rgb", "depth", "normal", "alpha"} & set(names):
        return None  # 8-bit and integer outputs only
    b = _batch(case, seed)
    if case["op"] == "shade":
        return _exact_shade(b, _image_gradient(b, seed))
    return _exact_images(b, names)
