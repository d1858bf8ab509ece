"""The patch kernel (rectangles of frames: small batches and frames beyond 256 x 256) against
the tiled path, bit for bit on every output, at the sizes and contents where it can go
wrong: patches of one pixel, odd widths and heights, one-column and one-row frames, frames cut
in two dimensions, objects that cross the near plane, the guard band or the frame's edge,
poses that are no similarity (the object cull has to hold for any affine pose), hidden
objects, no objects and no lights, more large triangles than the queue holds, and every
shading variant with every output.  Both paths use the same arithmetic, so nothing may
differ."""
import numpy as np
import pytest

from paper_1906_11633_amd import scenes as S

pytestmark = pytest.mark.gpu

TILED = (32, 32, 256, 0, 1)


@pytest.fixture(scope="module")
def renderer():
    import torch
    from paper_1906_11633_amd.renderer import Renderer
    assert torch.cuda.is_available()
    return Renderer(0)


def _resized(b, sizes):
    """Frame k with size sizes[k % len]."""
    wh = [sizes[k % len(sizes)] for k in range(b.n_frames)]
    return b.replace(width=np.array([w for w, _ in wh], np.int32), height=np.array([h for _, h in wh], np.int32),
                     intr=np.array([S.intrinsics(w, h) for w, h in wh], np.float32))


def _both(renderer, b, name, path):
    """Every output from `path` (patches) and from the tiled path, as numpy arrays."""
    import torch
    got = []
    for tuning in ((32, 32, 512, 0, path), TILED):
        job = renderer.prepare(b)
        job.layout.set_tuning(*tuning)
        inf = job.layout.info
        print(f"[patches] {name} frames={b.n_frames} tuning={tuning} frame_path={inf.frame_path_frames}", flush=True)
        out = renderer.alloc_outputs(job, tri_id=True, vis=True, stats=True, alpha=True, rgb8=True, track=True)
        for k, t in out.items():
            if k != "stats":
                t.view(torch.uint8).fill_(0x5a)
        renderer.render(job, out)
        torch.cuda.synchronize()
        got.append({k: t.view(torch.uint8).cpu().numpy() if k != "stats" else t.cpu().numpy() for k, t in out.items()})
    return got


def _check(renderer, b, name, path=0):
    got, want = _both(renderer, b, name, path)
    for k in want:
        if k == "stats":  # wait timeouts, near and guard vertices
            assert [got[k][w] for w in (0, 3, 4)] == [want[k][w] for w in (0, 3, 4)], (name, got[k], want[k])
        else:
            assert np.array_equal(got[k], want[k]), (name, k, int((got[k] != want[k]).sum()))


SIZES = {
    "one-pixel": [(1, 1)],
    "one-column": [(1, 131)],
    "one-row": [(131, 1)],
    "odd": [(3, 5), (63, 65), (65, 63), (7, 200)],
    "edges": [(64, 64), (128, 53), (200, 34), (256, 256)],
    "past-256": [(257, 256), (256, 257), (300, 41), (260, 700)],
    "wide": [(2500, 9), (9, 2500)],
}


@pytest.mark.parametrize("name", list(SIZES))
def test_sizes(renderer, name):
    _check(renderer, S.with_postprocessing(_resized(S.config2(3, 2, 100, 2), SIZES[name]), seed=1), name)


@pytest.mark.parametrize("kind", ["plain", "spot", "materials", "both"])
def test_shading_variants(renderer, kind):
    b = S.config2(4, 2, 96, 2)
    if kind in ("materials", "both"):
        b = S.with_materials(b, seed=3)
    if kind in ("spot", "both"):
        b = S.with_spot_lights(b, seed=4)
    _check(renderer, S.with_postprocessing(b, seed=5), kind)


def test_hidden_objects_and_frames_that_see_nothing(renderer):
    b = S.config2(5, 3, 90, 2)
    vis = b.object_visible.copy()
    vis[::3] = 0
    view = b.view.copy()
    view[1, :, 3] += np.array([0.0, 0.0, 50.0], np.float32)   # behind the camera
    view[2, 0, 3] += 3.0                                       # off to the side
    _check(renderer, b.replace(object_visible=vis, view=view), "hidden")


def test_near_plane_and_guard_band(renderer):
    """Objects through the camera: vertices behind it, nearer than the near plane and beyond
    the guard band, next to ones that are wholly in view."""
    b = S.config2(6, 2, 120, 2)
    pose = b.object_pose.copy()
    view = b.view.copy()
    eye = -np.einsum("fji,fj->fi", view[:, :, :3], view[:, :, 3])
    pose[:6, :, 3] = eye[0] + np.linspace(-0.02, 0.02, 6)[:, None]
    strip = S.plane_mesh(2, 1, 40.0, 0.01)
    extra = [(strip, S.make_pose(np.eye(3), (0.0, 0.015, -0.06))), (S.box_mesh(4), S.make_pose(np.eye(3), (0, 0, -0.4), 0.05))]
    _check(renderer, b.replace(object_pose=pose), "through the camera")
    _check(renderer, S.single_object_batch(strip, S.make_pose(np.eye(3), (0.0, 0.0, -0.03)), res=(300, 96),
                                           extra_objects=extra), "strips")


def test_poses_that_are_no_similarity(renderer):
    rng = np.random.default_rng(8)
    b = S.config2(7, 2, 110, 2)
    pose = b.object_pose.copy()
    pose[:, :, :3] = pose[:, :, :3] @ (np.eye(3) + rng.uniform(-0.8, 0.8, (b.n_objects, 3, 3))).astype(np.float32)
    _check(renderer, b.replace(object_pose=pose), "affine")


def test_no_lights_and_no_objects(renderer):
    b = S.config2(9, 2, 70, 1)
    _check(renderer, b.replace(scene_light_begin=np.zeros(3, np.int32), light_type=np.zeros(0, np.int32),
                               light_vec=np.zeros((0, 3), np.float32), light_intensity=np.zeros(0, np.float32)), "no lights")
    n = int(b.scene_object_begin[1])
    one = b.replace(scene_object_begin=np.array([0, 0, n], np.int32), object_mesh=b.object_mesh[:n],
                    **{k: getattr(b, k)[:n] for k in ("object_pose", "object_seg", "object_visible", "albedo", "roughness",
                                                      "specular")})
    _check(renderer, one, "no objects in one scene")


@pytest.mark.parametrize("n_obj,n,res", [(48, 3, 200), (1, 50, 256), (2, 40, 900), (12, 12, 640)])
def test_many_large_triangles(renderer, n_obj, n, res):
    """Overlapping planes: the most objects a scene may have, and more triangles of more
    than a few pixels in a patch than its queue holds (1,024), some beyond 64 pixels."""
    planes = [S.plane_mesh(n, n, 2.0, 2.0) for _ in range(n_obj)]
    pose = lambda k: S.make_pose(S.rot_axis("y", 0.04 * k), (0.01 * k, 0.0, -2.0 - 0.02 * k))
    b = S.single_object_batch(planes[0], pose(0), res=(res, res), rough=0.5, spec=0.4,
                              extra_objects=[(m, pose(k + 1)) for k, m in enumerate(planes[1:])],
                              lights=((0, (0.3, 0.4, 0.5), 1.5),))
    _check(renderer, b, f"planes {n_obj} x {2 * n * n}")


def _large_scenes(kind):
    if kind == "uneven":        # scenes on both sides of what fits in LDS
        return S.config3(14, 6, 2, min_tris=4000, max_tris=30000)
    if kind == "past-256":      # larger frames of larger scenes
        return _resized(S.config3(15, 2, 2, min_tris=16000, max_tris=20000), [(300, 200), (512, 70), (33, 400)])
    if kind == "127-objects":   # more than one group of 64 objects, the last of them in view
        box, cap = S.box_mesh(4), S.capsule_mesh(0.02, 0.05, 16, 8)
        rng = np.random.default_rng(16)
        pose = lambda k: S.make_pose(S.uniform_rotation(rng), rng.uniform(-0.4, 0.4, 3) - [0, 0, 1.2], 0.1 if k % 2 else 2.0)
        return S.single_object_batch(box, S.make_pose(np.eye(3), (0, 0, -1.0), 0.1), res=(200, 200), rough=0.5, spec=0.4,
                                     extra_objects=[(box if k % 2 else cap, pose(k)) for k in range(126)],
                                     lights=((0, (0.3, 0.4, 0.5), 1.5),))
    b = S.config3(17, 3, 2, min_tris=9000, max_tris=14000)
    vis = b.object_visible.copy()
    vis[::3] = 0
    view = b.view.copy()
    view[1, :, 3] += np.array([0.0, 0.0, 50.0], np.float32)
    return S.with_spot_lights(S.with_materials(b.replace(object_visible=vis, view=view), seed=2), seed=3)


@pytest.mark.parametrize("path", [0, 2])
@pytest.mark.parametrize("kind", ["uneven", "past-256", "127-objects", "every-feature"])
def test_scenes_beyond_lds(renderer, kind, path):
    """Patches that read the vertex kernel's records instead of LDS."""
    b = _large_scenes(kind)
    nv = [sum(b.meshes[m].n_verts for m in b.object_mesh[o0:o1]) for o0, o1 in
          zip(b.scene_object_begin[:-1], b.scene_object_begin[1:])]
    assert max(nv) > 6976 or np.diff(b.scene_object_begin).max() > 48
    _check(renderer, S.with_postprocessing(b, seed=4), kind, path)


def test_uneven_small_batch(renderer):
    """Frames of different sizes and costs in one call: cut into different numbers of patches."""
    b = S.config3(11, 9, 2, min_tris=600, max_tris=6000)
    _check(renderer, S.with_postprocessing(b, seed=2), "uneven")


@pytest.mark.parametrize("frames", [255, 256, 257, 300])
def test_last_round_of_a_uniform_batch(renderer, frames):
    """Whole rounds of frames on the frame kernel, the rest as patches (57 and 300 - 256
    frames), in one call."""
    _check(renderer, S.config2(12, frames, 72, 1), f"{frames} frames")


def test_graph_replays(renderer):
    """A captured call with patches, replayed with eager work and other exposures between."""
    import torch
    from paper_1906_11633_amd.renderer import Graph
    b = S.with_postprocessing(S.config2(13, 2, 150, 3), seed=1)
    job = renderer.prepare(b)
    out = renderer.alloc_outputs(job, track=True, stats=True, rgb8=True)
    s = torch.cuda.Stream()
    torch.cuda.synchronize()
    g = Graph(renderer.ctx, job.layout, job.state, out, job.workspace, s)
    for k in range(4):
        job.state["exposure"].mul_(1.25)
        want = renderer.render(job, track=True, rgb8=True)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        for name in want:
            assert torch.equal(out[name], want[name]), (k, name)
        _ = torch.randn(1000, device="cuda").sum().item()
    assert int(out["stats"][0]) == 0
    g.close()


@pytest.mark.parametrize("frames,res", [(56, 90), (58, 90), (78, 61), (126, 256), (114, 61), (117, 61), (104, 130), (106, 130), (129, 130), (150, 61), (152, 61)])
def test_grids_of_middle_batches(renderer, frames, res):
    """Both sides of each line between strips, pairs of rows, several columns and the fewest."""
    _check(renderer, S.config2(14, frames, res, 1), f"{frames} frames of {res}")
