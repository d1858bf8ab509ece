"""The autotuner times each different way to render the batch once: patches are tried, and tile
shapes are swept only where frames are left to the tiled path.  A vertex nearer than the near
plane counts once in every render, so the call's counter tells how many renders it made."""
import numpy as np
import pytest

from paper_1906_11633_amd import scenes as S
from tests.test_patches_gpu import renderer  # noqa: F401

pytestmark = pytest.mark.gpu

RENDERS = 4  # per candidate: one to warm up, three timed
SWEEP = 16   # four tile shapes, two bin capacities, persistent or not

SMALL, LARGE, TILED = (600, 4000), (16000, 30000), (70000, 80000)  # triangles: LDS, beyond, tiled only


def _scenes(kinds, n_each):
    """n_each scenes of every kind, one frame each, with one object through the camera."""
    parts = [S.config3(30 + k, n_each, 1, min_tris=lo, max_tris=hi) for k, (lo, hi) in enumerate(kinds)]
    b = parts[0]
    for p in parts[1:]:
        cat = lambda k: np.concatenate([getattr(b, k), getattr(p, k)])
        off = lambda k, add: np.concatenate([getattr(b, k), getattr(p, k)[1:] + add])
        assert len(b.meshes) == len(p.meshes)
        b = b.replace(scene_object_begin=off("scene_object_begin", b.n_objects),
                      scene_light_begin=off("scene_light_begin", b.n_lights),
                      frame_scene=np.concatenate([b.frame_scene, p.frame_scene + b.n_scenes]),
                      **{k: cat(k) for k in ("object_mesh", "light_type", "width", "height", "object_pose", "object_seg",
                                             "object_visible", "albedo", "roughness", "specular", "light_vec",
                                             "light_intensity", "view", "intr", "near", "exposure")})
    pose = b.object_pose.copy()
    first = b.scene_object_begin[:-1][b.frame_scene]
    pose[first, :, 3] = -np.einsum("fji,fj->fi", b.view[:, :, :3], b.view[:, :, 3])
    return b.replace(object_pose=pose)


@pytest.mark.parametrize("kinds,n_each,want", [
    ([SMALL], 4, 1 + SWEEP),                    # path 0 as patches, path 1
    ([LARGE], 4, 1 + SWEEP),                    # likewise; path 2 launches what path 0 does
    ([SMALL, LARGE], 3, 1 + SWEEP),             # likewise: no frame is left to the tiled path
    ([LARGE], 400, 1 + SWEEP + 3),              # path 2 on scratch, three bin capacities
    ([TILED], 2, SWEEP),                        # path 1 only
    ([SMALL, TILED], 2, 2 * SWEEP),             # path 0 leaves frames to the tiled path
], ids=["small", "large", "mixed", "large on scratch", "tiled", "small and tiled"])
def test_candidates(renderer, kinds, n_each, want):  # noqa: F811
    import torch
    from paper_1906_11633_amd.renderer import autotune
    b = _scenes(kinds, n_each)
    job = renderer.prepare(b)
    one = renderer.render(job, stats=True)
    out = renderer.alloc_outputs(job, stats=True)
    tuning, ms = autotune(renderer.ctx, job.layout, job.state, out, job.workspace)
    torch.cuda.synchronize()
    per_render, total = int(one["stats"][3]), int(out["stats"][3])
    print(f"[candidates] {kinds} x {n_each}: {tuning} {ms:.3f} ms, {per_render} near vertices, {total}", flush=True)
    assert per_render > 0 and total == want * RENDERS * per_render
    for k in ("rgb", "depth", "normal", "seg"):
        assert torch.equal(out[k], one[k]), k
