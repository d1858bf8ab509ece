"""Counters of frames that the frame kernel's scratch could have taken and that are rendered as
patches (path 2): its limits follow from those scenes alone, and frames of larger ones, which
it could not have taken, count nothing."""
import numpy as np
import pytest

from paper_1906_11633_amd import scenes as S
from tests.test_noalloc_limit_gpu import _padded
from tests.test_patches_gpu import renderer  # noqa: F401

pytestmark = pytest.mark.gpu


def test_overflow_is_counted_beside_a_scene_beyond_scratch(renderer):  # noqa: F811
    """Scene 0 (two 60 x 60 planes and 100 frame-filling quads, 14,600 triangles) has over 51,200
    (tile, triangle) entries, more than the 29,200 of its scratch bins at capacity 256; scene 1
    has 51,200 triangles and more vertices than scratch holds."""
    import torch
    fine, quad = S.plane_mesh(60, 60, 2.6, 2.6), S.plane_mesh(1, 1, 3.0, 3.0)
    large = _padded(S.plane_mesh(160, 160, 1.5, 1.5), 70000)
    extra = [(fine, S.make_pose(S.rot_axis("x", 0.15), (0.0, 0.0, -2.3)))]
    extra += [(quad, S.make_pose(S.rot_axis("y", 0.01 * k), (0.0, 0.0, -2.5 - 0.01 * k))) for k in range(100)]
    extra += [(large, S.make_pose(np.eye(3), (0.0, 0.0, -2.0)))]
    b = S.single_object_batch(fine, S.make_pose(np.eye(3), (0.0, 0.0, -2.0)), res=(256, 256), extra_objects=extra,
                              lights=((0, (0.3, 0.4, 0.5), 1.5),) * 2, spec=0.4, rough=0.5)
    r = lambda a: np.repeat(a, 2, 0)
    b = b.replace(scene_object_begin=np.array([0, 102, 103], np.int32), scene_light_begin=np.array([0, 1, 2], np.int32),
                  frame_scene=np.array([0, 1], np.int32), width=r(b.width), height=r(b.height), view=r(b.view),
                  intr=r(b.intr), near=r(b.near), exposure=r(b.exposure))
    job = renderer.prepare(b)
    job.layout.set_tuning(32, 32, 256, 0, 2)
    out = renderer.alloc_outputs(job, stats=True)
    renderer.render(job, out)
    torch.cuda.synchronize()
    stats = out["stats"].tolist()
    print(stats, flush=True)
    assert stats[:3] == [0, 1, 0]
