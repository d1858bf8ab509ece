"""Vertices transformed by a wave an object (batches of 2,048 objects and more, none above
1,024 vertices) and by a workgroup an object (one above), against frames whose vertices are
transformed elsewhere, bit for bit on every output: hidden objects, objects through the camera,
a last workgroup that is not full, objects of one triangle, 1,024 and 1,025 vertices."""
import numpy as np
import pytest

from paper_1906_11633_amd import scenes as S
from tests.test_patches_gpu import _check, renderer  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("frames", [73, 74, 75])  # 28 objects each: 2,044, 2,072, 2,100 items
def test_hand(renderer, frames):  # noqa: F811
    b = S.config2(23, frames, 50, 1)
    vis, pose = b.object_visible.copy(), b.object_pose.copy()
    vis[::5] = 0
    pose[1::7, :, 3] -= 0.3
    _check(renderer, b.replace(object_visible=vis, object_pose=pose), f"{frames} frames")


@pytest.mark.parametrize("ny", [31, 40])  # 32 x 32 = 1,024 and 25 x 41 = 1,025 vertices
def test_sizes(renderer, ny):  # noqa: F811
    big = S.plane_mesh(31, 31) if ny == 31 else S.plane_mesh(24, 40)
    assert big.n_verts == (1024 if ny == 31 else 1025)
    extra = [(S.plane_mesh(1, 1, 0.1, 0.1), S.make_pose(np.eye(3), (0.1 * k - 0.4, 0.2, -1.0))) for k in range(8)]
    b = S.single_object_batch(big, S.make_pose(np.eye(3), (0, 0, -2.0)), res=(40, 40), extra_objects=extra)
    r = lambda a: np.repeat(a, 229, 0)  # 9 objects: 2,061 items
    _check(renderer, b.replace(frame_scene=r(b.frame_scene), width=r(b.width), height=r(b.height), view=r(b.view),
                               intr=r(b.intr), near=r(b.near), exposure=r(b.exposure)), f"{big.n_verts} vertices")
