"""Frames claimed at run time (more frames than CUs, unequal costs) whose tile bins overflow, so
that their tiles are worked through in groups: a workgroup has to claim its next frame once
per frame, however few tiles the last group holds, or frames stay unrendered.  Every frame
against the tiled path, bit for bit, in destinations that start out filled."""
import numpy as np
import pytest

from paper_1906_11633_amd import scenes as S
from tests.test_patches_gpu import TILED, _resized, renderer  # noqa: F401

pytestmark = pytest.mark.gpu

PLAIN = {}
EVERY = dict(tri_id=True, vis=True, alpha=True, rgb8=True, track=True)


def _render(renderer, b, tuning, outputs):  # noqa: F811
    import torch
    job = renderer.prepare(b)
    job.layout.set_tuning(*tuning)
    print(f"[groups] {b.name} frames={b.n_frames} tuning={tuning}", flush=True)
    out = renderer.alloc_outputs(job, stats=True, **outputs)
    for k, t in out.items():
        if k != "stats":
            t.view(torch.uint8).fill_(0x5a)
    renderer.render(job, out)
    torch.cuda.synchronize()
    return {k: t.view(torch.uint8).cpu().numpy() if k != "stats" else t.cpu().numpy() for k, t in out.items()}


def _check(renderer, b, tuning, outputs):  # noqa: F811
    got, want = _render(renderer, b, tuning, outputs), _render(renderer, b, TILED, outputs)
    print(got["stats"], want["stats"], flush=True)
    assert got["stats"][0] == 0 and got["stats"][1] > 0  # no wait timed out, bins overflowed
    for k in want:
        if k != "stats":
            assert np.array_equal(got[k], want[k]), (k, int((got[k] != want[k]).sum()))


@pytest.mark.parametrize("outputs", [PLAIN, EVERY], ids=["plain", "every"])
def test_hand_frames_of_mixed_sizes(renderer, outputs):  # noqa: F811
    b = _resized(S.config2(2, 256, 256, 3), [(64, 64), (128, 128), (200, 200), (256, 256)])
    assert b.n_frames > 256
    _check(renderer, S.with_postprocessing(b, seed=1), (32, 32, 512, 0, 0), outputs)


@pytest.mark.parametrize("outputs", [PLAIN, EVERY], ids=["plain", "every"])
def test_scratch_held_frames_of_mixed_heights(renderer, outputs):  # noqa: F811
    """Scenes beyond LDS (two 60 x 60 planes and 100 frame-filling quads) under path 2: some 80
    tiles' entries fit the scratch bins, and heights in steps of a row of tiles leave last
    groups of every size."""
    fine, quad = S.plane_mesh(60, 60, 2.6, 2.6), S.plane_mesh(1, 1, 3.0, 3.0)
    extra = [(fine, S.make_pose(S.rot_axis("x", 0.15), (0.0, 0.0, -2.3), 1.0))]
    extra += [(quad, S.make_pose(S.rot_axis("y", 0.01 * k), (0.0, 0.0, -2.5 - 0.01 * k), 1.0)) for k in range(100)]
    b = S.single_object_batch(fine, S.make_pose(np.eye(3), (0.0, 0.0, -2.0), 1.0), res=(256, 256), extra_objects=extra,
                              lights=((0, (0.3, 0.4, 0.5), 1.5),), spec=0.4, rough=0.5)
    n = 400
    r = lambda a: np.repeat(a, n, 0)
    b = b.replace(frame_scene=r(b.frame_scene), width=r(b.width), height=r(b.height), view=r(b.view), intr=r(b.intr),
                  near=r(b.near), exposure=np.linspace(0.7, 1.3, n).astype(np.float32))
    b = _resized(b, [(256, h) for h in range(176, 257, 4)])
    _check(renderer, S.with_postprocessing(b, seed=1), (32, 32, 256, 0, 2), outputs)
