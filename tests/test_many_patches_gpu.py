"""Batches of more patches than one launch may start: a launch holds fewer than 2^32 threads,
4,194,303 workgroups of a patch's 1,024."""
import numpy as np
import pytest

from paper_1906_11633_amd import scenes as S
from tests.test_patches_gpu import TILED, renderer  # noqa: F401

pytestmark = pytest.mark.gpu


def test_more_frames_than_one_launch_of_patches(renderer):  # noqa: F811
    """2^22 + 3 frames of 3 x 3 pixels, a patch each, with exposures and positions of their
    own, against the tiled path."""
    import torch
    n = (1 << 22) + 3
    b = S.single_object_batch(S.box_mesh(1), S.make_pose(np.eye(3), (0.0, 0.0, -3.0)), res=(3, 3),
                              lights=((0, (0.3, 0.4, 0.5), 1.5),), spec=0.4, rough=0.5)
    r = lambda a: np.repeat(a, n, 0)
    view = r(b.view)
    view[:, 0, 3] = np.linspace(-0.8, 0.8, n)
    b = b.replace(frame_scene=r(b.frame_scene), width=r(b.width), height=r(b.height), view=view, intr=r(b.intr), near=r(b.near),
                  exposure=np.linspace(0.7, 1.3, n).astype(np.float32))
    got = []
    for tuning in ((32, 32, 256, 0, 0), TILED):
        job = renderer.prepare(b)
        job.layout.set_tuning(*tuning)
        print(f"[many] frames={n} tuning={tuning}", flush=True)
        out = renderer.alloc_outputs(job, vis=True, track=True)
        for t in out.values():
            t.view(torch.uint8).fill_(0x5a)
        renderer.render(job, out)
        torch.cuda.synchronize()
        got.append(out)
    for k in got[0]:
        assert torch.equal(got[0][k].view(torch.uint8), got[1][k].view(torch.uint8)), k
    assert int((got[0]["seg"] >= 0).sum()) > n
