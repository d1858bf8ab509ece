"""Batches that just fit the no-allocation entry point's scratch array (64 MiB): rendering some of
their frames as patches must not make them too large for it."""
import numpy as np
import pytest

from paper_1906_11633_amd import _lib as L
from paper_1906_11633_amd import scenes as S
from tests.test_patches_gpu import TILED, renderer  # noqa: F401

pytestmark = pytest.mark.gpu


def _padded(mesh, n_verts):
    """The mesh with unused vertices behind its own, n_verts in all."""
    extra = n_verts - mesh.n_verts
    return S.Mesh(np.concatenate([mesh.pos, np.repeat(mesh.pos[:1], extra, 0)]),
                  np.concatenate([mesh.nrm, np.repeat(mesh.nrm[:1], extra, 0)]), mesh.idx)


def _two_scenes(first, second, sizes):
    """Scene 0 holds mesh `first`, scene 1 `second`; frame 0 shows scene 0, the others scene 1."""
    pose = S.make_pose(S.rot_axis("x", 0.4), (0.0, 0.0, -2.0))
    b = S.single_object_batch(first, pose, extra_objects=[(second, pose)], lights=((0, (0.3, 0.4, 0.5), 1.5),) * 2,
                              spec=0.4, rough=0.5)
    n = len(sizes)
    r = lambda a: np.repeat(a, n, 0)
    return b.replace(scene_object_begin=np.array([0, 1, 2], np.int32), scene_light_begin=np.array([0, 1, 2], np.int32),
                     frame_scene=np.array([0] + [1] * (n - 1), np.int32), view=r(b.view), near=r(b.near),
                     width=np.array([w for w, _ in sizes], np.int32), height=np.array([h for _, h in sizes], np.int32),
                     intr=np.array([S.intrinsics(w, h) for w, h in sizes], np.float32),
                     exposure=np.linspace(0.7, 1.3, n).astype(np.float32))


def _largest_mesh_beside_patches():
    # vertex records of one frame, its object's, and the counters fill the array exactly
    n = (L.NOALLOC_SCRATCH_BYTES - 3 * 256) // 16
    return _two_scenes(_padded(S.box_mesh(1), n), S.box_mesh(2), [(64, 64)] + [(128, 128)] * 40)


def _more_vertex_records_than_scratch():
    # 112 kB of vertex records a frame, 2 triangles in all frames but one
    return _two_scenes(_padded(S.plane_mesh(80, 80, 1.5, 1.5), 7000), _padded(S.plane_mesh(1, 1, 1.5, 1.5), 7000),
                       [(200, 200)] + [(16, 16)] * 1000)


@pytest.mark.parametrize("make,path", [(_largest_mesh_beside_patches, 0), (_more_vertex_records_than_scratch, 2)])
def test_batches_that_fit_stay_accepted(renderer, make, path):  # noqa: F811
    import torch
    from paper_1906_11633_amd.renderer import render_batch_noalloc
    b = make()
    got = []
    for tuning in ((32, 32, 256, 0, path), TILED):
        job = renderer.prepare(b)
        job.layout.set_tuning(*tuning)
        print(f"[noalloc limit] {make.__name__} tuning={tuning} workspace={job.layout.info.workspace_bytes}", flush=True)
        out = renderer.alloc_outputs(job, vis=True, stats=True, track=True)
        for k, t in out.items():
            if k != "stats":
                t.view(torch.uint8).fill_(0x5a)
        if tuning == TILED:
            renderer.render(job, out)
        else:
            render_batch_noalloc(renderer.ctx, job.layout, job.state, out)
        torch.cuda.synchronize()
        got.append(out)
    for k in got[0]:
        if k != "stats":
            assert torch.equal(got[0][k].view(torch.uint8), got[1][k].view(torch.uint8)), k
    assert [got[0]["stats"][k].item() for k in (0, 3, 4)] == [got[1]["stats"][k].item() for k in (0, 3, 4)]
