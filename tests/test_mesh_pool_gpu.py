"""Device memory of the mesh pool: it may grow ahead of the meshes, but by a bounded amount."""
import numpy as np
import pytest

from paper_1906_11633_amd import scenes as S

pytestmark = pytest.mark.gpu


def test_pool_grows_by_a_bounded_amount():
    """A mesh of 6 M vertices (240 MB of positions, normals and texture coordinates), then a box."""
    import torch
    from paper_1906_11633_amd.renderer import Context
    box = S.box_mesh(1)
    extra = 6_000_000 - box.n_verts
    large = S.Mesh(np.concatenate([box.pos, np.repeat(box.pos[:1], extra, 0)]),
                   np.concatenate([box.nrm, np.repeat(box.nrm[:1], extra, 0)]), box.idx)
    ctx = Context(0)
    ctx.add_mesh(large)
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info(0)[0]
    for n in (1, 2, 3):
        ctx.add_mesh(S.box_mesh(n))
    grown = before - torch.cuda.mem_get_info(0)[0]
    print(f"pool grew by {grown >> 20} MB", flush=True)
    assert grown <= 100 << 20


def test_meshes_added_while_renders_run():
    """Renders queued on another stream read the pool while meshes are added to it, with room left
    and without; renders with the added meshes see them whole."""
    import torch
    from paper_1906_11633_amd.renderer import Renderer, render_batch
    r = Renderer(0)
    b = S.with_materials(S.config2(41, 16, 200), seed=1)
    job = r.prepare(b)
    want = r.render(job, vis=True)
    outs = [r.alloc_outputs(job, vis=True) for _ in range(4)]
    stream = torch.cuda.Stream()
    torch.cuda.synchronize()
    for k in range(40):
        render_batch(r.ctx, job.layout, job.state, outs[k % 4], job.workspace, stream)
        if k % 5 == 4:
            r.ctx.add_mesh(S.capsule_mesh(0.02, 0.05, 8 + k, 8))
    torch.cuda.synchronize()
    for out in outs:
        for k in want:
            assert torch.equal(out[k].view(torch.uint8), want[k].view(torch.uint8)), k
    fresh = Renderer(0)
    c = S.config3(42, 4, 2)  # meshes of its own, behind the added ones
    got, ref = r.render(r.prepare(c), vis=True), fresh.render(fresh.prepare(c), vis=True)
    torch.cuda.synchronize()
    for k in ref:
        assert torch.equal(got[k].view(torch.uint8), ref[k].view(torch.uint8)), k
