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
