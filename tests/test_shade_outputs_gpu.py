"""The differentiable render's image and gradients against a plain render and a plain adjoint
call on the same state, bit for bit: the pass keeps rgb and visibility only, on whole frames,
patches and the tiled path."""
import pytest
import torch

from paper_1906_11633_amd import autograd, renderer as R
from paper_1906_11633_amd import scenes as S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("frames,res,path,persistent", [(2, 67, 0, 0), (256, 100, 0, 0), (3, 90, 1, 0), (2, 300, 0, 0)])
def test_image_and_gradients(frames, res, path, persistent):
    r = R.Renderer(0)
    job = r.prepare(S.config2(21, frames, res, 1))
    job.layout.set_tuning(path=path, persistent=persistent)
    job.workspace = torch.empty(max(int(job.layout.info.workspace_bytes_any), 256), dtype=torch.uint8, device="cuda")
    params = [job.state[k].clone().requires_grad_() for k in autograd.PARAMS]
    rgb = autograd.shade(r, job, *params)
    g = torch.randn(rgb.shape, generator=torch.Generator().manual_seed(4)).cuda()
    grads = torch.autograd.grad(rgb, params, g)
    out = r.render(job, vis=True)
    want = R.shade_backward(r.ctx, job.layout, job.state, out["vis"], g)
    torch.cuda.synchronize()
    assert torch.equal(rgb.detach(), out["rgb"])
    for k, got in zip(autograd.PARAMS, grads):
        assert torch.equal(got, want[k]), k
