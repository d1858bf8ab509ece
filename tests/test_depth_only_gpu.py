"""Alpha and Tracker records of calls that ask for no shaded channel, from whole frames, patches
and the tiled path: the same as beside all channels."""
import pytest
import torch

from paper_1906_11633_amd import renderer as R
from paper_1906_11633_amd import scenes as S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("frames,res,path", [(256, 100, 0), (2, 60, 0), (2, 60, 1), (256, 100, 2)])
def test_alpha_and_track(frames, res, path):
    r = R.Renderer(0)
    job = r.prepare(S.config2(25, frames, res, 1))
    job.layout.set_tuning(path=path)
    job.workspace = torch.empty(max(int(job.layout.info.workspace_bytes_any), 256), dtype=torch.uint8, device="cuda")
    want = r.render(job, alpha=True, track=True)
    out = r.alloc_outputs(job, base=("depth", "seg"), alpha=True, track=True)
    for t in out.values():
        t.view(torch.uint8).fill_(0x5a)
    r.render(job, out)
    torch.cuda.synchronize()
    for k in out:
        assert torch.equal(out[k], want[k]), k
