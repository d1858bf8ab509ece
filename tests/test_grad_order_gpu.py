"""The adjoint's tiles in runs a frame long: each frame's exposure gradient, whose sum is over
that frame's tiles alone, equals the one the frame has in a call of its own, bit for bit, for
frames of different sizes and counts around sets of eight runs."""
import numpy as np
import pytest
import torch

from paper_1906_11633_amd import renderer as R
from paper_1906_11633_amd import scenes as S
from tests.test_patches_gpu import _resized

pytestmark = pytest.mark.gpu


def _exposure_gradient(r, b, g):
    job = r.prepare(b)
    out = r.render(job, vis=True)
    return R.shade_backward(r.ctx, job.layout, job.state, out["vis"], g)["exposure"]


@pytest.mark.parametrize("sizes", [[(64, 64)], [(33, 31), (100, 40), (64, 97)]])
@pytest.mark.parametrize("frames", [1, 7, 8, 9, 17])
def test_frames_alone(frames, sizes):
    r = R.Renderer(0)
    b = _resized(S.config2(29, frames, 64, 1), sizes)
    P = (b.width.astype(np.int64) * b.height).tolist()
    g = torch.randn(3 * sum(P), generator=torch.Generator().manual_seed(1)).cuda()
    got = _exposure_gradient(r, b, g)
    at = 0
    for f in range(frames):
        one = {k: getattr(b, k)[f:f + 1] for k in ("frame_scene", "width", "height", "view", "intr", "near", "exposure")}
        alone = _exposure_gradient(r, b.replace(**one), g[3 * at:3 * (at + P[f])].contiguous())
        assert torch.equal(got[f:f + 1], alone), f
        at += P[f]
