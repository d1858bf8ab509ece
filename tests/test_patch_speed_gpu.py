"""Patches of large frames write their outputs at least as fast as the tiled path does, into
buffers that are new in every call (columns write parts of 128-byte lines and fell behind it by up
to a factor of two).  Times of both paths in turn, the least of each; 15 % are allowed."""
import numpy as np
import pytest

from paper_1906_11633_amd import scenes as S
from tests.test_patches_gpu import TILED, _resized, renderer  # noqa: F401

pytestmark = pytest.mark.gpu


def _hidden(n):
    b = S.config2(5, n, 200, 1)
    return b.replace(object_visible=np.zeros_like(b.object_visible))


@pytest.mark.parametrize("make,n,size", [(_hidden, 48, (512, 512)), (_hidden, 200, (300, 300)),
                                         (_hidden, 128, (200, 200)), (lambda n: S.config1(5, n, 64), 100, (512, 512)),
                                         (lambda n: S.config2(5, n, 200, 1), 24, (1920, 1080))],
                         ids=["nothing in view", "nothing in view, 300", "nothing in view, 200", "boxes", "hands"])
def test_large_frames_in_new_buffers(renderer, make, n, size):  # noqa: F811
    import torch
    b = _resized(make(n), [size])
    jobs = {}
    for name, tuning in (("patches", (32, 32, 256, 0, 0)), ("tiled", TILED)):
        jobs[name] = renderer.prepare(b)
        jobs[name].layout.set_tuning(*tuning)
    outs = [renderer.alloc_outputs(jobs["tiled"]) for _ in range(2)]
    best = dict(patches=1e9, tiled=1e9)
    for _ in range(5):
        for name, job in jobs.items():
            renderer.render(job, outs[0])
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            for k in range(6):
                renderer.render(job, outs[(k + 1) % 2])
            e1.record()
            torch.cuda.synchronize()
            best[name] = min(best[name], e0.elapsed_time(e1) / 6)
    print(size, n, {k: f"{1e3 * v:.0f} us" for k, v in best.items()}, flush=True)
    assert best["patches"] <= 1.15 * best["tiled"]
