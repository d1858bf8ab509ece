"""Batches just large enough for the frame kernel to render their frames whole, at the contents its
fallbacks are for (fewer frames become patches, which have none), and both sides of the lines
between whole frames, patches and a last round of patches.  Every output against the tiled
path, bit for bit, and the choice itself: a layout of whole frames needs no workspace beyond
its 256 bytes of counters, patches that share a frame need sums, and each kernel is a launch."""
import numpy as np
import pytest

from paper_1906_11633_amd import scenes as S
from tests.test_frame_groups_gpu import FRAMES, _repeat
from tests.test_patches_gpu import TILED, _both, _resized, renderer  # noqa: F401

pytestmark = pytest.mark.gpu

WHOLE, PATCHES, SPLIT = (1, False), (1, True), (2, True)  # launches, sums (of calls with few or many bytes to write)


def _check(renderer, b, name, tuning, kind):  # noqa: F811
    job = renderer.prepare(b)
    job.layout.set_tuning(*tuning)
    inf = job.layout.info
    assert inf.frame_path_frames == b.n_frames
    assert (inf.render_kernels, tuning[4] == 0 and inf.workspace_bytes > 256) == kind, name
    assert tuning[2] == 512
    got, want = _both(renderer, b, name, tuning[4])
    for k in want:
        if k != "stats":
            assert np.array_equal(got[k], want[k]), (name, k, int((got[k] != want[k]).sum()))
    assert got["stats"][0] == 0
    return got["stats"]


def _few_outputs(renderer, b):  # noqa: F811
    """Depth alone and 8-bit RGB alone, which write few bytes, against the tiled path."""
    import torch
    b = S.with_postprocessing(b, seed=3)
    for kw in (dict(base=("depth",)), dict(base=(), rgb8=True)):
        got = []
        for tuning in ((32, 32, 512, 0, 0), TILED):
            job = renderer.prepare(b)
            job.layout.set_tuning(*tuning)
            out = renderer.alloc_outputs(job, **kw)
            for t in out.values():
                t.view(torch.uint8).fill_(0x5a)
            got.append(renderer.render(job, out))
        torch.cuda.synchronize()
        for k in got[0]:
            assert torch.equal(got[0][k].view(torch.uint8), got[1][k].view(torch.uint8)), k


def test_survivor_overflow_of_whole_frames(renderer):  # noqa: F811
    """6,498 front-facing triangles a frame (6,144 are remembered), 7,424 bin entries (7,680 fit)."""
    b = S.single_object_batch(S.plane_mesh(57, 57, 0.7, 0.7), S.make_pose(np.eye(3), (0.0, 0.0, -2.0), 1.0), res=(200, 200),
                              lights=((0, (0.3, 0.4, 0.5), 1.5),), spec=0.4, rough=0.5)
    st = _check(renderer, _repeat(b), "survivors", (32, 32, 512, 0, 0), WHOLE)
    assert st[1] == 0 and st[2] == FRAMES


def test_bin_overflow_of_whole_frames(renderer):  # noqa: F811
    mesh, R = S.plane_mesh(47, 47, 3.2, 3.2), S.rot_axis("x", 0.2)
    extra = [(mesh, S.make_pose(R, (0.02, -0.03, -2.2), 1.0)), (mesh, S.make_pose(R.T, (-0.01, 0.02, -2.4), 1.0))]
    b = S.single_object_batch(mesh, S.make_pose(np.eye(3), (0.0, 0.0, -2.0), 1.0), res=(256, 256), extra_objects=extra,
                              lights=((0, (0.3, 0.4, 0.5), 1.5),), spec=0.4, rough=0.5)
    st = _check(renderer, _repeat(b), "bins", (32, 32, 512, 0, 0), WHOLE)
    assert st[1] == FRAMES and st[2] == 0


def _entries(b):
    """(tile, triangle) pairs of a one-frame batch, from FP64 projections snapped to 1/256 pixel:
    front-facing triangles with a pixel centre in range, 64 x 4 tiles."""
    W, H = int(b.width[0]), int(b.height[0])
    V, K, n = b.view[0].astype(float), b.intr[0].astype(float), 0
    for k, m in enumerate(b.object_mesh):
        P, mesh = b.object_pose[k].astype(float), b.meshes[m]
        q = (mesh.pos.astype(float) @ P[:, :3].T + P[:, 3]) @ V[:, :3].T + V[:, 3]
        X = np.rint(256 * (K[0] * q[:, 0] / -q[:, 2] + K[2]))
        Y = np.rint(256 * (K[3] - K[1] * q[:, 1] / -q[:, 2]))
        x, y = X[mesh.idx], Y[mesh.idx]
        area = (x[:, 1] - x[:, 0]) * (y[:, 2] - y[:, 0]) - (y[:, 1] - y[:, 0]) * (x[:, 2] - x[:, 0])
        lo = lambda v: np.maximum(np.ceil((v.min(1) - 128) / 256), 0)
        hi = lambda v, size: np.minimum(np.floor((v.max(1) - 128) / 256), size - 1)
        i0, i1, j0, j1 = lo(x), hi(x, W), lo(y), hi(y, H)
        keep = (area < 0) & (i0 <= i1) & (j0 <= j1)  # counter-clockwise with y down
        n += int((((i1 // 64 - i0 // 64 + 1) * (j1 // 4 - j0 // 4 + 1))[keep]).sum())
    return n


@pytest.mark.parametrize("quads", [40, 100, 119])
def test_scratch_bins_of_whole_frames(renderer, quads):  # noqa: F811
    """Two 60 x 60 planes before frame-filling quads: entries on both sides of the four per triangle
    that scratch holds at capacity 512."""
    fine, quad = S.plane_mesh(60, 60, 2.6, 2.6), S.plane_mesh(1, 1, 3.0, 3.0)
    extra = [(fine, S.make_pose(S.rot_axis("x", 0.15), (0.0, 0.0, -2.3), 1.0))]
    extra += [(quad, S.make_pose(S.rot_axis("y", 0.01 * k), (0.0, 0.0, -2.5 - 0.01 * k), 1.0)) for k in range(quads)]
    b = S.single_object_batch(fine, S.make_pose(np.eye(3), (0.0, 0.0, -2.0), 1.0), res=(256, 256), extra_objects=extra,
                              lights=((0, (0.3, 0.4, 0.5), 1.5),), spec=0.4, rough=0.5)
    entries, bins = _entries(b), 4 * (2 * 7200 + 2 * quads)
    print(f"[scratch] {quads} quads: {entries} entries, {bins} bins", flush=True)
    assert (entries > bins) == (quads >= 100)
    st = _check(renderer, _repeat(b), f"scratch bins, {quads} quads", (32, 32, 512, 0, 2), WHOLE)
    assert st[1] == (FRAMES if entries > bins else 0), st


@pytest.mark.parametrize("size,frames,kind", [
    ((90, 90), 134, PATCHES), ((90, 90), 135, PATCHES), ((90, 90), 150, PATCHES), ((90, 90), 151, WHOLE), ((90, 90), 256, WHOLE),
    ((90, 90), 257, SPLIT), ((90, 90), 320, SPLIT), ((90, 90), 321, WHOLE), ((90, 90), 512, WHOLE),
    ((200, 200), 134, PATCHES), ((200, 200), 135, PATCHES), ((200, 200), 192, PATCHES), ((200, 200), 193, WHOLE),
    ((200, 200), 320, SPLIT), ((200, 200), 321, WHOLE)])
def test_rounds_of_a_uniform_batch(renderer, size, frames, kind):  # noqa: F811
    """Frames of more than one patch: all patches (of one cut or another, by the bytes that a call
    writes), whole frames, or whole rounds and the rest as patches.  256 CUs."""
    b = _resized(S.config2(12, frames, 90, 1), [size])
    _check(renderer, b, f"{frames} frames of {size}", (32, 32, 512, 0, 0), kind)
    _few_outputs(renderer, b)
