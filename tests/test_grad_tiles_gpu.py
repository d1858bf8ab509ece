"""Edges of the adjoint kernel's 32 x 32 tiles and of its rounds of 64 object slots,
through properties that hold exactly or to the rounding of the results:

* an upstream gradient that is zero outside one object's pixels gives that object the
  same bits as the full gradient (its terms are added in the same places), and every
  other object exact zeros;
* the gradients of the tiles taken one at a time add up to the whole (each result is
  an FP64 sum rounded once to fp32, so within 2^-23 of the absolute parts);
* a frame that sees nothing gives exact zeros.

(test_grad_gpu.py compares the values with the oracle.)"""
import numpy as np
import pytest

import oracle
from paper_1906_11633_amd import scenes as S

pytestmark = pytest.mark.gpu

OBJECT_KINDS = ("albedo", "roughness", "specular")
TILE = 32


@pytest.fixture(scope="module")
def renderer():
    import torch
    from paper_1906_11633_amd.renderer import Renderer
    assert torch.cuda.is_available()
    return Renderer(0)


def _grid(n, res):
    """n x n small boxes in front of the camera, every one in view, three lights."""
    box = S.box_mesh(1)
    at = [((i - (n - 1) / 2) / n, (j - (n - 1) / 2) / n) for j in range(n) for i in range(n)]
    poses = [S.make_pose(S.rot_axis("x", 0.3) @ S.rot_axis("y", 0.4), (0.7 * x, 0.7 * y, -1.0), 0.5 / n) for x, y in at]
    return S.single_object_batch(box, poses[0], res=(res, res), extra_objects=[(box, p) for p in poses[1:]], rough=0.5,
                                 spec=0.3, lights=((0, (0.2, 0.3, 0.4), 1.0), (1, (0.1, -0.2, -1.0), 0.7),
                                                   (0, (-0.5, 0.1, 0.2), 1.5)))


def _hand(width, height):
    b = S.config2(2, 1, height)
    intr = np.tile(S.intrinsics(width, height), (b.n_frames, 1)).astype(np.float32)
    return b.replace(width=np.full(b.n_frames, width, np.int32), height=np.full(b.n_frames, height, np.int32), intr=intr)


def _plane(width, height, n_lights):
    rng = np.random.default_rng(5)
    lights = [(k % 2, tuple(rng.uniform(-0.5, 0.5, 2)) + ((0.2,) if k % 2 == 0 else (-1.0,)), 0.5 + 0.2 * k)
              for k in range(n_lights)]
    return S.single_object_batch(S.plane_mesh(3, 3, 9.0, 9.0), S.make_pose(S.rot_axis("x", 0.2), (0.0, 0.0, -2.0)),
                                 res=(width, height), rough=0.4, spec=0.5, lights=tuple(lights))


def _backward(renderer, batch):
    """(function: upstream gradient [3P] numpy -> gradients as FP64 numpy arrays)."""
    import torch
    from paper_1906_11633_amd.renderer import shade_backward
    job = renderer.prepare(batch)
    out = renderer.render(job, vis=True)

    def run(c):
        g = shade_backward(renderer.ctx, job.layout, job.state, out["vis"], torch.from_numpy(c).cuda())
        torch.cuda.synchronize()
        return {k: v.cpu().numpy() for k, v in g.items()}
    return run


def _masked(batch, c, mask):
    """c where the per-pixel mask [P] is set, else 0 (planar rgb)."""
    po = batch.pixel_offset
    return c * np.concatenate([np.tile(mask[po[f]:po[f + 1]], 3) for f in range(batch.n_frames)]).astype(np.float32)


@pytest.mark.parametrize("n,res", [(8, 32), (9, 32), (13, 32), (9, 40)])
def test_each_object_alone_gives_the_same_bits(renderer, n, res):
    """64 objects in a tile (one round of slots), 81 (two), 169 (three), and 81 over a
    frame of partial tiles."""
    b = _grid(n, res)
    print(f"[grad tiles] grid {n}x{n} at {res}", flush=True)
    obj = oracle.render(b)["obj_id"]
    run = _backward(renderer, b)
    c = np.random.default_rng(1).uniform(-1, 1, 3 * b.total_pixels).astype(np.float32)
    whole = run(c)
    shown = np.unique(obj[obj >= 0])
    assert shown.size > 0.9 * n * n
    for o in shown[:: max(1, shown.size // 12)]:
        alone = run(_masked(b, c, obj == o))
        for k in OBJECT_KINDS:
            assert np.array_equal(alone[k][o], whole[k][o]), (k, o)
            assert not np.delete(alone[k], o, 0).any(), (k, o)


CASES = {
    "hand-31x33": lambda: _hand(31, 33),
    "hand-32x32": lambda: _hand(32, 32),
    "hand-65x40": lambda: _hand(65, 40),
    "whole-tiles-8-lights": lambda: _plane(64, 33, 8),
    "whole-one-row": lambda: _plane(45, 1, 1),
}


@pytest.mark.parametrize("name", list(CASES))
def test_tiles_add_up(renderer, name):
    b = CASES[name]()
    print(f"[grad tiles] {name} frames={b.n_frames}", flush=True)
    run = _backward(renderer, b)
    c = np.random.default_rng(2).uniform(-1, 1, 3 * b.total_pixels).astype(np.float32)
    whole = run(c)
    W, H = int(b.width[0]), int(b.height[0])
    jj, ii = np.divmod(np.arange(W * H), W)
    total = {k: np.zeros(v.shape) for k, v in whole.items()}
    bound = {k: np.abs(v.astype(np.float64)) for k, v in whole.items()}
    for ty in range((H + TILE - 1) // TILE):
        for tx in range((W + TILE - 1) // TILE):
            m = np.tile((ii // TILE == tx) & (jj // TILE == ty), b.n_frames)
            g = run(_masked(b, c, m))
            for k, v in g.items():
                total[k] += v
                bound[k] += np.abs(v.astype(np.float64))
    for k in whole:
        assert np.abs(whole[k]).max() > 0, k
        assert (np.abs(total[k] - whole[k]) <= 2.0 ** -23 * bound[k]).all(), k


def test_empty_frames(renderer):
    """Everything behind the camera: no tile holds a fragment."""
    b = S.config2(2, 1, 40)
    view = b.view.copy()
    view[:, 2, 3] += 50.0
    b = b.replace(view=view)
    g = _backward(renderer, b)(np.ones(3 * b.total_pixels, np.float32))
    for k, v in g.items():
        assert not v.any(), k
