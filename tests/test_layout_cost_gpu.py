"""Building the patches of a layout costs the host no more than the tile lists of the tiled path
did for the same frames (a factor of three allowed; they are about level)."""
import time

import pytest

from paper_1906_11633_amd import scenes as S
from tests.test_patches_gpu import TILED, _resized

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("size", [(2048, 2048), (1024, 768)])
def test_large_frames(size):
    from paper_1906_11633_amd.renderer import Context, Layout
    lay = Layout(Context(0), _resized(S.config2(2, 100, 200), [size]))
    best = {}
    for name, tuning in (("tiled", (32, 32, 256, 0, 1)), ("patches", (32, 32, 256, 0, 0))):
        times = []
        for _ in range(9):
            lay.set_tuning(*((32, 32, 256, 0, 0) if name == "tiled" else TILED))
            t = time.perf_counter()
            lay.set_tuning(*tuning)
            times.append(time.perf_counter() - t)
        best[name] = min(times)
    print(size, {k: f"{1e3 * v:.3f} ms" for k, v in best.items()}, flush=True)
    assert best["patches"] <= 3 * best["tiled"]
