"""Texel wrapping on the GPU: the fp32 quotient of ordinary tilings, its limits (2^20 repeats,
2^30 texels) and the 64-bit remainder beyond them, on both signs, sizes that divide nothing
and one texel, against the oracle at the parity bar."""
import numpy as np
import pytest

import oracle
from tests import parity
from tests.test_materials_gpu import _render, renderer  # noqa: F401
from tests.test_oracle_materials import _plane

pytestmark = pytest.mark.gpu

# repeats (exact in fp32); FP64 texel coordinates keep 2^-20 of a texel at 2^26 repeats
OFFSETS = [-1.0, 1000.0, -1000.0, 2.0 ** 20 - 2, 2.0 ** 20, -(2.0 ** 20), 2.0 ** 24, -(2.0 ** 24), 2.0 ** 26]


@pytest.mark.parametrize("offset", OFFSETS)
@pytest.mark.parametrize("h,w", [(1, 1), (7, 3), (32, 48)])
def test_wrapped_texels(renderer, offset, h, w):  # noqa: F811
    tex = np.random.default_rng(h * w).uniform(0, 1, (h, w, 3))
    b = _plane(tex, (2.5, 1.5, offset, -offset), emission=0.3)
    gpu, _ = _render(renderer, b)
    st = parity.compare(b, gpu, oracle.render(b))
    assert st["covered"] == 64 * 64
