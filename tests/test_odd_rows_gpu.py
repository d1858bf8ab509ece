"""Whole frames (too large for one patch) whose rows start at any alignment: the frame kernel's four-pixel stores at
every width modulo 4, with every output, against the tiled path bit for bit."""
import pytest

from paper_1906_11633_amd import scenes as S
from tests.test_patches_gpu import _check, _resized, renderer  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("width,height", [(29, 250), (66, 131), (67, 131), (129, 61), (253, 31)])
def test_widths(renderer, width, height):  # noqa: F811
    b = _resized(S.config2(17, 256, 48, 1), [(width, height)])
    _check(renderer, S.with_postprocessing(b, seed=3), f"{width} x {height}")
