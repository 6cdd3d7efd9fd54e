"""The camera on frames a pixel or a few wide or high: a wave's tile takes
another shape than 16 x 4 where that leaves fewer lanes idle (1 x 64 to 64 x 1).
Images and gradients against the FP64 oracle, as on the tiles' edges (1e-4 and
1e-3, on pixels whose hit object is the same when every body moves by 1e-4)."""
from __future__ import annotations

import pytest

from test_gpu_camera_tiles import test_tiles_match_the_oracle as check_frame

pytestmark = pytest.mark.gpu


# 1 x 64, 2 x 32, 4 x 16, 8 x 8, 32 x 2 and 64 x 1 tiles, whole and with remainders
@pytest.mark.parametrize("width,height", [(1, 64), (1, 333), (2, 65), (3, 250), (4, 16), (7, 129), (8, 24), (250, 1),
                                          (64, 1), (65, 2), (193, 2), (31, 2)])
def test_narrow_frames_match_the_oracle(width, height):
    check_frame(width, height, 3.0 / max(width, height), (0.3, -3.5, 1.6), (0.0, 0.0, 0.3), (32, 16))
