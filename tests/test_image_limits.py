"""Image calls at the largest sizes that their cameras can state (CPU only: host arithmetic)."""
import os

import numpy as np
import pytest

from paper_2501_14534_amd import gs, scenes

INT_MAX = 2 ** 31 - 1


@pytest.fixture(scope="module")
def lib():
    if not os.path.exists(gs.LIB):
        pytest.skip("libgs.so not built")
    return gs.load()


def _align(x):
    return (x + 255) // 256 * 256


@pytest.mark.parametrize("w,h", [(INT_MAX, 1), (INT_MAX - 99, 1), (INT_MAX - 114, 2), (1, INT_MAX), (116, INT_MAX - 14),
                                 (117, 33)])
def test_loss_workspace_counts_every_tile(lib, w, h):
    """Nine words a pixel, two a tile of 116 x 16 and plane, a double a view."""
    cam = scenes.Camera(np.eye(3, dtype=np.float32), np.zeros(3, np.float32), 1.0, 1.0, 0.0, 0.0, w, h)
    tiles = 3 * -(-w // 116) * -(-h // 16)
    assert gs.loss_workspace_size(gs.cameras([cam]), 1) == _align(36 * w * h) + _align(8 * tiles) + _align(
        8 * gs.MAX_VIEWS)
