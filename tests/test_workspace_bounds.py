"""The workspace of tgs_bin (sizes only, no GPU): the repair lists hold every
run that the parts of split groups can queue."""
import ctypes

import numpy as np
import pytest

import scenes

tg = pytest.importorskip("paper_2609_03613_amd")
from paper_2609_03613_amd import _lib as L  # noqa: E402
from paper_2609_03613_amd.api import camera_struct  # noqa: E402


def workspace(n, capacity, width, height, **params):
    cam = camera_struct(scenes.camera(np.eye(3), np.zeros(3), 100.0, 100.0, width / 2, height / 2, width, height))
    p = tg.Params(**params).c()
    return tg.lib().tgs_bin_workspace_size(n, capacity, ctypes.byref(cam), ctypes.byref(p), L.ORDER_BINNED)


@pytest.mark.parametrize("width", [16, 128])
@pytest.mark.parametrize("bins, sub", [(1, 2), (1, 8), (4, 2), (4, 8)])
def test_repair_lists_grow_with_the_buckets_of_long_parts(width, bins, sub):
    # every entry takes a pair, a code and a tile (12 bytes); a run of 513 equal
    # depths is queued by itself, in any of the eight lists' worth of {begin,
    # length}, whatever the number of tiles, bins and sub-bins
    c0, c1 = 1 << 20, 3 << 20
    grown = workspace(1000, c1, width, 16, num_bins=bins, sub_bins=sub) - workspace(
        1000, c0, width, 16, num_bins=bins, sub_bins=sub)
    assert grown >= (c1 - c0) * 12 + 8 * 8 * ((c1 - c0) // 513) - 4096
