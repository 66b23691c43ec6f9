"""The workspace of tgs_bin (sizes only, no GPU): the repair lists hold every
run that the parts of split groups can queue, and a workspace sized for n
Gaussians and a capacity holds every smaller n and capacity."""
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


@pytest.mark.parametrize("width, height, params", [
    (4096, 4096, dict(num_bins=64, tile_size=16)),               # 8192 groups
    (1920, 1080, dict()),
    (640, 360, dict(num_bins=16, repair="rules")),
    (1920, 1080, dict(num_bins=128, tile_size=32, sub_bins=2)),
])
def test_workspace_does_not_shrink(width, height, params):
    edges = [0, 1, 255, 256, 257, 65024, 65025, 65536, 65537, 130048, 130049, 131072, 260096, 260097, 262144, 262145,
             524288, 524289, 3_000_000]
    ns = sorted(set(edges) | {int(1.07 ** k) for k in range(220)})
    sizes = [workspace(n, 100_000, width, height, **params) for n in ns]
    assert all(a <= b for a, b in zip(sizes, sizes[1:]))
    caps = [workspace(50_000, c, width, height, **params) for c in sorted({int(1.11 ** k) for k in range(200)})]
    assert all(a <= b for a, b in zip(caps, caps[1:]))
