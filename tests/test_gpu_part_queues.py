"""Parts of split groups that queue several runs of one sub-segment: many layers
of more than 512 equal depths in few tiles and bins, so that the queued runs
outnumber the sub-segments, beside single codes of more than 4096 and 8192
entries. Streams, bin offsets and the repaired-entry count bit-exact against the
oracle's schedule."""
import numpy as np
import pytest
import torch

import oracle
import scenes

pytestmark = pytest.mark.gpu

tg = pytest.importorskip("paper_2609_03613_amd")


def layered(tiles, layers, size, big, seed=0):
    """In each tile `layers` depths of `size` entries; `big` more entries at the
    middle one in tile 0."""
    rng = np.random.default_rng(seed)
    z = np.geomspace(2.0, 20.0, layers).astype(np.float32)
    depth = np.concatenate([np.tile(np.repeat(z, size), tiles), np.full(big, z[layers // 2], np.float32)])
    tile = np.concatenate([np.repeat(np.arange(tiles), layers * size), np.zeros(big, np.int64)])
    p = rng.permutation(len(depth))
    return depth[p], tile[p]


CASES = [
    # tiles of the image, tiles used, layers, entries of a layer, extra entries, bins, sub-bins
    (1, 1, 56, 513, 0, 1, 8),       # 10 runs, 8 sub-segments
    (1, 1, 40, 520, 0, 4, 2),       # 40 runs, 8 sub-segments
    (1, 1, 224, 550, 0, 4, 8),      # 85 runs, 32 sub-segments
    (8, 8, 14, 700, 9000, 1, 2),    # 48 runs, 16 sub-segments
    (8, 2, 56, 600, 5000, 1, 8),    # codes past 4096 and 8192 entries beside the runs
    (8, 3, 224, 550, 0, 4, 8),      # 255 runs
    (1, 1, 420, 513, 5000, 16, 2),  # codes past 4096 only
    (1, 1, 40, 512, 0, 4, 2),       # layers that are not queued
]


# the second capacity: from there on the entries carry their tile instead of a code
@pytest.mark.parametrize("capacity", [None, (6 << 20) + 1])
@pytest.mark.parametrize("case", range(len(CASES)))
def test_layers_of_equal_depths(case, capacity):
    tx, used, layers, size, big, K, sub = CASES[case]
    depth, tile = layered(used, layers, size, big, case)
    n = len(depth)
    rect = np.stack([tile, np.zeros(n, np.int64), tile + 1, np.ones(n, np.int64)], 1)
    ref = oracle.schedule(depth, rect, tx, 1, K=K, znear=0.01, zfar=1e10)
    dev = torch.device("cuda:0")
    cam = scenes.camera(np.eye(3), np.zeros(3), 100.0, 100.0, 8.0 * tx, 8.0, 16 * tx, 16)
    r = tg.Renderer(cam, tg.Params(num_bins=K, sub_bins=sub), device=dev)
    info = torch.as_tensor(scenes.make_info(depth, rect).view(np.int32)).to(dev)
    b = r.bin(torch.zeros((n, 16), dtype=torch.float32, device=dev), info, "binned", capacity=capacity)
    torch.cuda.synchronize()
    off = b.offsets.cpu().numpy().view(np.uint32)
    assert np.array_equal(off, ref["bin_offsets"])
    assert np.array_equal(b.pairs.cpu().numpy()[:n].view(np.uint64), ref["stream"])
    seg = np.diff(off.astype(np.int64))
    assert b.counters.tolist() == [n, n, 0, int(seg[seg >= 2].sum())]
