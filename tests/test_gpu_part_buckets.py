"""Buckets of the parts of split groups around the lengths where they are ordered
differently: by rank up to 64 pairs, by a wavefront of the same workgroup up to
512, queued above, and by rank again once a workgroup holds as many as it keeps.
Bit-exact against the oracle's schedule."""
import numpy as np
import pytest
import torch

import oracle
import scenes

pytestmark = pytest.mark.gpu

tg = pytest.importorskip("paper_2609_03613_amd")


def check(depth, tile, tx, K, sub, capacity=None):
    n = len(depth)
    rect = np.stack([tile, np.zeros(n, np.int64), tile + 1, np.ones(n, np.int64)], 1)
    ref = oracle.schedule(depth, rect, tx, 1, K=K, znear=0.01, zfar=1e10)
    dev = torch.device("cuda:0")
    cam = scenes.camera(np.eye(3), np.zeros(3), 100.0, 100.0, 8.0 * tx, 8.0, 16 * tx, 16)
    r = tg.Renderer(cam, tg.Params(num_bins=K, sub_bins=sub), device=dev)
    info = torch.as_tensor(scenes.make_info(depth, rect).view(np.int32)).to(dev)
    b = r.bin(torch.zeros((n, 16), dtype=torch.float32, device=dev), info, "binned", capacity=capacity)
    torch.cuda.synchronize()
    assert np.array_equal(b.offsets.cpu().numpy().view(np.uint32), ref["bin_offsets"])
    assert np.array_equal(b.pairs.cpu().numpy()[:n].view(np.uint64), ref["stream"])


# the second capacity: from there on the entries carry their tile instead of a code
@pytest.mark.parametrize("capacity", [None, (6 << 20) + 1])
@pytest.mark.parametrize("spread", [0.0, 1e-6])
@pytest.mark.parametrize("size", [63, 64, 65, 128, 129, 256, 257, 511, 512, 513])
def test_clusters_of_a_size(size, spread, capacity):
    rng = np.random.default_rng(size)
    tx, layers = 4, 60000 // (4 * size)
    z = np.geomspace(2.0, 20.0, layers)
    depth = np.tile(np.repeat(z, size), tx) * (1.0 + spread * rng.random(tx * layers * size))
    tile = np.repeat(np.arange(tx), layers * size)
    depth = np.concatenate([depth, rng.uniform(2.0, 20.0, 5000)]).astype(np.float32)
    tile = np.concatenate([tile, rng.integers(0, tx, 5000)])
    p = rng.permutation(len(depth))
    for K, sub in ((16, 2), (64, 8)):
        check(depth[p], tile[p], tx, K, sub, capacity)


def test_more_clusters_than_a_workgroup_keeps():
    # some ten parts per workgroup with 47 clusters of 65 each
    tx, size = 64, 65
    layers = 17_000_000 // (tx * size)
    z = np.geomspace(2.0, 20.0, layers).astype(np.float32)
    depth = np.tile(np.repeat(z, size), tx)
    tile = np.repeat(np.arange(tx), layers * size)
    p = np.random.default_rng(5).permutation(len(depth))
    check(depth[p], tile[p], tx, 64, 8, capacity=len(depth))
