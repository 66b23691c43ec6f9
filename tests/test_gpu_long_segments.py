"""Segments of 513..8192 pairs around the lengths and clusters where their sort
changes: buckets ordered by rank (up to 64 pairs) or, past 2048 pairs, by a
wavefront (up to 512), else the network, with and without records, queued as
segments and as sub-segments, fewer and more of them than workgroups.
Bit-exact against the oracle's schedule."""
import numpy as np
import pytest
import torch

import oracle
import scenes

pytestmark = pytest.mark.gpu

tg = pytest.importorskip("paper_2609_03613_amd")

LENGTHS = (513, 1024, 1025, 2047, 2048, 2049, 4095, 4096, 4097, 6000, 8191, 8192, 8193)
CLUSTERS = {
    "none": (),
    "ranks": (63, 64),
    "wavefronts": (65, 128, 129),
    "longest wavefront": (256, 257),
    "a full bucket": (512,),
    "more than a bucket": (513,),
    "all equal": None,
}


def segments(lengths, clusters, spread, seed):
    """One tile per length; the tile's depths uniform over its own range but for
    the clusters, each within `spread` of one depth."""
    rng = np.random.default_rng(seed)
    depth, tile = [], []
    for t, n in enumerate(lengths):
        lo = 2.0 + t % 20
        z = rng.uniform(lo, lo + 0.5, n)
        if clusters is None:
            z[:] = lo
        at = 0
        for k, size in enumerate(clusters or ()):
            z[at:at + size] = lo + 0.1 * (k + 1) + spread * rng.random(size)
            at += size
        depth.append(z.astype(np.float32))
        tile.append(np.full(n, t))
    depth, tile = np.concatenate(depth), np.concatenate(tile)
    p = rng.permutation(len(depth))
    return depth[p], tile[p]


@pytest.mark.parametrize("packed, sub", [(0, 1), (1, 1), (0, 2)])
@pytest.mark.parametrize("spread", [0.0, 2e-6])
@pytest.mark.parametrize("clusters", list(CLUSTERS))
def test_long_segments(clusters, spread, packed, sub):
    check(LENGTHS, CLUSTERS[clusters], spread, packed, sub)


@pytest.mark.parametrize("packed", [0, 1])
@pytest.mark.parametrize("count", [256, 257, 600])
@pytest.mark.parametrize("clusters", ["none", "ranks", "wavefronts", "a full bucket", "all equal"])
def test_many_long_segments(clusters, count, packed):
    # more of them than the launch has workgroups
    lengths = [(513, 600, 1024, 1025, 1500, 2048)[k % 6] for k in range(count)]
    check(lengths, CLUSTERS[clusters], 0.0, packed, 1)


def check(lengths, clusters, spread, packed, sub):
    depth, tile = segments(lengths, clusters, spread, len(clusters or ()))
    n, tx = len(depth), len(lengths)
    rect = np.stack([tile, np.zeros(n, np.int64), tile + 1, np.ones(n, np.int64)], 1)
    ref = oracle.schedule(depth, rect, tx, 1, K=1, znear=0.01, zfar=1e10)
    dev = torch.device("cuda:0")
    cam = scenes.camera(np.eye(3), np.zeros(3), 100.0, 100.0, 8.0 * tx, 8.0, 16 * tx, 16)
    r = tg.Renderer(cam, tg.Params(num_bins=1, sub_bins=sub, packed=packed), device=dev)
    info = torch.as_tensor(scenes.make_info(depth, rect).view(np.int32)).to(dev)
    splats = torch.zeros((n, 16), dtype=torch.float32, device=dev)
    b = r.bin(splats, info, "binned")
    torch.cuda.synchronize()
    assert np.array_equal(b.offsets.cpu().numpy().view(np.uint32), ref["bin_offsets"])
    assert np.array_equal(b.pairs.cpu().numpy()[:n].view(np.uint64), ref["stream"])
    if packed:
        ids = (ref["stream"] & np.uint64(0xFFFFFFFF)).astype(np.int64)
        rec = b.records.cpu().numpy()[:n]
        assert np.array_equal(rec[:, 9].copy().view(np.int32), ids)
