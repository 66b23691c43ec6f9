"""Both sides of the rules on the capacity by which groups are split and pairs
carry their tile: the same stream, bit-exact against the oracle's schedule, with
groups past the group sort's stage and past the split length."""
import numpy as np
import pytest
import torch

import oracle
import scenes

pytestmark = pytest.mark.gpu

tg = pytest.importorskip("paper_2609_03613_amd")

SIDE = 128  # tiles a side of the larger image: 2048 groups of 8 tiles


def check(depth, tile, side, rows, capacity, **params):
    n = len(depth)
    x, y = tile % side, tile // side
    rect = np.stack([x, y, x + 1, y + 1], 1)
    K = params.get("num_bins", 64)
    ref = oracle.schedule(depth, rect, side, rows, K=K, znear=0.01, zfar=1e10)
    dev = torch.device("cuda:0")
    cam = scenes.camera(np.eye(3), np.zeros(3), 100.0, 100.0, 8.0 * side, 8.0 * rows, 16 * side, 16 * rows)
    r = tg.Renderer(cam, tg.Params(**params), device=dev)
    info = torch.as_tensor(scenes.make_info(depth, rect).view(np.int32)).to(dev)
    b = r.bin(torch.zeros((n, 16), dtype=torch.float32, device=dev), info, "binned", capacity=capacity)
    torch.cuda.synchronize()
    assert np.array_equal(b.offsets.cpu().numpy().view(np.uint32), ref["bin_offsets"])
    assert np.array_equal(b.pairs.cpu().numpy()[:n].view(np.uint64), ref["stream"])
    seg = np.diff(ref["bin_offsets"].astype(np.int64))
    assert b.counters.tolist() == [n, n, 0, int(seg[seg >= 2].sum())]


def scene(tiles, heavy, seed):
    """A few entries everywhere and `heavy` more in one tile."""
    rng = np.random.default_rng(seed)
    tile = np.concatenate([rng.integers(0, tiles, 40000), np.full(heavy, tiles // 2)])
    depth = rng.uniform(2.0, 20.0, len(tile)).astype(np.float32)
    p = rng.permutation(len(tile))
    return depth[p], tile[p]


@pytest.mark.parametrize("sub", [2, 8])
@pytest.mark.parametrize("heavy", [5000, 20000])
@pytest.mark.parametrize("capacity", [8 * 12288, 8 * 12288 + 1])
def test_capacity_per_group(capacity, heavy, sub):
    depth, tile = scene(64, heavy, 1)  # eight groups
    check(depth, tile, 64, 1, capacity, sub_bins=sub)


@pytest.mark.parametrize("heavy", [5000, 20000])
@pytest.mark.parametrize("capacity", [6 << 20, (6 << 20) + 1, 2048 * 4096, 2048 * 4096 + 1, 16 << 20, (16 << 20) + 1,
                                      2048 * 12288 + 1])
@pytest.mark.parametrize("params", [dict(), dict(sub_bins=1), dict(num_bins=24)])
def test_many_entries(params, capacity, heavy):
    depth, tile = scene(SIDE * SIDE, heavy, 2)
    check(depth, tile, SIDE, SIDE, capacity, **params)
