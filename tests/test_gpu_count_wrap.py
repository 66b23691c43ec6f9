"""Entry counts of 2^32 and more (which no 32-bit position can hold), without a
host count: flagged with the exact count, and the stream is empty, so that
whatever follows stays in range, where groups would be split, with tagged pairs
and without either."""
import numpy as np
import pytest
import torch

import scenes

pytestmark = pytest.mark.gpu

tg = pytest.importorskip("paper_2609_03613_amd")

SIDE = 256  # tiles a side


@pytest.mark.parametrize("capacity", [100_000, 1 << 20, (6 << 20) + 1])
def test_wrapped_entry_count(capacity):
    n = SIDE * SIDE + 1  # each covers every tile: 2^32 + 2^16 entries
    M = n * SIDE * SIDE
    assert M == (1 << 32) + (1 << 16)
    rect = np.tile(np.array([[0, 0, SIDE, SIDE]], np.int64), (n, 1))
    depth = np.random.default_rng(1).uniform(2.0, 20.0, n).astype(np.float32)
    dev = torch.device("cuda:0")
    px = 8 * SIDE
    cam = scenes.camera(np.eye(3), np.zeros(3), 100.0, 100.0, px / 2, px / 2, px, px)
    r = tg.Renderer(cam, tg.Params(tile_size=8, num_bins=1), device=dev)
    s = torch.zeros((n, 16), dtype=torch.float32, device=dev)
    i = torch.as_tensor(scenes.make_info(depth, rect).view(np.int32)).to(dev)
    b = r.bin(s, i, "binned", capacity=capacity, sync=False)
    out = r.rasterize(s, i, b)
    torch.cuda.synchronize()
    assert b.counters.tolist() == [M, n, 1, 0]
    assert not b.offsets.any()
    assert not b.repaired.any()
    order = b.dispatch_order().cpu().numpy()
    assert np.array_equal(np.sort(order), np.arange(SIDE * SIDE))
    assert torch.isnan(out["rgb"]).all()
