"""The batched raster's item dispatch at its edges: item counts below one
workgroup, not multiples of the four items of a workgroup or of the 128 items
of a round over the XCDs, and exactly a round. Every view bitwise equal to the
unsplit per-view raster (the same block walk on the same stream)."""
import numpy as np
import pytest
import torch

import scenes

pytestmark = pytest.mark.gpu

tg = pytest.importorskip("paper_2609_03613_amd")


@pytest.mark.parametrize("sizes,tile", [
    ([(7, 5)], 8),                          # one item
    ([(24, 8), (8, 16)], 8),                # 3 + 2 items
    ([(64, 128)], 8),                       # 128 items, one round
    ([(64, 136)], 16),                      # 34 tiles of 4 blocks, the last row half outside
    ([(100, 70), (33, 90), (512, 40)], 32),  # ragged 32-pixel tiles over several rounds
])
def test_batch_items_cover_every_block(sizes, tile):
    dev = torch.device("cuda:0")
    gnp, _ = scenes.small_forward(seed=3, n=3000)
    g = tg.to_device(gnp, dev)
    cams = [scenes.camera(np.eye(3), np.zeros(3), max(w, h), max(w, h), w / 2.0, h / 2.0, w, h) for w, h in sizes]
    params = [tg.Params(tile_size=tile, num_bins=16, split_entries=0) for _ in cams]
    br = tg.BatchRenderer(cams, params, device=dev, bg=(0.3, 0.2, 0.1))
    for o in br.outs:
        o["rgb"].fill_(-5.0)
        o["alpha"].fill_(-5.0)
        o["last"].fill_(-5)
    br.frame(g, sync=True)
    torch.cuda.synchronize()
    for c, p, o in zip(cams, params, br.outs):
        r = tg.Renderer(c, p, device=dev)
        ref = r.render(g, bg=(0.3, 0.2, 0.1))
        for k in ("rgb", "alpha", "last"):
            assert torch.equal(o[k], ref[k]), (c["width"], c["height"], k)
