"""The raster backward's matrix-product batches: entry counts around a batch
of 8 (and around a 64-entry chunk) composited in one block, wide splats whose
mean lies far outside the block, and upstream gradients that are not finite
at one pixel, which may reach only the entries composited there."""
import numpy as np
import pytest
import torch

import oracle
import scenes
from test_gpu_backward import GRAD_TOL, cam_for, grad_err, gpu_raster_backward, upstream

pytestmark = pytest.mark.gpu


def stack(n, W, H, seed, reach):
    """n faint splats over a W x H image, means up to `reach` px outside it."""
    rng = np.random.default_rng(seed)
    sp = np.zeros((n, 16), np.float32)
    sp[:, 0] = rng.uniform(-reach, W + reach, n)
    sp[:, 1] = rng.uniform(-reach, H + reach, n)
    s = rng.uniform(1.0, 2.0, n) * (reach + 6.0)
    sp[:, 4], sp[:, 5], sp[:, 6] = 1.0 / s ** 2, 0.3 / s ** 2, 1.5 / s ** 2
    sp[:, 7] = rng.uniform(0.02, 0.06, n)
    sp[:, 8:11] = rng.uniform(0.0, 1.0, (n, 3))
    rect = np.tile([0, 0, (W + 15) // 16, (H + 15) // 16], (n, 1))
    return sp, scenes.make_info(rng.uniform(1.0, 9.0, n).astype(np.float32), rect)


@pytest.mark.parametrize("n,reach", [(1, 0.0), (7, 2.0), (8, 2.0), (9, 30.0), (63, 4.0), (64, 300.0), (73, 4.0)])
def test_batches_match_oracle(n, reach):
    W, H = 11, 9  # one whole and three ragged blocks
    splats, info = stack(n, W, H, n, reach)
    proj = oracle.splats_to_proj(splats, info)
    mask = oracle.render(proj, W, H)["flags"] == 0
    d_img, d_alpha = upstream(W, H, mask, n)
    ref = oracle.composite_adjoint(proj, W, H, d_img=d_img, d_alpha=d_alpha)
    g = gpu_raster_backward(splats, info, cam_for(W, H), "binned", d_img, d_alpha, (0.0, 0.0, 0.0))
    e = [grad_err(g[:, k], ref["d_proj"][:, k]) for k in range(9)]
    assert max(e) <= GRAD_TOL, e


@pytest.mark.parametrize("value", [np.nan, np.inf])
def test_non_finite_upstream_stays_at_its_pixel(value):
    W, H = 8, 8
    splats, info = stack(12, W, H, 5, 0.0)
    splats[:6, 0], splats[:6, 1] = 1.0, 1.0  # the first six reach the left columns only
    splats[:6, 4], splats[:6, 5], splats[:6, 6] = 2.0, 0.0, 2.0
    splats[:, 7] = 0.3
    d_img, _ = upstream(W, H, np.ones((H, W)), 1)
    bad = d_img.copy()
    bad[6, 6, 1] = value  # seen by the last six
    clean = gpu_raster_backward(splats, info, cam_for(W, H), "binned", d_img, None, (0.0, 0.0, 0.0))
    g = gpu_raster_backward(splats, info, cam_for(W, H), "binned", bad, None, (0.0, 0.0, 0.0))
    assert np.isfinite(g[:6]).all()
    assert grad_err(g[:6, :9], clean[:6, :9]) <= GRAD_TOL
    assert not np.isfinite(g[6:, 7]).any()          # the green gradient
    assert np.isfinite(g[6:, [6, 8]]).all()         # red and blue are not touched
    assert not np.isfinite(g[6:, 5]).any()          # opacity, through dL/dalpha
