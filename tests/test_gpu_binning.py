"""Tile lists of the cell binning at the edges of its splits: every list is in
compositing order within its surfels' rects, and every surfel is in as many
lists as its band has tiles (counted per surfel by the preprocess, one band
row at a time, without cells)."""
import numpy as np
import pytest
import torch

from paper_2609_30741_amd import api, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,W,H,log_scale", [
    (1, 1, 1, (-1.0, 0.1)),             # one tile of one cell
    (65, 128, 128, (-2.0, 0.5)),        # one whole cell, two chunks of the order
    (3000, 129, 1030, (-3.0, 0.5)),     # one tile past a cell's edge both ways
    (40_000, 333, 257, (-3.5, 0.5)),    # past the small chunks at the front of the order
    (900, 1600, 1064, (0.0, 0.3)),      # more entries in a chunk than the emission keeps
    (130, 4300, 4200, (-1.5, 0.7)),     # over 1024 cells and over 20480 tiles
])
def test_tile_lists_by_cell(n, W, H, log_scale):
    sc = synth.scene_uniform_cube(11, n, log_scale=log_scale)
    cam = synth.look_at((0.0, -4.0, 0.0), (0, 0, 0), (0, 0, 1), W, H, 1.1 * max(W, 2))
    ctx = api.Context(sync=True)
    ds = api.DeviceScene(sc)
    zkey, rects, counts = (t.cpu().numpy() for t in ctx.preprocess_debug(ds, cam))
    zkey, counts = zkey.view(np.uint32), counts.astype(np.int64)
    ranges, vals, nk = ctx.tile_lists_debug(ds, cam, capacity=int(counts.sum()) + 1)
    ranges, vals = ranges.cpu().numpy().astype(np.int64), vals.cpu().numpy()
    torch.cuda.synchronize()
    assert nk == counts.sum() == vals.size
    assert np.array_equal(ranges[1:, 0], ranges[:-1, 1]) and ranges[0, 0] == 0 and ranges[-1, 1] == nk
    assert np.array_equal(np.bincount(vals, minlength=n), counts)
    tile = np.repeat(np.arange(ranges.shape[0]), ranges[:, 1] - ranges[:, 0])
    tx, ty = tile % ((W + 15) // 16), tile // ((W + 15) // 16)
    r = rects[vals]
    assert np.all((r[:, 0] <= tx) & (tx <= r[:, 2]) & (r[:, 1] <= ty) & (ty <= r[:, 3]))
    order = zkey[vals].astype(np.uint64) << np.uint64(32) | vals.astype(np.uint64)
    same = tile[1:] == tile[:-1]
    assert np.all(order[1:][same] > order[:-1][same])
