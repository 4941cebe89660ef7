"""A frame with more tile keys than its workspace holds keeps the first keys
in compositing order, and of the surfel that the capacity cuts its first
tiles: tile by tile the same image, bit for bit, as the scene with only the
surfels in front, with or without the one that is cut."""
import numpy as np
import pytest
import torch

from paper_2609_30741_amd import api, synth

pytestmark = pytest.mark.gpu


# Sizes on both sides of the line up to which the emission scans its own
# counts, and surfels that span many cells.
@pytest.mark.parametrize("n,W,H,log_scale,share", [(400, 150, 140, (-1.5, 0.4), 0.3), (400, 150, 140, (-1.5, 0.4), 0.8),
                                                   (6000, 1283, 717, (-1.2, 0.6), 0.5), (300, 700, 500, (0.0, 0.3), 0.6)])
def test_first_keys_are_kept(n, W, H, log_scale, share):
    sc = synth.scene_uniform_cube(3, n, log_scale=log_scale)
    cam = synth.look_at((0.0, -4.0, 0.0), (0, 0, 0), (0, 0, 1), W, H, 1.1 * W)
    ctx = api.Context(sync=True)
    zkey, rects, counts = (t.cpu().numpy() for t in ctx.preprocess_debug(api.DeviceScene(sc), cam))
    order = np.lexsort((np.arange(n), zkey.view(np.uint32)))
    ends = np.cumsum(counts[order].astype(np.int64))

    small = api.Context(sync=False)
    nbytes = small._ws_bytes(n, W, H, int(ends[-1] * share))
    lo, hi = int(ends[-1] * share), int(ends[-1] * share) + 4096  # the keys that this workspace holds
    while lo < hi:
        mid = (lo + hi + 1) // 2
        lo, hi = (mid, hi) if small._ws_bytes(n, W, H, mid) <= nbytes else (lo, mid - 1)
    assert lo < ends[-1]
    small.ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
    got = small.render_dominant(api.DeviceScene(sc), cam)
    torch.cuda.synchronize()

    cut = int(np.searchsorted(ends, lo, side="right"))  # whole surfels
    images = []
    for m in (cut, cut + 1):
        front = np.sort(order[:m])  # index order decides between equal depths
        images.append(ctx.render_dominant(api.DeviceScene(sc.subset(front)), cam))
    part = lo - (int(ends[cut - 1]) if cut else 0)  # keys of the surfel that is cut
    # Its tiles are those where it is listed, row by row.
    ds = api.DeviceScene(sc)
    ranges, vals, _ = ctx.tile_lists_debug(ds, cam, capacity=int(ends[-1]) + 1)
    ranges, vals = ranges.cpu().numpy().astype(np.int64), vals.cpu().numpy()
    tx = (W + 15) // 16
    tiles = [t for t in range(ranges.shape[0]) if (vals[ranges[t, 0]:ranges[t, 1]] == order[cut]).any()]
    assert len(tiles) == counts[order[cut]]
    with_cut = np.zeros((H, W), bool)
    for t in tiles[:part]:
        with_cut[t // tx * 16:t // tx * 16 + 16, t % tx * 16:t % tx * 16 + 16] = True
    for k in ("rgb", "depth_raw", "alpha"):
        want = np.where(with_cut, images[1][k].cpu().numpy(), images[0][k].cpu().numpy())
        assert np.array_equal(got[k].cpu().numpy(), want), k
