"""Overflowing frames of surfels smaller than a tile, whose entries (one per
surfel and cell) outnumber the keys that the workspace holds, and overflowing
ROI patches: the first keys in compositing order are kept wherever in the
image they lie, bit for bit the image of the surfels in front."""
import numpy as np
import pytest
import torch

import test_gpu_overflow_frames as frames
from paper_2609_30741_amd import api, synth

pytestmark = pytest.mark.gpu


# Both forms of the emission, and images of one and of several windows.
@pytest.mark.parametrize("n,W,H,log_scale,share", [(2000, 150, 140, (-6.0, 0.3), 0.3),
                                                   (20_000, 1283, 717, (-6.5, 0.3), 0.4),
                                                   (20_000, 1283, 717, (-6.5, 0.3), 0.02),
                                                   (20_000, 4300, 4200, (-7.5, 0.3), 0.3)])
def test_first_small_keys_are_kept(n, W, H, log_scale, share):
    frames.test_first_keys_are_kept(n, W, H, log_scale, share)


@pytest.mark.parametrize("n,W,H,log_scale,share", [(3000, 150, 140, (-5.5, 0.5), 0.4),
                                                   (20_000, 1283, 717, (-6.5, 0.3), 0.4),
                                                   (6000, 1283, 717, (-2.5, 0.6), 0.6)])
def test_first_roi_keys_are_kept(n, W, H, log_scale, share):
    sc = synth.scene_uniform_cube(3, n, log_scale=log_scale)
    cam = synth.look_at((0.0, -4.0, 0.0), (0, 0, 0), (0, 0, 1), W, H, 1.1 * W)
    tx, ty = (W + 15) // 16, (H + 15) // 16
    mask = np.random.default_rng(1).random((ty, tx)) < 0.4
    ctx, small = api.Context(sync=True), api.Context(sync=False)
    for c in (ctx, small):
        c.set_blend_split(0, 0)  # a segment's sums round as its list is cut
    ds = api.DeviceScene(sc)
    zkey, _, counts = (t.cpu().numpy() for t in ctx.preprocess_debug(ds, cam))
    order = np.lexsort((np.arange(n), zkey.view(np.uint32)))
    ranges, vals, _ = ctx.tile_lists_debug(ds, cam, capacity=int(counts.sum()) + 1)
    ranges, vals = ranges.cpu().numpy().astype(np.int64), vals.cpu().numpy()
    tile = np.repeat(np.arange(tx * ty), ranges[:, 1] - ranges[:, 0])
    on = mask.reshape(-1)[tile]
    counts = np.bincount(vals[on], minlength=n)
    ends = np.cumsum(counts[order])

    nbytes = small._ws_bytes(n, W, H, int(ends[-1] * share))
    lo, hi = int(ends[-1] * share), int(ends[-1] * share) + 4096  # the keys that this workspace holds
    while lo < hi:
        mid = (lo + hi + 1) // 2
        lo, hi = (mid, hi) if small._ws_bytes(n, W, H, mid) <= nbytes else (lo, mid - 1)
    assert lo < ends[-1]
    small.ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
    tmask = torch.from_numpy(mask.astype(np.uint8)).cuda()

    def patched(c, scene):
        o = dict(rgb=torch.full((3, H, W), 0.25, device="cuda"), z=torch.full((H, W), 7.0, device="cuda"),
                 alpha=torch.full((H, W), 0.5, device="cuda"),
                 cls=torch.zeros((H, W), dtype=torch.uint8, device="cuda"))
        c.patch_rois(api.DeviceScene(scene), cam, tmask, o["rgb"], o["z"], o["alpha"], o["cls"])
        return {k: v.cpu().numpy() for k, v in o.items()}

    got = patched(small, sc)
    stats = small.poll_status()
    assert stats["overflow"] & 1 and stats["n_keys_roi"] == ends[-1]
    cut = int(np.searchsorted(ends, lo, side="right"))
    images = [patched(ctx, sc.subset(np.sort(order[:m]))) for m in (cut, cut + 1)]
    part = lo - (int(ends[cut - 1]) if cut else 0)  # keys of the surfel that is cut
    tiles = np.unique(tile[on & (vals == order[cut])])
    assert tiles.size == counts[order[cut]]
    with_cut = np.zeros((H, W), bool)
    for t in tiles[:part]:
        with_cut[t // tx * 16:t // tx * 16 + 16, t % tx * 16:t % tx * 16 + 16] = True
    for k in ("rgb", "z", "alpha", "cls"):
        assert np.array_equal(got[k], np.where(with_cut, images[1][k], images[0][k])), k
