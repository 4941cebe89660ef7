"""Surfels without extent along one axis or both: their plane coordinates are
not numbers, so only the low-pass term draws them.  Among ordinary surfels
against the oracle (1e-4, as every render), and alone in closed form, at
image sizes of both forms of the blend."""
import numpy as np
import pytest
import torch

from paper_2609_30741_amd import api, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lowpass", [True, False])
@pytest.mark.parametrize("axis", [0, 1])
@pytest.mark.parametrize("W,H", [(111, 85), (700, 500)])
def test_flat_axis_among_others(oracle, W, H, axis, lowpass):
    sc = synth.scene_uniform_cube(3, 1500, log_scale=(-2.5, 0.7))
    sc.scale[axis, ::20] = 0.0
    cam = synth.look_at((0, -4, 0.3), (0, 0, 0), (0, 0, 1), W, H, 3.1 * H)
    got = api.Context(sync=True).render_dominant(api.DeviceScene(sc), cam, api.Raster(lowpass=lowpass))
    rng = np.random.default_rng(5)
    pix = np.stack([rng.integers(0, W, 4000), rng.integers(0, H, 4000)], axis=1).astype(np.int32)
    want = oracle.render(sc, cam, oracle.Raster(lowpass=lowpass), pixels=pix)
    ok = ~np.asarray(want["amb"]).astype(bool).reshape(-1)
    assert ok.mean() > 0.99
    at = (pix[ok, 1], pix[ok, 0])
    assert np.abs(got["rgb"].cpu().numpy()[:, at[0], at[1]] - want["rgb"][:, ok]).max() <= 1e-4
    assert np.abs(got["alpha"].cpu().numpy()[at] - want["alpha"][ok]).max() <= 1e-4


@pytest.mark.parametrize("W,H", [(111, 85), (700, 500)])
@pytest.mark.parametrize("scale", [(0.0, 0.0), (0.0, 0.3), (np.nan, np.nan), (1e-37, 1e-37)])
def test_single_dot(W, H, scale):
    sc = synth.scene_uniform_cube(4, 1)
    sc.pos[:, 0] = 0.0
    sc.scale[:, 0] = scale
    sc.opacity[0] = 0.8
    cam = synth.look_at((0, -4, 0.0), (0, 0, 0), (0, 0, 1), W, H, 1.1 * W)
    x, y = np.meshgrid(np.arange(W) - (W - 1) / 2, np.arange(H) - (H - 1) / 2)
    dot = 0.8 * np.exp(-(x * x + y * y))
    dot = np.where(dot >= 1 / 255, dot, 0.0)
    for lowpass in (True, False):
        got = api.Context(sync=True).render_dominant(api.DeviceScene(sc), cam, api.Raster(lowpass=lowpass))
        torch.cuda.synchronize()
        err = np.abs(got["alpha"].cpu().numpy() - (dot if lowpass else 0.0))
        if not lowpass:
            err[x * x + y * y < 1.0] = 0.0  # the centre itself may count as the surfel's one point
        assert err.max() <= 1e-5, lowpass
