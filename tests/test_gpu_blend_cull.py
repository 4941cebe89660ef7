"""The blend's region test on single footprints: needles at every angle, specks
about the size of the low-pass disc, and discs, far enough apart that no pixel
sees two.  A record dropped for a region it reaches would leave its pixels
empty, so wherever the oracle's weight is at least twice alpha_min the GPU's
must be there: alpha's relative error is that of its exponent, at most ln 255
times the fp32 error of u^2 + v^2, which a needle of 1:50 raises from 1e-7 to
under 1e-3, so within 1e-2."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2609_30741_amd import api, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["needles", "specks", "discs"])
@pytest.mark.parametrize("lowpass", [True, False])
def test_region_test_keeps_every_footprint(kind, lowpass):
    rng = np.random.default_rng(23)
    gx, gy = np.meshgrid(np.linspace(-1.2, 1.2, 9), np.linspace(-0.9, 0.9, 7))
    n = gx.size
    pos = np.stack([gx.ravel(), np.zeros(n), gy.ravel()], axis=1) + rng.uniform(-0.02, 0.02, size=(n, 3))
    tu, tv = rng.normal(size=(n, 3)), rng.normal(size=(n, 3))
    tu /= np.linalg.norm(tu, axis=1, keepdims=True)
    tv -= (tv * tu).sum(1, keepdims=True) * tu
    su, sv = {"needles": (0.03, 0.0006), "specks": (0.002, 0.002), "discs": (0.03, 0.03)}[kind]
    sc = synth.explicit_scene(pos, tu, tv, np.full(n, su), np.full(n, sv), rng.uniform(0.2, 0.95, n),
                              rng.uniform(0.2, 1.0, size=(n, 3)))
    cam = synth.look_at((0.0, -4.0, 0.0), (0.0, 0.0, 0.0), (0.0, 0.0, 1.0), 333, 251, 500.0)
    out = api.Context().render_dominant(api.DeviceScene(sc), cam, api.Raster(lowpass=lowpass))
    torch.cuda.synchronize()
    a, ref = out["alpha"].cpu().numpy(), O.render(sc, cam, O.Raster(lowpass=lowpass))["alpha"]
    seen = ref >= 2.0 / 255.0
    assert seen.sum() > (20 if kind == "specks" and not lowpass else 200)
    assert np.all(np.abs(a[seen] - ref[seen]) <= 1e-2 * ref[seen])
