"""A frame with more than 2^32 tile keys: its count stops there and reports
the overflow (it does not come round to a number that fits)."""
import pytest

from paper_2609_30741_amd import api, synth

pytestmark = pytest.mark.gpu


# 2^20 tiles of 16384x16384, each met by every surfel: the disc of one that
# reaches behind the camera is bounded by the whole image.  (262200: more
# than 2^32 entries too, one per surfel and cell.)
@pytest.mark.parametrize("n", [4100, 262_200])
def test_more_keys_than_a_word_counts(n):
    W = H = 16384
    sc = synth.scene_uniform_cube(2, n, log_scale=(3.0, 0.1))
    cam = synth.look_at((0.0, -4.0, 0.0), (0, 0, 0), (0, 0, 1), W, H, 1.1 * W)
    ctx = api.Context(sync=False)
    ds = api.DeviceScene(sc)
    _, _, counts = ctx.preprocess_debug(ds, cam)
    assert int(counts.long().sum()) > 1 << 32
    ctx.reserve(n, W, H, 6 << 20)
    ctx.render_dominant(ds, cam)
    stats = ctx.poll_status()
    assert stats["overflow"] & 1 and stats["n_keys_dom"] == (1 << 32) - 1
