"""Component labels at the edges of the 64x16 labelling tiles, on masks whose
pieces touch along borders, at corners only, and along long detours: bit
exact against the oracle."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_2609_30741_amd import api
    return api.Context()


def masks(H, W):
    y, x = np.mgrid[0:H, 0:W]
    rng = np.random.default_rng(H * 1000 + W)
    yield "diagonals down", (x - y) % 5 == 0
    yield "diagonals up", (x + y) % 7 == 0
    yield "comb", (x % 2 == 0) | (y == H - 1)
    yield "rings", np.maximum(abs(x - W // 2), abs(y - H // 2)) % 2 == 0
    yield "crossing", ((x - y) % 16 == 0) | ((x + y) % 16 == 15)
    for d in (0.35, 0.5, 0.62):
        yield f"noise {d}", rng.uniform(size=(H, W)) < d


@pytest.mark.parametrize("H,W", [(16, 64), (15, 63), (17, 65), (33, 129), (48, 192), (1, 200), (70, 1), (130, 331)])
@pytest.mark.parametrize("conn", [4, 8])
def test_labels_across_tiles(ctx, oracle, H, W, conn):
    for name, mask in masks(H, W):
        mask = mask.astype(np.uint8)
        lab = ctx.label_components(torch.from_numpy(mask).cuda(), conn).cpu().numpy()
        assert np.array_equal(lab, oracle.label_components(mask, conn)), name
