"""Labels of components that run back and forth across many labelling tiles,
whose pieces are joined through long paths: bit exact against the oracle, and
the same from call to call."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def serpentine(H, W, step):
    m = np.zeros((H, W), bool)
    m[::step] = True
    for i, y in enumerate(range(0, H - step, step)):
        m[y:y + step, 0 if i % 2 else W - 1] = True
    return m


def spiral(H, W):
    m = np.zeros((H, W), bool)
    a, b, c, d = 0, 0, H - 1, W - 1
    while a + 2 < c and b + 2 < d:
        m[a, b:d + 1] = m[a:c + 1, d] = m[c, b:d + 1] = m[a + 2:c + 1, b] = m[a + 2, b:b + 3] = True
        a, b, c, d = a + 2, b + 2, c - 2, d - 2
    return m


@pytest.mark.parametrize("conn", [4, 8])
@pytest.mark.parametrize("name,mask", [("serpentine", serpentine(601, 1503, 2)), ("broad", serpentine(901, 1003, 8)),
                                       ("upright", serpentine(903, 701, 2).T), ("spiral", spiral(701, 903)),
                                       ("checker", np.indices((700, 900)).sum(0) % 2 == 0)])
def test_long_paths(oracle, name, mask, conn):
    from paper_2609_30741_amd import api
    mask = np.ascontiguousarray(mask).astype(np.uint8)
    ctx, m = api.Context(), torch.from_numpy(mask).cuda()
    want = oracle.label_components(mask, conn)
    for _ in range(5):
        assert np.array_equal(ctx.label_components(m, conn).cpu().numpy(), want), name
