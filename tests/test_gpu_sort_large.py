"""Sorts past one workgroup, on both sides of the sizes at which a block's
chunk takes more threads or keys, and where the last sub-chunk of a chunk is
nearly empty or the last blocks have no chunk: bit for bit against a stable
reference sort."""
import numpy as np
import pytest
import torch

from paper_2609_30741_amd import api, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [16641, 524288, 524289, 1048576, 1048577, 2097152, 2097153, 4194305, 2500001])
@pytest.mark.parametrize("bits", [3, 13, 32])
def test_large_sorts_bit_exact(n, bits):
    keys, vals = synth.random_sort_keys(n, seed=n + bits, key_bits=32)
    if bits == 3:
        keys[n // 3:] = keys[0]  # a digit with most of the keys, across blocks
    kt = torch.from_numpy(keys.view(np.int32).copy()).cuda()
    vt = torch.from_numpy(vals.view(np.int32).copy()).cuda()
    api.Context().sort_pairs(kt, vt, bits)
    torch.cuda.synchronize()
    order = np.argsort(keys & np.uint32((1 << bits) - 1), kind="stable")
    assert np.array_equal(kt.cpu().numpy().view(np.uint32), keys[order])
    assert np.array_equal(vt.cpu().numpy().view(np.uint32), vals[order])
