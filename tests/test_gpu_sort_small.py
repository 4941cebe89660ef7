"""The one-workgroup sort at the edges of its instances (2, 6, 10 and 16 keys
a thread of 1024) and just past it, bit for bit against a stable reference
sort; keys that differ in the sorted bits only by their order must stay."""
import numpy as np
import pytest
import torch

from paper_2609_30741_amd import api, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [2, 63, 64, 65, 1025, 2048, 2049, 6144, 6145, 10240, 10241, 16383, 16384, 16385])
def test_small_sorts_bit_exact(n):
    ctx = api.Context()
    for bits in (1, 7, 8, 9, 17, 24, 32):
        keys, vals = synth.random_sort_keys(n, seed=n + bits, key_bits=32)
        if bits == 9:
            keys[:] = keys[0]  # one digit holds everything
        kt = torch.from_numpy(keys.view(np.int32).copy()).cuda()
        vt = torch.from_numpy(vals.view(np.int32).copy()).cuda()
        ctx.sort_pairs(kt, vt, bits)
        torch.cuda.synchronize()
        order = np.argsort(keys & np.uint32((1 << bits) - 1), kind="stable")
        assert np.array_equal(kt.cpu().numpy().view(np.uint32), keys[order]), bits
        assert np.array_equal(vt.cpu().numpy().view(np.uint32), vals[order]), bits
