"""Inference forms the network's input inside the first layer and writes the
repaired image from the last; training keeps both as tensors.  The same sums
in the same order, so the two give the same image bit for bit, at the edges
of the 64-pixel blocks, with and without the error channel, and in place."""
import numpy as np
import pytest
import torch

from paper_2609_30741_amd import repair

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,H,W", [(1, 4, 4), (2, 12, 64), (1, 20, 68), (3, 36, 132)])
def test_inference_image_equals_the_training_pass(B, H, W):
    rng = np.random.default_rng(H * W)
    hole = torch.from_numpy((rng.uniform(size=(B, H, W)) < 0.3).astype(np.uint8)).cuda()
    rgb = torch.from_numpy(rng.uniform(size=(B, 3, H, W)).astype(np.float32)).cuda()
    z = torch.from_numpy(np.where(rng.uniform(size=(B, H, W)) < 0.2, np.inf,
                                  rng.uniform(1.5, 4.0, size=(B, H, W))).astype(np.float32)).cuda()
    net = repair.Repair(seed=4)
    trained, err = torch.empty_like(rgb), torch.empty_like(z)
    net.grad_step(rgb, z, hole, rgb, rgb_out=trained)
    out = net.forward(rgb, z, hole, err=err)
    bare = net.forward(rgb, z, hole)
    again = rgb.clone()
    net.forward(again, z, hole, out=again)
    torch.cuda.synchronize()
    for got in (out, bare, again):
        assert torch.equal(got, trained)
    assert torch.all(err[hole == 0] == 0) and torch.all(torch.isfinite(err)) and float(err.abs().max()) > 0
