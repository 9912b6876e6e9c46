"""Edges of single kernels (tile remainders, smallest and largest of a range,
special values) through the public entry points."""
import numpy as np
import pytest
import torch

from oracle import mlp as M
from paper_1904_08553_amd import dc

pytestmark = pytest.mark.gpu


def dev_bits(bits):
    return torch.from_numpy(bits.astype(np.uint16).view(np.int16)).cuda().contiguous()


@pytest.mark.parametrize("n", [15, 17, 65_536 + 3])
def test_forward_tiles_and_nan_rows(n):
    """The logit of a sample depends on that sample alone, wherever its tile
    lies in a wave's walk, and a NaN feature makes every first-layer unit's
    activation 0: exactly the logit of a network without its first layer."""
    print(f"case: mlp forward tiles n={n}", flush=True)
    rng = np.random.default_rng(n)
    w = M.init_weights(n)
    w[M.OFF_B2:M.OFF_W3] = 0.05
    bits = M.bf16_bits(rng.uniform(-1, 1, (n, 8))).reshape(n, 8)
    nan = rng.random(n) < 0.1
    bits[nan, rng.integers(0, 8)] = 0x7FC0
    net = dc.MLP(w)
    z = net.forward(dev_bits(bits)).cpu().numpy()
    off = 16 * (n // 32) + 3  # other tiles, other lanes
    z_off = net.forward(dev_bits(bits[off:])).cpu().numpy()
    assert np.array_equal(z[off:], z_off)
    w0 = w.copy()
    w0[:M.OFF_W2] = 0.0  # W1 and b1
    net0 = dc.MLP(w0)
    z0 = net0.forward(dev_bits(np.zeros((1, 8), np.uint16))).cpu().numpy()[0]
    assert np.all(z[nan] == z0)
    assert np.all(np.isfinite(z))
    net.close()
    net0.close()
