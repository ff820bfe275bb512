"""The streaming 1x1 convolution kernel at its edges: pixel counts that are no multiple of a block or of the chip, channel
counts below a tile and over several tiles, reductions that are no multiple of a matrix step, residuals, channel slices of
wider buffers; against the oracle."""
import numpy as np
import pytest

from oracle import nn
from oracle.rounding import round_storage
from paper_2502_01277_amd import synth, zoo
from helpers import TOL, rel_err

pytestmark = pytest.mark.gpu

CASES = [
    # (n, h, w, cin, cout, act, res_mode, x_extra, y_extra): extra = channels of a wider buffer around the tensor
    (3, 107, 103, 96, 96, nn.ACT_SILU, nn.RES_NONE, 0, 0),             # 33063 pixels: 1033 blocks and 7 pixels
    (1, 181, 181, 24, 40, nn.ACT_RELU, nn.RES_AFTER_ACT, 8, 16),       # three vectors of K, 40 channels on a 64-channel tile
    (2, 131, 127, 16, 32, nn.ACT_NONE, nn.RES_NONE, 0, 0),             # the shortest reduction, 32-channel tile
    (5, 40, 41, 128, 520, nn.ACT_RELU, nn.RES_BEFORE_ACT, 0, 8),       # nine channel tiles, the last one of 8 channels
    (9, 64, 33, 64, 256, nn.ACT_RELU, nn.RES_BEFORE_ACT, 64, 0),       # 128-channel tiles
    (2, 160, 111, 192, 192, nn.ACT_SILU, nn.RES_AFTER_ACT, 0, 192),    # the longest reduction
]


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("case", CASES)
def test_streaming_1x1_parity(octo, dtype, case):
    import torch
    n, h, w, cin, cout, act, res_mode, xe, ye = case
    rng = np.random.default_rng(41)
    x = zoo.round_to_dtype(rng.uniform(-1, 1, (n, h, w, cin)).astype(np.float32), dtype)
    wt = zoo.round_to_dtype((rng.standard_normal((cout, 1, 1, cin)) / np.sqrt(cin)).astype(np.float32), dtype)
    bias = rng.uniform(-0.1, 0.1, cout).astype(np.float32)
    layer = octo.ConvOp(synth.to_storage(wt, dtype), bias, dtype, 1, 0, act)
    res = zoo.round_to_dtype(rng.uniform(-1, 1, (n, h, w, cout)).astype(np.float32), dtype) if res_mode else None
    y = x.reshape(-1, cin).astype(np.float64) @ wt.reshape(cout, cin).astype(np.float64).T + bias.astype(np.float64)
    y = y.reshape(n, h, w, cout)
    if res_mode == nn.RES_BEFORE_ACT:
        y = nn.activation(y + res, act)
    else:
        y = nn.activation(y, act) + (res if res_mode else 0.0)
    dx = torch.full((n, h, w, cin + xe), 5.0, dtype=octo.torch_dtype(dtype), device="cuda")
    dx[..., :cin] = octo.to_device(x, dtype)
    dy = torch.full((n, h, w, cout + ye), -7.0, dtype=octo.torch_dtype(dtype), device="cuda")
    kid = octo.op_conv(layer, dx[..., :cin], dy[..., :cout], octo.to_device(res, dtype) if res_mode else None, res_mode)
    torch.cuda.synchronize()
    assert 1500000000 <= kid < 1600000000
    assert rel_err(dy[..., :cout].float().cpu().numpy(), round_storage(y, dtype)) <= TOL[dtype]
    assert (dy[..., cout:].float().cpu().numpy() == -7.0).all()
