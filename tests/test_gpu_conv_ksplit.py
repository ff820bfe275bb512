"""The split-K convolution kernel at the sizes where it can go wrong: ragged pixel and channel counts, reductions shorter
than the number of wavefronts that share them, element-wise stores, residuals, fp32 output; against the oracle.  The
kernel id says that the launch took the shape meant (split, channel tile, pixel tile)."""
import numpy as np
import pytest

from oracle import nn
from oracle.rounding import round_storage
from paper_2502_01277_amd import synth, zoo
from helpers import TOL, rel_err

pytestmark = pytest.mark.gpu

CASES = [
    # (n, h, w, cin, cout, k, stride, pad, act, res_mode, shape in the 16-bit types)
    (1, 19, 21, 256, 250, 3, 1, 1, nn.ACT_SILU, nn.RES_AFTER_ACT, (8, 32, 32)),     # 399 pixels, channel tail, odd pitch
    (1, 20, 20, 256, 256, 3, 1, 1, nn.ACT_RELU, nn.RES_BEFORE_ACT, (8, 32, 32)),
    (1, 13, 7, 72, 40, 1, 1, 0, nn.ACT_SILU, nn.RES_NONE, (4, 32, 32)),             # two K steps for four wavefronts, the second a fragment
    (1, 1, 1, 64, 10, 1, 1, 0, nn.ACT_NONE, nn.RES_NONE, (4, 32, 32)),              # one pixel, one K step
    (2, 23, 19, 520, 130, 1, 1, 0, nn.ACT_RELU, nn.RES_BEFORE_ACT, (4, 32, 32)),    # 17 K steps in bf16: unequal shares
    (3, 41, 37, 128, 200, 3, 2, 1, nn.ACT_SILU, nn.RES_NONE, (4, 64, 32)),          # stride 2 over image borders
    (6, 14, 14, 256, 256, 3, 1, 1, nn.ACT_RELU, nn.RES_AFTER_ACT, (4, 64, 32)),
    (5, 78, 82, 128, 120, 3, 2, 1, nn.ACT_SILU, nn.RES_BEFORE_ACT, (4, 64, 64)),    # tiles over several images
]


@pytest.mark.parametrize("dtype", ["bf16", "f16", "f32"])
@pytest.mark.parametrize("case", CASES)
def test_split_k_parity(octo, dtype, case):
    import torch
    n, h, w, cin, cout, k, stride, pad, act, res_mode, shape = case
    rng = np.random.default_rng(31)
    x = zoo.round_to_dtype(rng.uniform(-1, 1, (n, h, w, cin)).astype(np.float32), dtype)
    wt = zoo.round_to_dtype((rng.standard_normal((cout, k, k, cin)) / np.sqrt(k * k * cin)).astype(np.float32), dtype)
    bias = rng.uniform(-0.1, 0.1, cout).astype(np.float32)
    layer = octo.ConvOp(synth.to_storage(wt, dtype), bias, dtype, stride, pad, act)
    ho, wo = layer.out_hw(h, w)
    res = zoo.round_to_dtype(rng.uniform(-1, 1, (n, ho, wo, cout)).astype(np.float32), dtype) if res_mode else None
    y = nn.conv2d(x, wt, stride, pad) + bias.astype(np.float64)
    if res_mode == nn.RES_BEFORE_ACT:
        y = nn.activation(y + res, act)
    else:
        y = nn.activation(y, act) + (res if res_mode else 0.0)
    dx = octo.to_device(x, dtype)
    dres = octo.to_device(res, dtype) if res_mode else None
    dy = torch.full((n, ho, wo, cout + 5), -7.0, dtype=octo.torch_dtype(dtype), device="cuda")
    kid = octo.op_conv(layer, dx, dy[..., :cout], dres, res_mode)
    dy32 = torch.full((n, ho, wo, cout), -7.0, dtype=torch.float32, device="cuda")
    octo.op_conv(layer, dx, dy32, dres, res_mode, out_f32=True)
    torch.cuda.synchronize()
    assert 1600000000 <= kid < 1700000000
    if dtype != "f32":
        ks, bc, bp = shape
        assert kid == 1600000000 + ks * 1000000 + bc * 1000 + bp
    assert rel_err(dy[..., :cout].float().cpu().numpy(), round_storage(y, dtype)) <= TOL[dtype]
    assert (dy[..., cout:].float().cpu().numpy() == -7.0).all()                     # nothing beyond the channels
    assert rel_err(dy32.cpu().numpy(), y) <= (1e-4 if dtype == "f32" else 2e-3)
