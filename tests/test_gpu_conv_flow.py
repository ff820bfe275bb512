"""The convolution kernel whose stream of loads runs across tiles, at its edges: pixel and channel counts that are no multiple of a tile,
workgroups with several tiles, two K steps, reductions that end inside a step, windows over image borders, strides over odd images,
residuals, channel slices of wider buffers; against the oracle's arithmetic.  The kernel id says which tile and which kind of
addresses a launch took."""
import numpy as np
import pytest

from oracle import nn
from oracle.rounding import round_storage
from paper_2502_01277_amd import synth, zoo
from helpers import TOL, rel_err

pytestmark = pytest.mark.gpu

CASES = [
    # (n, h, w, cin, cout, k, stride, act, res_mode, x_extra, y_extra, kernel id)
    (15, 53, 16, 128, 464, 1, 1, nn.ACT_SILU, nn.RES_NONE, 0, 8, 1200962568),
    (27, 60, 61, 128, 120, 1, 1, nn.ACT_RELU, nn.RES_BEFORE_ACT, 64, 0, 1201280648),
    (60, 40, 41, 192, 96, 1, 1, nn.ACT_SILU, nn.RES_AFTER_ACT, 0, 0, 1200962568),
    (9, 41, 39, 256, 72, 1, 1, nn.ACT_NONE, nn.RES_NONE, 0, 64, 1200640648),
    (33, 40, 40, 384, 384, 1, 1, nn.ACT_SILU, nn.RES_NONE, 0, 0, 1201921288),
    (9, 41, 40, 192, 255, 1, 1, nn.ACT_NONE, nn.RES_NONE, 0, 1, 1201281288),
    (9, 41, 40, 192, 253, 1, 1, nn.ACT_SILU, nn.RES_NONE, 0, 3, 1201281288),
    (31, 80, 79, 64, 250, 3, 2, nn.ACT_RELU, nn.RES_NONE, 0, 6, 1212561288),
    (7, 33, 31, 520, 172, 1, 1, nn.ACT_RELU, nn.RES_NONE, 0, 4, 1221280648),
    (40, 57, 55, 64, 128, 1, 2, nn.ACT_NONE, nn.RES_NONE, 0, 0, 1211281288),             # one K step
    (40, 57, 55, 56, 190, 1, 2, nn.ACT_RELU, nn.RES_NONE, 0, 2, 1221921288),             # three quarters of one
    (33, 40, 41, 256, 64, 1, 1, nn.ACT_SILU, nn.RES_NONE, 0, 0, 1200641288),
    (9, 159, 157, 128, 120, 3, 2, nn.ACT_RELU, nn.RES_NONE, 0, 0, 1211282568),
    (25, 61, 63, 64, 128, 3, 2, nn.ACT_RELU, nn.RES_NONE, 0, 0, 1211281288),
    (70, 55, 57, 128, 256, 3, 2, nn.ACT_SILU, nn.RES_NONE, 0, 0, 1212561288),
    (6, 131, 127, 128, 192, 3, 2, nn.ACT_SILU, nn.RES_AFTER_ACT, 8, 8, 1211921288),
    (8, 160, 163, 48, 96, 3, 2, nn.ACT_SILU, nn.RES_NONE, 0, 0, 1220962568),
    (31, 59, 51, 168, 392, 1, 2, nn.ACT_SILU, nn.RES_NONE, 0, 0, 1222561288),
    (17, 54, 34, 184, 376, 5, 1, nn.ACT_RELU, nn.RES_AFTER_ACT, 0, 0, 1221921288),
    (23, 48, 52, 200, 176, 2, 2, nn.ACT_RELU, nn.RES_BEFORE_ACT, 0, 0, 1221281288),
    (81, 40, 40, 128, 64, 3, 2, nn.ACT_RELU, nn.RES_NONE, 0, 0, 1064064837),             # two 64 x 64 tiles per compute unit at most: general kernel
    (82, 40, 40, 128, 64, 3, 2, nn.ACT_RELU, nn.RES_NONE, 0, 0, 1210640648),             # 513
]


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("case", CASES)
def test_flow_parity(octo, dtype, case):
    import torch
    n, h, w, cin, cout, k, stride, act, res_mode, xe, ye, want = case
    pad = k // 2
    rng = np.random.default_rng(59)
    x = zoo.round_to_dtype(rng.uniform(-1, 1, (n, h, w, cin)).astype(np.float32), dtype)
    wt = zoo.round_to_dtype((rng.standard_normal((cout, k, k, cin)) / np.sqrt(k * k * cin)).astype(np.float32), dtype)
    bias = rng.uniform(-0.1, 0.1, cout).astype(np.float32)
    layer = octo.ConvOp(synth.to_storage(wt, dtype), bias, dtype, stride, pad, act)
    ho, wo = layer.out_hw(h, w)
    res = zoo.round_to_dtype(rng.uniform(-1, 1, (n, ho, wo, cout)).astype(np.float32), dtype) if res_mode else None
    xp = np.zeros((n, h + 2 * pad, w + 2 * pad, cin), np.float32)
    xp[:, pad:pad + h, pad:pad + w] = x
    y = np.zeros((n * ho * wo, cout), np.float32)
    for r in range(k):
        for s in range(k):
            y += np.ascontiguousarray(xp[:, r:r + stride * ho:stride, s:s + stride * wo:stride][:, :ho, :wo]).reshape(-1, cin) @ np.ascontiguousarray(wt[:, r, s].T)
    y = (y + bias).reshape(n, ho, wo, cout)
    if res_mode == nn.RES_BEFORE_ACT:
        y = nn.activation(y + res, act)
    else:
        y = nn.activation(y, act) + (res if res_mode else 0.0)
    dx = torch.full((n, h, w, cin + xe), float("inf"), dtype=octo.torch_dtype(dtype), device="cuda")
    dx[..., :cin] = octo.to_device(x, dtype)
    dy = torch.full((n, ho, wo, cout + ye), -7.0, dtype=octo.torch_dtype(dtype), device="cuda")
    kid = octo.op_conv(layer, dx[..., :cin], dy[..., :cout], octo.to_device(res, dtype) if res_mode else None, res_mode)
    torch.cuda.synchronize()
    assert kid == want
    assert rel_err(dy[..., :cout].float().cpu().numpy(), round_storage(y, dtype)) <= TOL[dtype]
    assert (dy[..., cout:].float().cpu().numpy() == -7.0).all()
