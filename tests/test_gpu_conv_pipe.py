"""The pipelined shapes of the general convolution kernel at their edges: pixel counts and channel counts that are no multiple of a tile,
reductions that end inside a K step, strides over odd images, residuals, wider output buffers; against the oracle's arithmetic."""
import numpy as np
import pytest

from oracle import nn
from oracle.rounding import round_storage
from paper_2502_01277_amd import synth, zoo
from helpers import TOL, rel_err

pytestmark = pytest.mark.gpu

CASES = [
    # (n, h, w, cin, cout, k, stride, act, res_mode, kernel id)
    (17, 79, 83, 40, 120, 3, 2, nn.ACT_SILU, nn.RES_NONE, 1128064827),
    (53, 16, 9, 1032, 504, 1, 1, nn.ACT_RELU, nn.RES_BEFORE_ACT, 1128064827),
    (17, 29, 31, 520, 192, 1, 1, nn.ACT_SILU, nn.RES_AFTER_ACT, 1064128827),
    (7, 53, 51, 64, 250, 3, 2, nn.ACT_RELU, nn.RES_NONE, 1064064837),
    (9, 57, 83, 96, 192, 3, 2, nn.ACT_SILU, nn.RES_NONE, 1064064837),
    (4, 223, 225, 64, 200, 3, 2, nn.ACT_SILU, nn.RES_NONE, 1128256427),
    (200, 16, 17, 552, 256, 1, 1, nn.ACT_RELU, nn.RES_BEFORE_ACT, 1128256427),
]


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("case", CASES)
def test_pipelined_shapes(octo, dtype, case):
    import torch
    n, h, w, cin, cout, k, stride, act, res_mode, want = case
    pad = k // 2
    rng = np.random.default_rng(53)
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
    dy = torch.full((n, ho, wo, cout + 6), -7.0, dtype=octo.torch_dtype(dtype), device="cuda")
    kid = octo.op_conv(layer, octo.to_device(x, dtype), dy[..., :cout], octo.to_device(res, dtype) if res_mode else None, res_mode)
    torch.cuda.synchronize()
    assert kid == want
    assert rel_err(dy[..., :cout].float().cpu().numpy(), round_storage(y, dtype)) <= TOL[dtype]
    assert (dy[..., cout:].float().cpu().numpy() == -7.0).all()
