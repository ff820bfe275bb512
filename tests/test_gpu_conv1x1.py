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
    (5, 40, 41, 120, 520, nn.ACT_RELU, nn.RES_BEFORE_ACT, 0, 8),       # nine channel tiles, the last one of 8 channels
    (9, 64, 33, 64, 256, nn.ACT_RELU, nn.RES_BEFORE_ACT, 64, 0),       # 128-channel tiles
    (2, 160, 111, 184, 192, nn.ACT_SILU, nn.RES_AFTER_ACT, 0, 192),    # the longest reduction that is never the other kernel's
    (9, 160, 163, 192, 192, nn.ACT_SILU, nn.RES_AFTER_ACT, 0, 192),    # the longest of all, whose tensors exceed the memory-side cache
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


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("cin,cout,res", [(64, 32, False), (96, 32, False), (64, 64, False), (128, 64, True)])
def test_results_do_not_change_with_the_running_item_count(octo, dtype, cin, cout, res):
    """1x1 layers of a downstream model: the running average of its item counts must not choose between kernels that sum in different
    orders.  The model's capacity stands in for the average before the first batch, so the same frame repeated, and then beside frames
    with many more objects, runs with three different averages.  A larger count is stated last, for which the other order is right."""
    import torch
    det = zoo.traffic_cascade(dtype).models[0]
    det.batch_size = 4
    B = zoo._Builder("child", dtype, 32, 32, "classifier", np.random.default_rng(19))
    a = B.conv(0, cin, 3, 2, act=zoo.ACT_RELU)
    a = B.conv(a, cout, 1, 1, act=zoo.ACT_NONE, **(dict(res=B.conv(a, cout, 3, 1), res_mode=zoo.RES_BEFORE_ACT) if res else {}))
    at = len(B.m.layers)
    B.m.outputs = [B.fc(B.gap(a), 10)]
    B.m.batch_size = 400
    spec = zoo.PipelineSpec("items", [det, B.m], [zoo.Edge(0, 1)], 1000.0, 540, 960, 4, 100)
    rng = np.random.default_rng(zoo.SEED0 + 92)
    scene = synth.make_scene(rng, 4, 540, 960, [9, 120, 120, 120], 16, 200, log_uniform=True)
    planted = synth.planted_heads(rng, det, scene, 540, 960, octo.letterbox_geometry(540, 960, det.in_h, det.in_w))
    heads = [octo.to_device(v, dtype) for v in planted]
    frames = [torch.from_numpy(f).cuda() for f in scene.frames]
    P = octo.Pipeline(spec, keep_all_tensors=1)
    for l, v in enumerate(heads):
        P.set_head(0, l, v)
    kernels = []
    for expected in (8, 400):
        P.set_expected_items(1, expected)
        first = None
        for n in (1, 1, 1, 4, 4, 4, 1):
            P.submit(frames[:n])
            P.run()
            P.collect()
            assert len(P.get_rois(0)) > (4 if n == 1 else 200)
            got = P.get_tensor(1, at, 5)
            first = got if first is None else first
            assert np.array_equal(got, first), (expected, n, P.layer_info(1)[1])
        kernels.append(int(P.layer_info(1)[1][at - 1]) // 100000000)
    P.close()
    assert kernels[1] != 16 and (kernels[0] == 16 or cout == 64), kernels
