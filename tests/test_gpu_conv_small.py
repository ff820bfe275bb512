"""The convolution kernel for launches of few tiles at its edges: one pixel, pixel and channel counts that are no multiple of a tile, every tile
and kind of addresses, reductions of one step, of part of one and of many, windows over every border, residuals, channel slices of
wider buffers, a last vector of less than eight channels; against the oracle's arithmetic, in fp32 against 64 bits."""
import numpy as np
import pytest

import bench
from oracle import nn
from oracle.rounding import round_storage
from paper_2502_01277_amd import synth, zoo
from helpers import TOL, rel_err, small_root

CASES = [
    # (n, h, w, cin, cout, k, stride, act, res_mode, x_extra, y_extra, kernel id)
    (1, 1, 1, 64, 40, 1, 1, nn.ACT_SILU, nn.RES_NONE, 0, 0, 1300320322),                  # one pixel
    (1, 20, 21, 256, 256, 1, 1, nn.ACT_SILU, nn.RES_AFTER_ACT, 64, 8, 1300320322),        # 32 x 32 tiles, four pixels over
    (3, 31, 33, 128, 136, 1, 1, nn.ACT_RELU, nn.RES_BEFORE_ACT, 0, 0, 1300320641),        # 32 x 64, 8 channels of the last tile
    (5, 40, 41, 256, 255, 1, 1, nn.ACT_NONE, nn.RES_NONE, 0, 1, 1301280644),              # 128 x 64, 7 of the last 8 channels
    (7, 57, 55, 64, 192, 1, 1, nn.ACT_SILU, nn.RES_NONE, 0, 0, 130),                       # one K step, more tiles than workgroups
    (2, 56, 57, 24, 256, 1, 1, nn.ACT_RELU, nn.RES_NONE, 8, 0, 132),                      # part of one K step
    (1, 81, 80, 200, 40, 1, 1, nn.ACT_SILU, nn.RES_AFTER_ACT, 0, 0, 1320640322),          # 64 x 32, 8 of the fourth step
    (6, 28, 27, 256, 24, 1, 1, nn.ACT_SILU, nn.RES_NONE, 0, 8, 1300320322),               # less than 32 channels
    (15, 61, 59, 64, 24, 1, 1, nn.ACT_SILU, nn.RES_AFTER_ACT, 0, 8, 1300320641),          # the same of one K step, beyond three tiles per compute unit
    (5, 80, 79, 64, 64, 3, 1, nn.ACT_SILU, nn.RES_AFTER_ACT, 0, 64, 1310640642),          # nine taps of one step
    (2, 7, 9, 128, 264, 3, 1, nn.ACT_RELU, nn.RES_BEFORE_ACT, 0, 0, 131),
    (8, 57, 83, 96, 192, 3, 2, nn.ACT_SILU, nn.RES_NONE, 0, 0, 132),                      # steps across taps
    (1, 160, 161, 64, 128, 3, 2, nn.ACT_SILU, nn.RES_NONE, 8, 0, 131),
    (3, 14, 15, 16, 200, 5, 1, nn.ACT_RELU, nn.RES_AFTER_ACT, 0, 0, 132),
    (40, 3, 4, 64, 96, 2, 2, nn.ACT_NONE, nn.RES_NONE, 0, 0, 131),                        # a tile over several images
    (1, 1, 401, 64, 256, 3, 2, nn.ACT_RELU, nn.RES_NONE, 0, 0, 131),                      # taps that no pixel can use
]


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("case", CASES)
def test_small_launch_parity(octo, dtype, case):
    import torch
    n, h, w, cin, cout, k, stride, act, res_mode, xe, ye, want = case
    pad = k // 2
    rng = np.random.default_rng(83)
    x = zoo.round_to_dtype(rng.uniform(-1, 1, (n, h, w, cin)).astype(np.float32), dtype)
    wt = zoo.round_to_dtype((rng.standard_normal((cout, k, k, cin)) / np.sqrt(k * k * cin)).astype(np.float32), dtype)
    bias = rng.uniform(-0.1, 0.1, cout).astype(np.float32)
    layer = octo.ConvOp(synth.to_storage(wt, dtype), bias, dtype, stride, pad, act)
    ho, wo = layer.out_hw(h, w)
    res = zoo.round_to_dtype(rng.uniform(-1, 1, (n, ho, wo, cout)).astype(np.float32), dtype) if res_mode else None
    y = nn.conv2d(x, wt, stride, pad) + bias
    if res_mode == nn.RES_BEFORE_ACT:
        y = nn.activation(y + res, act)
    else:
        y = nn.activation(y, act) + (res if res_mode else 0.0)
    dx = torch.full((n, h, w, cin + xe), float("inf"), dtype=octo.torch_dtype(dtype), device="cuda")
    dx[..., :cin] = octo.to_device(x, dtype)
    dy = torch.full((n, ho, wo, cout + ye), -7.0, dtype=octo.torch_dtype(dtype), device="cuda")
    kid = octo.op_conv(layer, dx[..., :cin], dy[..., :cout], octo.to_device(res, dtype) if res_mode else None, res_mode)
    torch.cuda.synchronize()
    assert want in (kid, kid // 10000000), kid
    # one rounding to storage on either side; sums of products in fp32
    assert rel_err(dy[..., :cout].float().cpu().numpy(), round_storage(y, dtype)) <= TOL[dtype]
    assert (dy[..., cout:].float().cpu().numpy() == -7.0).all()


CASES_F32 = [
    (1, 1, 1, 32, 20, 1, 1, nn.ACT_SILU, nn.RES_NONE, 0, 0, 1300320322),                   # one pixel, one step
    (2, 320, 321, 4, 16, 3, 2, nn.ACT_SILU, nn.RES_NONE, 0, 4, 132),                       # part of a second step, across taps
    (3, 16, 17, 64, 192, 1, 1, nn.ACT_RELU, nn.RES_AFTER_ACT, 4, 0, 130),
    (5, 56, 57, 128, 255, 1, 1, nn.ACT_NONE, nn.RES_NONE, 0, 1, 130),                      # three of the last four channels
    (1, 33, 31, 44, 72, 1, 1, nn.ACT_SILU, nn.RES_BEFORE_ACT, 20, 0, 133),                 # 12 of the second step's channels
    (9, 31, 33, 36, 136, 1, 2, nn.ACT_RELU, nn.RES_NONE, 12, 8, 134),                      # the same with a stride
    (20, 56, 57, 72, 256, 1, 1, nn.ACT_SILU, nn.RES_AFTER_ACT, 60, 0, 1330640642),         # 64 x 64, several per workgroup
    (2, 57, 55, 64, 96, 3, 2, nn.ACT_SILU, nn.RES_NONE, 0, 0, 131),
    (7, 13, 15, 32, 40, 3, 1, nn.ACT_RELU, nn.RES_BEFORE_ACT, 0, 0, 131),
    (40, 3, 4, 32, 96, 2, 2, nn.ACT_NONE, nn.RES_NONE, 0, 0, 131),                         # a tile over several images
    (1, 1, 401, 32, 256, 3, 2, nn.ACT_RELU, nn.RES_NONE, 0, 0, 131),                       # taps that no pixel can use
    (1, 16, 17, 512, 64, 3, 1, nn.ACT_RELU, nn.RES_NONE, 0, 0, 16),                        # few tiles, 144 steps: split-K
]


@pytest.mark.gpu
@pytest.mark.parametrize("case", CASES_F32)
def test_small_launch_parity_in_fp32(octo, case):
    """Against sums in 64 bits: eight chains of at most K / 8 products (four of K / 4 in 64 x 64 tiles), whose roundings are at most
    2^-24 of the sum of the magnitudes each; with random signs the error is far below K / 4 of them.  Channels behind the slice are
    infinite, and those behind the output stay as they are."""
    import torch
    n, h, w, cin, cout, k, stride, act, res_mode, xe, ye, want = case
    pad = k // 2
    rng = np.random.default_rng(89)
    x = rng.uniform(-1, 1, (n, h, w, cin)).astype(np.float32)
    wt = (rng.standard_normal((cout, k, k, cin)) / np.sqrt(k * k * cin)).astype(np.float32)
    bias = rng.uniform(-0.1, 0.1, cout).astype(np.float32)
    layer = octo.ConvOp(wt, bias, "f32", stride, pad, act)
    ho, wo = layer.out_hw(h, w)
    res = rng.uniform(-1, 1, (n, ho, wo, cout)).astype(np.float32) if res_mode else None
    y = torch.nn.functional.conv2d(torch.from_numpy(x).double().permute(0, 3, 1, 2), torch.from_numpy(wt).double().permute(0, 3, 1, 2),
                                   stride=stride, padding=pad).permute(0, 2, 3, 1).numpy() + bias
    r = res if res_mode else 0.0
    silu = lambda v: v / (1.0 + np.exp(-v)) if act == nn.ACT_SILU else np.maximum(v, 0.0) if act == nn.ACT_RELU else v   # noqa: E731
    y = silu(y + r) if res_mode == nn.RES_BEFORE_ACT else silu(y) + r
    dx = torch.full((n, h, w, cin + xe), float("inf"), device="cuda")
    dx[..., :cin] = octo.to_device(x, "f32")
    dy = torch.full((n, ho, wo, cout + ye), -7.0, device="cuda")
    kid = octo.op_conv(layer, dx[..., :cin], dy[..., :cout], octo.to_device(res, "f32") if res_mode else None, res_mode)
    torch.cuda.synchronize()
    assert str(kid).startswith(str(want)), kid
    assert rel_err(dy[..., :cout].cpu().numpy(), y) <= TOL["f32"] and np.abs(dy[..., :cout].cpu().numpy() - y).max() <= (k * k * cin / 4 + 8) * 2.0 ** -24 * 4
    assert (dy[..., cout:].cpu().numpy() == -7.0).all()


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
def test_two_layers_in_one_small_launch(octo, dtype):
    """Two 1x1 layers in one launch, the second one's channels beginning inside a tile: bit for bit what the layers give on their own."""
    B = zoo._Builder("t", dtype, 20, 22, "classifier", np.random.default_rng(85))
    B.ch = [16]
    B.m.in_c = 16
    x = B.conv(0, 128, 1, 1, act=zoo.ACT_SILU)
    a, b = B.conv(x, 40, 1, 1, act=zoo.ACT_SILU), B.conv(x, 88, 1, 1, act=zoo.ACT_SILU)
    d = B.conv(B.cat([a, b]), 96, 3, 2, act=zoo.ACT_SILU)
    B.m.outputs = [B.fc(B.gap(d), 10)]
    B.m.batch_size = 3
    v = zoo.round_to_dtype(np.random.default_rng(86).uniform(-1, 1, (3, 20, 22, 16)).astype(np.float32), dtype)
    ref = nn.run_model(B.m, v, keep_all=True)
    got, kids = {}, {}
    for keep in (1, 2):                                  # every layer on its own; fused, with every buffer kept
        P = octo.Pipeline(zoo.PipelineSpec("t", [small_root(dtype), B.m], [], 200.0, 32, 32, 1, 1), keep_all_tensors=keep)
        P.run_model_on(1, octo.to_device(v, dtype))
        got[keep], kids[keep] = [P.get_tensor(1, q, 3) for q in (a, b, d)], [int(q) for q in P.layer_info(1)[1]]
        P.close()
    assert kids[2][a - 1] // 100000000 == 13 and kids[2][b - 1] == 0, kids
    for j, q in enumerate((a, b, d)):
        assert rel_err(got[2][j], ref[q]) <= TOL[dtype], q
        assert np.array_equal(got[2][j], got[1][j]), q


def test_the_names_of_the_instances():
    for (bc, bp), (wp, minb) in bench.SMALL.items():
        for mode in range(3):
            wc = {(32, 32): 2, (32, 64): 1, (64, 32): 2, (64, 64): 2, (128, 64): 4}[(bc, bp)]
            kid = 1300000000 + mode * 10000000 + bc * 10000 + bp * 10 + wc
            assert bench.conv_name(kid, "bf16") == "octo::conv_small_kernel<__bf16, %d, %d, %d, %d, %d, %d>" % (bc, bp, wc, wp, minb, mode)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_more_items_on_the_device_than_expected(octo, dtype):
    """Layers of a downstream model shaped for three items whose batches bring hundreds: a workgroup has many tiles, and while the weights are the larger operand of
    the expected items tiles go round channels outside, pixels inside, by a number of pixel tiles that only the device knows.  Every tensor of some ROIs against the
    oracle on the GPU's own crops; a small batch leaves the rest of the larger one's results as they are."""
    import torch
    det = zoo.traffic_cascade(dtype).models[0]
    det.batch_size = 4
    B = zoo._Builder("child", dtype, 8, 8, "classifier", np.random.default_rng(91))
    a = B.conv(0, 64, 3, 2, act=zoo.ACT_RELU)
    b = B.conv(a, 264, 1, 1, act=zoo.ACT_SILU)
    c = B.conv(b, 512, 3, 2, act=zoo.ACT_RELU)
    d = B.conv(c, 1024, 1, 1, act=zoo.ACT_SILU)
    e = B.conv(d, 1000, 1, 1, act=zoo.ACT_RELU)
    B.m.outputs = [B.fc(B.gap(e), 10)]
    B.m.batch_size = 480
    spec = zoo.PipelineSpec("items", [det, B.m], [zoo.Edge(0, 1)], 1000.0, 540, 960, 4, 120)
    rng = np.random.default_rng(92)
    geo = octo.letterbox_geometry(540, 960, det.in_h, det.in_w)
    scenes = [synth.make_scene(rng, 4, 540, 960, counts, 16, 200, log_uniform=True) for counts in ([0, 2, 0, 1], [120] * 4, [1, 0, 2, 0])]
    n_t = len(B.m.layers)
    P = octo.Pipeline(spec, keep_all_tensors=1)
    P.set_expected_items(1, 3)
    before = None
    for k, sc in enumerate(scenes):
        heads = [octo.to_device(v, dtype) for v in synth.planted_heads(rng, det, sc, 540, 960, geo)]
        for l, v in enumerate(heads):
            P.set_head(0, l, v)
        P.submit([torch.from_numpy(f).cuda() for f in sc.frames])
        P.run()
        P.collect()
        n = len(P.get_rois(0))
        assert (1 <= n < 5, n > 200, 1 <= n < 5)[k], n
        kids = [int(v) for v in P.layer_info(1)[1]]
        # (the second batch finds tiles shaped for the three items of the first)
        assert all(kids[t - 1] // 100000000 == 13 for t in (b, d, e)) and (k != 1 or kids[d - 1] % 10000000 == 320322), kids
        at = sorted({0, n // 2, n - 1})
        got = [np.concatenate([P.get_tensor(1, t, 1, first=i) for i in at]) for t in range(n_t + 1)]
        beyond = [np.concatenate([P.get_tensor(1, t, 1, first=i) for i in (60, 120, 199)]) for t in range(n_t + 1)]
        ref = nn.run_model(B.m, got[0], keep_all=True)
        for t in range(1, n_t + 1):
            assert rel_err(got[t].reshape(ref[t].shape), ref[t]) <= TOL[dtype], (k, t)
            if k == 2:
                assert np.array_equal(beyond[t], before[t]), t
        before = beyond
    P.close()
