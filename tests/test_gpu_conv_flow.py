"""The convolution kernel whose stream of loads runs across tiles, at its edges: pixel and channel counts that are no multiple of a tile,
workgroups with several tiles, two K steps, reductions that end inside a step, windows over image borders, strides over odd images,
residuals, channel slices of wider buffers; against the oracle's arithmetic.  The kernel id says which tile and which kind of
addresses a launch took."""
import numpy as np
import pytest

from oracle import nn
from oracle.rounding import round_storage
from paper_2502_01277_amd import synth, zoo
from helpers import TOL, rel_err, small_root

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
# maps no taller than the padding: in the last image's tiles, taps that no pixel can use start behind the end of the tensor.  Any tile
FLAT = [
    (1, 1, 40001, 64, 256, 3, 2, nn.ACT_RELU, nn.RES_NONE, 0, 0, 121),
    (1, 2, 40003, 64, 256, 5, 2, nn.ACT_NONE, nn.RES_NONE, 8, 0, 121),
    (3, 1, 20003, 128, 192, 3, 2, nn.ACT_SILU, nn.RES_BEFORE_ACT, 0, 8, 121),
]
# maps smaller than the window, a tile over hundreds of images
TINY = [
    (40000, 2, 2, 64, 128, 3, 2, nn.ACT_RELU, nn.RES_NONE, 0, 0, 121),
    (9000, 3, 4, 128, 96, 3, 2, nn.ACT_SILU, nn.RES_NONE, 0, 8, 121),
    (6000, 4, 3, 72, 200, 2, 2, nn.ACT_RELU, nn.RES_AFTER_ACT, 0, 0, 122),
]
# a residual, written into channel slices
SLICES = [
    (5, 40, 41, 128, 520, 1, 1, nn.ACT_RELU, nn.RES_BEFORE_ACT, 0, 8, 120),
    (2, 160, 111, 192, 192, 1, 1, nn.ACT_SILU, nn.RES_AFTER_ACT, 0, 192, 120),
]


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("case", CASES + FLAT + TINY + SLICES)
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
    assert want in (kid, kid // 10000000), kid
    assert rel_err(dy[..., :cout].float().cpu().numpy(), round_storage(y, dtype)) <= TOL[dtype]
    assert (dy[..., cout:].float().cpu().numpy() == -7.0).all()


@pytest.mark.parametrize("n,h,w,cin,cout,k,stride,res,xe,ye,mode", [
    (33, 40, 41, 384, 400, 1, 1, nn.RES_BEFORE_ACT, 0, 16, 0),     # three whole K steps, 16 of the last tile's channels
    (9, 41, 39, 256, 80, 1, 1, nn.RES_NONE, 128, 0, 0),            # two steps, several channel tiles of 64
    (60, 40, 41, 96, 96, 1, 1, nn.RES_AFTER_ACT, 0, 0, 2),         # one step, part of it
    (21, 56, 55, 64, 256, 1, 1, nn.RES_NONE, 0, 0, 2),             # half a step, the widest channel tile
    (5, 33, 31, 528, 176, 1, 1, nn.RES_NONE, 16, 32, 2),           # 16 of the fifth step
    (25, 61, 63, 128, 128, 3, 2, nn.RES_BEFORE_ACT, 0, 0, 1),      # a tap per step, windows over every border
    (8, 160, 163, 48, 96, 3, 2, nn.RES_NONE, 0, 0, 2),             # steps across taps
    (17, 54, 34, 112, 368, 5, 1, nn.RES_AFTER_ACT, 0, 0, 2),
    (1, 1, 80011, 128, 256, 3, 2, nn.RES_NONE, 0, 0, 1),           # a map no taller than the padding
])
def test_flow_fp8(octo, n, h, w, cin, cout, k, stride, res, xe, ye, mode):
    import torch
    rng = np.random.default_rng(61)
    pad = k // 2
    f8 = lambda shape: torch.from_numpy(rng.standard_normal(shape).astype(np.float32)).to(torch.float8_e4m3fn)
    x, wt = f8((n, h, w, cin)), f8((cout, k, k, cin))
    scale, bias = (rng.uniform(0.5, 1.0, cout) / np.sqrt(k * k * cin)).astype(np.float32), rng.uniform(-0.1, 0.1, cout).astype(np.float32)
    layer = octo.ConvOp(wt.view(torch.uint8).numpy(), bias, "f8", stride, pad, nn.ACT_RELU, scale=scale)
    ho, wo = layer.out_hw(h, w)
    r = f8((n, ho, wo, cout)) if res else None
    dx = torch.full((n, h, w, cin + xe), 0x7F, dtype=torch.uint8, device="cuda")       # NaN beside the tensor
    dx[..., :cin] = x.view(torch.uint8).cuda()
    dy = torch.full((n, ho, wo, cout + ye), 0x55, dtype=torch.uint8, device="cuda")
    kid = octo.op_conv(layer, dx[..., :cin], dy[..., :cout], r.view(torch.uint8).cuda() if res else None, res, res_scale=0.5, y_inv_scale=2.0)
    torch.cuda.synchronize()
    assert kid // 10000000 == 120 + mode, kid
    xf, wf = np.zeros((n, h + 2 * pad, w + 2 * pad, cin), np.float32), wt.float().numpy()
    xf[:, pad:pad + h, pad:pad + w] = x.float().numpy()
    acc = np.zeros((n * ho * wo, cout), np.float32)
    for p in range(k):
        for q in range(k):
            acc += np.ascontiguousarray(xf[:, p:p + stride * ho:stride, q:q + stride * wo:stride][:, :ho, :wo]).reshape(-1, cin) @ np.ascontiguousarray(wf[:, p, q].T)
    v = (acc * scale + bias).reshape(n, ho, wo, cout)
    add = 0.5 * r.float().numpy() if res else 0.0
    v = np.maximum(v + add, 0.0) if res == nn.RES_BEFORE_ACT else np.maximum(v, 0.0) + add
    want = torch.from_numpy(np.clip(v * 2.0, -448.0, 448.0)).to(torch.float8_e4m3fn)
    # one code apart at most, and that only where the sum lies next to a rounding boundary: the matrix instruction cuts products off at 2^-13
    # of the largest of eight, a code is 2^-4 .. 2^-3 of its value wide, so fewer than one in a hundred.  Codes run as signed magnitudes
    code = lambda t: torch.where(t.view(torch.uint8) < 128, t.view(torch.uint8).int(), 128 - t.view(torch.uint8).int())
    diff = (code(dy[..., :cout].cpu().contiguous().view(torch.float8_e4m3fn)) - code(want)).abs()
    assert int(diff.max()) <= 1 and float((diff > 0).float().mean()) < 0.01, (int(diff.max()), float((diff > 0).float().mean()))
    assert bool((dy[..., cout:] == 0x55).all())


@pytest.mark.parametrize("n,h,w,cin,cout,k,stride,res,xe,ye,mode", [
    (33, 40, 41, 384, 408, 1, 1, nn.RES_BEFORE_ACT, 0, 8, 0),      # half a vector at the end of the last tile's second block
    (9, 41, 39, 256, 88, 1, 1, nn.RES_AFTER_ACT, 128, 0, 0),       # in the upper half of a block
    (60, 40, 41, 96, 104, 1, 1, nn.RES_AFTER_ACT, 0, 24, 2),       # one step, part of it
    (21, 56, 55, 64, 648, 1, 1, nn.RES_NONE, 0, 0, 2),             # one step, several channel tiles
    (23, 56, 57, 128, 1024, 1, 1, nn.RES_AFTER_ACT, 0, 0, 0),      # the same with whole vectors
    (209, 34, 38, 256, 24, 1, 1, nn.RES_NONE, 0, 0, 0),            # less than 32 channels
    (25, 61, 63, 128, 152, 3, 2, nn.RES_BEFORE_ACT, 0, 0, 1),
])
def test_flow_fp8_half_vectors_and_single_steps(octo, n, h, w, cin, cout, k, stride, res, xe, ye, mode):
    test_flow_fp8(octo, n, h, w, cin, cout, k, stride, res, xe, ye, mode)


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("case", [
    (40, 41, 256, 96, 128, 9),         # the second layer begins inside a channel tile, whatever its width, and ends inside one
    (40, 40, 128, 32, 64, 20),         # at the first block of 32 channels
    (20, 20, 520, 160, 352, 16),       # a reduction that ends inside a step
])
def test_two_layers_in_one_flowing_launch(octo, dtype, case):
    """Two 1x1 layers of one input, computed by one launch that writes each to a tensor of its own: both against the oracle and, bit for
    bit, against the launches of their own."""
    h, w, cin, c1, c2, n = case
    B = zoo._Builder("t", dtype, h, w, "classifier", np.random.default_rng(63))
    B.ch = [16]
    B.m.in_c = 16
    x = B.conv(0, cin, 1, 1, act=zoo.ACT_SILU)
    a, b = B.conv(x, c1, 1, 1, act=zoo.ACT_SILU), B.conv(x, c2, 1, 1, act=zoo.ACT_SILU)
    B.m.outputs = [B.fc(B.gap(B.cat([B.conv(a, c1, 1, 1), b])), 10)]
    B.m.batch_size = n
    v = zoo.round_to_dtype(np.random.default_rng(64).uniform(-1, 1, (n, h, w, 16)).astype(np.float32), dtype)
    got, kids = {}, {}
    for keep in (1, 2):
        P = octo.Pipeline(zoo.PipelineSpec("t", [small_root(dtype), B.m], [], 200.0, 32, 32, 1, 1), keep_all_tensors=keep)
        P.run_model_on(1, octo.to_device(v, dtype))
        got[keep], kids[keep] = [P.get_tensor(1, t, n) for t in (a, b)], [int(k) for k in P.layer_info(1)[1]][1:3]
        P.close()
    assert kids[2][0] // 100000000 == 12 and kids[2][1] == 0, kids
    ref = nn.run_model(B.m, v, keep_all=True)
    for j, t in enumerate((a, b)):
        assert rel_err(got[2][j], ref[t]) <= TOL[dtype], t
        assert np.array_equal(got[2][j], got[1][j]), t


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_flow_with_the_item_count_on_the_device(octo, dtype):
    """1x1 and strided layers of a downstream model: the grid is sized for 480 items, and batches bring hundreds, a few dozen and one of
    them, so that some or nearly all workgroups find no tile.  Every tensor of some ROIs against the oracle on the GPU's own crops; what
    the larger batch left beyond the smaller one's items is untouched."""
    import torch
    det = zoo.traffic_cascade(dtype).models[0]
    det.batch_size = 4
    B = zoo._Builder("child", dtype, 56, 56, "classifier", np.random.default_rng(65))
    a = B.conv(0, 64, 3, 2, act=zoo.ACT_RELU)
    b = B.conv(B.conv(a, 128, 3, 2, act=zoo.ACT_SILU), 256, 1, 1, act=zoo.ACT_RELU)      # a tap per step; nothing but channels
    c = B.conv(b, 104, 1, 1, act=zoo.ACT_SILU)
    d = B.conv(c, 192, 3, 2, act=zoo.ACT_RELU)                                           # steps across taps
    B.m.outputs = [B.fc(B.gap(d), 10)]
    B.m.batch_size = 480
    spec = zoo.PipelineSpec("items", [det, B.m], [zoo.Edge(0, 1)], 1000.0, 540, 960, 4, 120)
    rng = np.random.default_rng(zoo.SEED0 + 93)
    geo = octo.letterbox_geometry(540, 960, det.in_h, det.in_w)
    scenes = [synth.make_scene(rng, 4, 540, 960, counts, 16, 200, log_uniform=True) for counts in ([120] * 4, [5, 0, 17, 9], [0, 1, 0, 0])]
    n_t = len(B.m.layers)
    P = octo.Pipeline(spec, keep_all_tensors=1)
    P.set_expected_items(1, 480)                         # none of these layers is split, whatever the batch brings
    before, modes = None, set()
    for k, sc in enumerate(scenes):
        heads = [octo.to_device(v, dtype) for v in synth.planted_heads(rng, det, sc, 540, 960, geo)]
        for l, v in enumerate(heads):
            P.set_head(0, l, v)
        P.submit([torch.from_numpy(f).cuda() for f in sc.frames])
        P.run()
        P.collect()
        n = len(P.get_rois(0))
        assert (n > 200, 20 < n < 60, 1 <= n < 5)[k], n
        at = sorted({0, n // 2, n - 1})
        got = [np.concatenate([P.get_tensor(1, t, 1, first=i) for i in at]) for t in range(n_t + 1)]
        beyond = [np.concatenate([P.get_tensor(1, t, 1, first=i) for i in (60, 120, 199)]) for t in range(n_t + 1)]
        ref = nn.run_model(B.m, got[0], keep_all=True)
        for t in range(1, n_t + 1):
            assert rel_err(got[t].reshape(ref[t].shape), ref[t]) <= TOL[dtype], (k, t)
            if before is not None:
                assert np.array_equal(beyond[t], before[t]), (k, t)
        before = beyond
        modes |= {int(v) // 10000000 for v in P.layer_info(1)[1]}
    P.close()
    assert {120, 121, 122} <= modes, modes
