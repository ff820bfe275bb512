"""The 3x3 kernel with the input patch in LDS at its edges: widths that no tile divides, tiles that span several images, images of
one row or column's width, channel counts below and over a tile, input channels that do not fill the last slice, residuals, unaligned
and wider output buffers, an item count taken on the device; against the oracle."""
import numpy as np
import pytest

from oracle import nn
from oracle.rounding import round_storage
from paper_2502_01277_amd import synth, zoo
from helpers import TOL, rel_err

pytestmark = pytest.mark.gpu

CASES = [
    # (n, h, w, cin, cout, act, res_mode, x_extra, y_extra, pixel-tile digit, channel tile, channels in LDS)
    (3, 57, 83, 48, 64, nn.ACT_SILU, nn.RES_NONE, 16, 0, 2, 64, 128),              # 64 x 64 tiles; ragged columns, 3/4 of a slice
    (7, 14, 14, 256, 256, nn.ACT_RELU, nn.RES_BEFORE_ACT, 0, 0, None, 0, 0),       # too few tiles: split-K
    (21, 14, 14, 256, 256, nn.ACT_RELU, nn.RES_BEFORE_ACT, 0, 8, 2, 64, 128),      # 64 x 64 tiles across images
    (10, 14, 14, 256, 256, nn.ACT_RELU, nn.RES_NONE, 0, 0, None, 0, 0),            # either side of the line: 0.24 tiles per compute unit
    (11, 14, 14, 256, 256, nn.ACT_RELU, nn.RES_NONE, 0, 0, 2, 64, 128),            # 0.26
    (25, 7, 7, 512, 512, nn.ACT_RELU, nn.RES_NONE, 0, 0, None, 0, 0),              # 0.30, a long reduction
    (10, 28, 28, 96, 96, nn.ACT_SILU, nn.RES_AFTER_ACT, 0, 0, None, 0, 0),         # 0.48, half of the last slice of 64 channels
    (11, 28, 28, 96, 96, nn.ACT_SILU, nn.RES_AFTER_ACT, 0, 0, 0, 96, 64),          # 0.53
    (10, 40, 40, 72, 72, nn.ACT_SILU, nn.RES_NONE, 0, 0, None, 0, 0),              # 0.98, 8 of the last 32 channels
    (11, 40, 40, 72, 72, nn.ACT_SILU, nn.RES_NONE, 0, 0, 0, 96, 64),               # 1.07
    (61, 14, 30, 192, 136, nn.ACT_SILU, nn.RES_AFTER_ACT, 0, 0, 0, 64, 128),       # slices of 128 bytes, 8 of the last 64 channels
    (90, 14, 14, 248, 96, nn.ACT_RELU, nn.RES_BEFORE_ACT, 0, 0, 3, 64, 128),       # patch of five passes, 8 of the last slice
    (5, 80, 81, 64, 64, nn.ACT_RELU, nn.RES_BEFORE_ACT, 64, 64, 0, 64, 64),        # one slice of each buffer, columns 41 + 40
    (400, 3, 37, 56, 100, nn.ACT_SILU, nn.RES_AFTER_ACT, 0, 1, 0, 64, 64),         # unaligned output, 4 of the last 8 channels
    (8, 83, 80, 32, 32, nn.ACT_SILU, nn.RES_AFTER_ACT, 0, 0, 0, 32, 64),           # 32-channel tiles
    (17, 112, 112, 32, 32, nn.ACT_RELU, nn.RES_BEFORE_ACT, 32, 0, 5, 32, 32),      # resident weights, 16 x 16 tiles
    (7, 160, 176, 24, 24, nn.ACT_SILU, nn.RES_NONE, 0, 8, 5, 32, 32),              # 8 of the second 16 channels, on both sides
    (60, 30, 60, 32, 64, nn.ACT_SILU, nn.RES_AFTER_ACT, 0, 0, 5, 64, 32),          # 64 output channels over 32 input channels
    (65, 56, 56, 40, 56, nn.ACT_NONE, nn.RES_AFTER_ACT, 8, 8, 5, 64, 48),          # 4 x 28 tiles, half of the third 16 channels
    (130, 48, 32, 64, 64, nn.ACT_RELU, nn.RES_BEFORE_ACT, 0, 64, 5, 64, 64),       # 4 x 32 tiles
    (5400, 6, 7, 64, 64, nn.ACT_SILU, nn.RES_NONE, 0, 0, 0, 64, 64),               # no tile divides the image
    (3, 160, 111, 96, 96, nn.ACT_SILU, nn.RES_AFTER_ACT, 0, 0, 0, 96, 64),         # 96-channel tiles
    (12, 160, 144, 96, 88, nn.ACT_NONE, nn.RES_NONE, 0, 8, 1, 96, 64),             # 96 channels x 256 pixels
    (650, 28, 28, 96, 128, nn.ACT_RELU, nn.RES_BEFORE_ACT, 0, 0, 1, 64, 64),       # 64 channels x 256 pixels
    (33000, 1, 7, 64, 40, nn.ACT_RELU, nn.RES_NONE, 0, 0, 0, 64, 64),              # one-row images: every tap row but one is outside
]


def reference(x, wt, bias, res, act, res_mode):
    n, h, w, cin = x.shape
    xp = np.zeros((n, h + 2, w + 2, cin), np.float32)
    xp[:, 1:-1, 1:-1] = x
    y = np.zeros((n * h * w, wt.shape[0]), np.float32)
    for r in range(3):
        for s in range(3):
            y += np.ascontiguousarray(xp[:, r:r + h, s:s + w]).reshape(-1, cin) @ np.ascontiguousarray(wt[:, r, s].T)
    y = (y + bias).reshape(n, h, w, -1)
    if res_mode == nn.RES_BEFORE_ACT:
        return nn.activation(y + res, act)
    return nn.activation(y, act) + (res if res_mode else 0.0)


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("case", CASES)
def test_patch_3x3_parity(octo, dtype, case):
    import torch
    n, h, w, cin, cout, act, res_mode, xe, ye, q, bc, chan = case
    rng = np.random.default_rng(43)
    x = zoo.round_to_dtype(rng.uniform(-1, 1, (n, h, w, cin)).astype(np.float32), dtype)
    wt = zoo.round_to_dtype((rng.standard_normal((cout, 3, 3, cin)) / np.sqrt(9 * cin)).astype(np.float32), dtype)
    bias = rng.uniform(-0.1, 0.1, cout).astype(np.float32)
    layer = octo.ConvOp(synth.to_storage(wt, dtype), bias, dtype, 1, 1, act)
    res = zoo.round_to_dtype(rng.uniform(-1, 1, (n, h, w, cout)).astype(np.float32), dtype) if res_mode else None
    dx = torch.full((n, h, w, cin + xe), 5.0, dtype=octo.torch_dtype(dtype), device="cuda")
    dx[..., :cin] = octo.to_device(x, dtype)
    dy = torch.full((n, h, w, cout + ye), -7.0, dtype=octo.torch_dtype(dtype), device="cuda")
    kid = octo.op_conv(layer, dx[..., :cin], dy[..., :cout], octo.to_device(res, dtype) if res_mode else None, res_mode)
    torch.cuda.synchronize()
    family = {1400000000, 1700000000, 1800000000}
    assert (kid // 100000000 * 100000000 in family) == (q is not None), kid
    if q is not None:
        assert kid % 100000000 == q * 1000000 + bc * 1000 + chan, kid
    assert rel_err(dy[..., :cout].float().cpu().numpy(), round_storage(reference(x, wt, bias, res, act, res_mode), dtype)) <= TOL[dtype]
    assert (dy[..., cout:].float().cpu().numpy() == -7.0).all()


@pytest.mark.parametrize("n,h,w,cin,cout,res,bc", [
    (90, 14, 14, 192, 136, True, 64),          # three slices, 8 of the last 64 channels
    (20, 41, 37, 112, 64, False, 64),          # three quarters of the second slice, ragged columns
    (1100, 14, 14, 64, 256, True, 128),        # one slice, 128-channel tiles
])
def test_patch_3x3_fp8(octo, n, h, w, cin, cout, res, bc):
    import torch
    rng = np.random.default_rng(47)
    f8 = lambda shape, s: torch.from_numpy((rng.standard_normal(shape) * s).astype(np.float32)).to(torch.float8_e4m3fn)
    x, wt = f8((n, h, w, cin), 1.0), f8((cout, 3, 3, cin), 2.0)
    r = f8((n, h, w, cout), 1.0) if res else None
    scale, bias = (0.02 + 0.01 * rng.random(cout)).astype(np.float32), rng.uniform(-0.1, 0.1, cout).astype(np.float32)
    layer = octo.ConvOp(wt.view(torch.uint8).numpy(), bias, "f8", 1, 1, nn.ACT_RELU, scale=scale)
    y = torch.zeros((n, h, w, cout), dtype=torch.uint8, device="cuda")
    kid = octo.op_conv(layer, x.view(torch.uint8).cuda(), y, r.view(torch.uint8).cuda() if res else None, nn.RES_BEFORE_ACT if res else 0, res_scale=0.5, y_inv_scale=2.0)
    torch.cuda.synchronize()
    assert kid // 100000000 in (14, 17, 18) and kid % 100000000 == bc * 1000 + 128, kid
    acc = reference(x.float().numpy(), wt.float().numpy(), np.zeros(cout, np.float32), None, nn.ACT_NONE, nn.RES_NONE)
    want = np.maximum(acc * scale + bias + (0.5 * r.float().numpy() if res else 0.0), 0.0) * 2.0
    want = torch.from_numpy(np.minimum(want, 448.0)).to(torch.float8_e4m3fn)
    got = y.cpu().view(torch.float8_e4m3fn)
    # one code apart at most, and that only where the fp32 sum lies next to a rounding boundary
    diff = (got.view(torch.uint8).int() - want.view(torch.uint8).int()).abs()
    assert int(diff.max()) <= 1 and float((diff != 0).float().mean()) < 1e-3


# Several tiles per workgroup, so that one tile's K loop runs into the next one's: large tiles, outputs and residuals in whole vectors
# and in pieces.
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("case", [
    (860, 14, 14, 136, 120, nn.ACT_RELU, nn.RES_BEFORE_ACT, 8, 8, 1, 128, 64),     # 128 x 256, a quarter of the last slice, 8 channels short
    (860, 14, 14, 128, 128, nn.ACT_SILU, nn.RES_AFTER_ACT, 0, 1, 1, 128, 64),      # the same, output rows of odd pitch
    (860, 14, 14, 128, 124, nn.ACT_NONE, nn.RES_NONE, 0, 0, 1, 128, 64),           # half a vector at the end of a row
    (14, 80, 80, 192, 192, nn.ACT_SILU, nn.RES_AFTER_ACT, 0, 0, 1, 96, 64),        # 96 x 256 where 128 channels would pad
    (1300, 3, 37, 56, 100, nn.ACT_RELU, nn.RES_BEFORE_ACT, 0, 1, 0, 64, 64),       # 64 x 128 in pieces
])
def test_patch_3x3_tile_after_tile(octo, dtype, case):
    test_patch_3x3_parity(octo, dtype, case)


@pytest.mark.parametrize("n,h,w,cin,cout,res", [(430, 14, 14, 128, 256, True), (420, 14, 14, 144, 248, True), (860, 14, 14, 128, 128, False)])
def test_patch_3x3_fp8_large_tiles(octo, n, h, w, cin, cout, res):
    test_patch_3x3_fp8(octo, n, h, w, cin, cout, res, 1128)      # 128 channels x 256 pixels (digit 1); 248 channels leave in pieces of 8


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_patch_3x3_with_the_item_count_on_the_device(octo, dtype):
    """3x3 layers of a downstream model, whose item count stays on the device: a batch with a few hundred ROIs, then one with a few
    dozen, on kernels chosen for 400, 60 and 3 items.  Every tensor of the first, last and some other ROIs against the oracle on the
    GPU's own crops; what the larger batch left beyond the smaller one's items is untouched."""
    import torch
    det = zoo.traffic_cascade(dtype).models[0]
    det.batch_size = 4
    B = zoo._Builder("child", dtype, 56, 56, "classifier", np.random.default_rng(17))
    a = B.conv(B.conv(0, 64, 3, 2, act=zoo.ACT_RELU), 64, 3, act=zoo.ACT_NONE)
    a = B.conv(a, 64, 3, act=zoo.ACT_RELU, res=1, res_mode=zoo.RES_BEFORE_ACT)
    b = B.conv(B.conv(a, 96, 3, act=zoo.ACT_SILU), 192, 3, 2, act=zoo.ACT_RELU)
    c = B.conv(B.conv(b, 192, 3, act=zoo.ACT_RELU), 40, 3, act=zoo.ACT_SILU)
    B.m.outputs = [B.fc(B.gap(c), 10)]
    B.m.batch_size = 400
    spec = zoo.PipelineSpec("items", [det, B.m], [zoo.Edge(0, 1)], 1000.0, 540, 960, 4, 100)
    rng = np.random.default_rng(zoo.SEED0 + 91)
    geo = octo.letterbox_geometry(540, 960, det.in_h, det.in_w)
    scenes = [synth.make_scene(rng, 4, 540, 960, counts, 16, 200, log_uniform=True) for counts in ([120] * 4, [5, 0, 17, 9])]
    heads = [[octo.to_device(v, dtype) for v in synth.planted_heads(rng, det, s, 540, 960, geo)] for s in scenes]
    frames = [[torch.from_numpy(f).cuda() for f in s.frames] for s in scenes]
    n_t = len(B.m.layers)
    P = octo.Pipeline(spec, keep_all_tensors=1)
    families, refs = set(), {}
    for expected in (400, 60, 3):
        P.set_expected_items(1, expected)
        before = None
        for k in (0, 1):
            for l, v in enumerate(heads[k]):
                P.set_head(0, l, v)
            P.submit(frames[k])
            P.run()
            P.collect()
            n = len(P.get_rois(0))
            assert n > 200 if k == 0 else 20 < n < 60
            at = [0, n // 2, n - 1]
            got = [np.concatenate([P.get_tensor(1, t, 1, first=i) for i in at]) for t in range(n_t + 1)]
            beyond = [np.concatenate([P.get_tensor(1, t, 1, first=i) for i in (60, 120, 199)]) for t in range(n_t + 1)]
            if k not in refs:
                refs[k] = nn.run_model(B.m, got[0], keep_all=True)
            for t in range(1, n_t + 1):
                assert rel_err(got[t].reshape(refs[k][t].shape), refs[k][t]) <= TOL[dtype], (expected, k, t)
                if before is not None:
                    assert np.array_equal(beyond[t], before[t]), (expected, t)
            before = beyond
        families |= {int(v) // 100000000 for v in P.layer_info(1)[1][1:7]}
    P.close()
    assert {16, 17, 18} <= families, families             # split-K, patch kernels of more and of up to 64 channels
