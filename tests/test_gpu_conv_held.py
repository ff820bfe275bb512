"""3x3 layers of a model whose whole input patch is held in LDS (conv3x3_held_kernel) at the edges of their tiles: every tile and stride, tiles over several images
and over part of a row, widths and heights that are no multiple of a tile, one to eight slices of channels, residuals, a channel slice as destination, and more
items on the device than the launch was shaped for.  Against sums in 64 bits of the layer's own input, and against the oracle."""
import numpy as np
import pytest
import torch

import bench
from oracle import nn
from paper_2502_01277_amd import synth, zoo
from helpers import TOL, rel_err, small_root

T32, T64, T128 = 2014064032, 2014064064, 2012064128        # stride 1
S32, S64 = 2024064032, 2024064064                          # stride 2

CASES = [
    # (n, h, w, cin, cout, stride, act, res_mode, kernel id)
    (1, 20, 20, 256, 256, 1, zoo.ACT_SILU, zoo.RES_AFTER_ACT, T32),
    (1, 40, 40, 128, 128, 1, zoo.ACT_SILU, zoo.RES_AFTER_ACT, T32),
    (3, 13, 27, 192, 128, 1, zoo.ACT_RELU, zoo.RES_BEFORE_ACT, T32),        # nothing divides
    (2, 4, 4, 512, 64, 1, zoo.ACT_NONE, zoo.RES_NONE, T32),                 # fewer pixels than a tile
    (4, 31, 33, 320, 192, 1, zoo.ACT_SILU, zoo.RES_AFTER_ACT, T64),         # five slices
    (8, 20, 20, 256, 256, 1, zoo.ACT_SILU, zoo.RES_NONE, T64),
    (29, 7, 7, 512, 512, 1, zoo.ACT_RELU, zoo.RES_BEFORE_ACT, T64),         # tiles over several images
    (8, 79, 80, 64, 64, 1, zoo.ACT_SILU, zoo.RES_AFTER_ACT, T128),          # one slice
    (16, 20, 20, 256, 256, 1, zoo.ACT_SILU, zoo.RES_AFTER_ACT, T128),
    (63, 7, 7, 512, 448, 1, zoo.ACT_RELU, zoo.RES_NONE, T128),              # a patch of nearly all of LDS
    (9, 41, 39, 192, 192, 1, zoo.ACT_SILU, zoo.RES_BEFORE_ACT, T128),
    (3, 40, 40, 256, 256, 2, zoo.ACT_SILU, zoo.RES_NONE, S32),
    (11, 14, 13, 512, 256, 2, zoo.ACT_RELU, zoo.RES_NONE, S32),             # an odd width
    (40, 8, 8, 128, 256, 2, zoo.ACT_RELU, zoo.RES_NONE, S32),
    (27, 16, 15, 256, 512, 2, zoo.ACT_SILU, zoo.RES_NONE, S64),
]


def _check(dtype, L, x, y, res, stride, act, res_mode):
    """The layer's output against sums in 64 bits of its own input.  One rounding to storage (half a unit in the last place), and fp32 sums of K products in parts of at most K / 2: with random signs
    far below K / 8 roundings of 2^-24 of the sum of the magnitudes."""
    nchw = lambda t: torch.from_numpy(np.ascontiguousarray(t)).double().permute(0, 3, 1, 2)   # noqa: E731
    conv = lambda a, b: torch.nn.functional.conv2d(a, b, stride=stride, padding=1).permute(0, 2, 3, 1).numpy()   # noqa: E731
    s, mag = conv(nchw(x), nchw(L.weight)) + L.bias, conv(nchw(x).abs(), nchw(L.weight).abs())
    res = res.astype(np.float64) if res_mode else 0.0
    f = {zoo.ACT_SILU: lambda t: t / (1.0 + np.exp(-t)), zoo.ACT_RELU: lambda t: np.maximum(t, 0.0), zoo.ACT_NONE: lambda t: t}[act]
    ref = f(s + res) if res_mode == zoo.RES_BEFORE_ACT else f(s) + res
    half_ulp = {"bf16": 2.0 ** -9, "f16": 2.0 ** -12}[dtype] * 2
    bound = half_ulp * np.abs(ref) + (9 * x.shape[3] / 8 + 16) * 2.0 ** -24 * (mag + np.abs(res) + 1.0)
    err = np.abs(y - ref)
    assert (err <= bound).all(), (err / bound).max()


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("case", CASES)
def test_parity(octo, dtype, case):
    n, h, w, cin, cout, stride, act, res_mode, want = case
    B = zoo._Builder("t", dtype, h, w, "classifier", np.random.default_rng(17))
    B.ch = [16]
    B.m.in_c = 16
    x = B.conv(0, cin, 1, 1, act=zoo.ACT_RELU)
    r = (x if cin == cout else B.conv(0, cout, 1, 1, act=zoo.ACT_NONE)) if res_mode else None
    y = B.conv(x, cout, 3, stride, act=act, res=r, res_mode=res_mode)
    z = B.conv(0, 64, 1, stride, act=zoo.ACT_NONE)
    B.m.outputs = [B.fc(B.gap(B.cat([z, y])), 8)]
    B.m.batch_size = n
    v = zoo.round_to_dtype(np.random.default_rng(18).uniform(-1, 1, (n, h, w, 16)).astype(np.float32), dtype)
    got = {}
    for keep in (1, 0):                                  # every tensor in a buffer of its own; buffers reused
        P = octo.Pipeline(zoo.PipelineSpec("t", [small_root(dtype), B.m], [], 200.0, 32, 32, 1, 1), keep_all_tensors=keep)
        P.run_model_on(1, octo.to_device(v, dtype))
        kid = int(P.layer_info(1)[1][y - 1])
        assert kid == want, kid
        got[keep] = {t: P.get_tensor(1, t, n) for t in ((x, y, B.m.outputs[0]) + ((r,) if r else ()) if keep else (B.m.outputs[0],))}
        P.close()
    assert np.array_equal(got[0][B.m.outputs[0]], got[1][B.m.outputs[0]])
    _check(dtype, B.m.layers[y - 1], got[1][x], got[1][y], got[1][r] if res_mode else None, stride, act, res_mode)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("n,h,w,c,cout,stride,want", [(1, 20, 20, 256, 256, 1, T32), (8, 20, 21, 256, 256, 1, T64), (9, 41, 39, 192, 192, 1, T128), (3, 40, 40, 256, 192, 2, S32),
                                                      (27, 16, 15, 256, 512, 2, S64)])
def test_channel_slices_of_wider_tensors(octo, dtype, n, h, w, c, cout, stride, want):
    """Input, residual and output each in the channels behind others of a concatenation: pitches and first channels of their own."""
    B = zoo._Builder("t", dtype, h, w, "classifier", np.random.default_rng(19))
    B.ch = [16]
    B.m.in_c = 16
    x = B.conv(0, c, 1, 1, act=zoo.ACT_RELU)
    r = B.conv(0, cout, 1, stride, act=zoo.ACT_NONE)
    y = B.conv(x, cout, 3, stride, act=zoo.ACT_SILU, res=r, res_mode=zoo.RES_BEFORE_ACT)
    wide_x = B.cat([B.conv(0, 72, 1, 1, act=zoo.ACT_NONE), x])
    wide_r = B.cat([B.conv(0, 40, 1, stride, act=zoo.ACT_NONE), r])
    wide_y = B.cat([B.conv(0, 24, 1, stride, act=zoo.ACT_NONE), y])
    B.m.outputs = [B.fc(B.gap(B.cat([B.conv(wide_x, 64, 1, stride), B.conv(wide_r, 64, 1), B.conv(wide_y, 64, 1)])), 8)]
    B.m.batch_size = n
    v = zoo.round_to_dtype(np.random.default_rng(20).uniform(-1, 1, (n, h, w, 16)).astype(np.float32), dtype)
    P = octo.Pipeline(zoo.PipelineSpec("t", [small_root(dtype), B.m], [], 200.0, 32, 32, 1, 1), keep_all_tensors=1)
    P.run_model_on(1, octo.to_device(v, dtype))
    assert int(P.layer_info(1)[1][y - 1]) == want
    got = {t: P.get_tensor(1, t, n) for t in (x, r, y, wide_x, wide_r, wide_y)}
    P.close()
    for t, wide, first in ((x, wide_x, 72), (r, wide_r, 40), (y, wide_y, 24)):
        assert np.array_equal(got[t], got[wide][..., first:])
    _check(dtype, B.m.layers[y - 1], got[x], got[y], got[r], stride, zoo.ACT_SILU, zoo.RES_BEFORE_ACT)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_more_items_on_the_device_than_expected(octo, dtype):
    """A downstream model shaped for three items whose batches bring hundreds: workgroups go through several tiles each.  Every tensor of some ROIs against the oracle on
    the GPU's own crops; a small batch leaves the rest of the larger one's results as they are."""
    det = zoo.traffic_cascade(dtype).models[0]
    det.batch_size = 4
    B = zoo._Builder("child", dtype, 32, 32, "classifier", np.random.default_rng(91))
    a = B.conv(0, 128, 3, 2, act=zoo.ACT_RELU)
    b = B.conv(a, 256, 3, 1, act=zoo.ACT_SILU)
    c = B.conv(b, 256, 3, 2, act=zoo.ACT_RELU)
    d = B.conv(c, 512, 3, 1, act=zoo.ACT_SILU)
    e = B.conv(d, 512, 3, 1, act=zoo.ACT_RELU, res=d, res_mode=zoo.RES_BEFORE_ACT)
    B.m.outputs = [B.fc(B.gap(e), 10)]
    B.m.batch_size = 480
    spec = zoo.PipelineSpec("items", [det, B.m], [zoo.Edge(0, 1)], 1000.0, 540, 960, 4, 120)
    rng = np.random.default_rng(92)
    geo = octo.letterbox_geometry(540, 960, det.in_h, det.in_w)
    scenes = [synth.make_scene(rng, 4, 540, 960, counts, 16, 200, log_uniform=True) for counts in ([0, 2, 0, 1], [120] * 4, [120] * 4, [1, 0, 2, 0])]
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
        assert n > 200 if k in (1, 2) else 1 <= n < 5, n
        kids = [int(v) for v in P.layer_info(1)[1]]
        assert all(kids[t - 1] // 10000000 in (201, 202) for t in (b, c, d, e)), kids
        if k == 2:
            assert kids[e - 1] == T64, kids              # the running count chooses among the tiles of one order
        at = sorted({0, n // 2, n - 1})
        got = [np.concatenate([P.get_tensor(1, t, 1, first=i) for i in at]) for t in range(n_t + 1)]
        beyond = [np.concatenate([P.get_tensor(1, t, 1, first=i) for i in (60, 120, 199)]) for t in range(n_t + 1)]
        ref = nn.run_model(B.m, got[0], keep_all=True)
        for t in range(1, n_t + 1):
            assert rel_err(got[t].reshape(ref[t].shape), ref[t]) <= TOL[dtype], (k, t)
            if k == 3:
                assert np.array_equal(beyond[t], before[t]), t
        before = beyond
    P.close()


def test_the_names_of_the_instances():
    for kid, args in ((T32, "2, 1, 4, 1"), (T64, "2, 2, 4, 1"), (T128, "2, 2, 2, 1"), (S32, "2, 1, 4, 2"), (S64, "2, 2, 4, 2")):
        assert bench.conv_name(kid, "bf16") == "octo::conv3x3_held_kernel<__bf16, %s>" % args
