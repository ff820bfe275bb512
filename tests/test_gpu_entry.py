"""The first layers of a detector in one launch (entry_kernel): maps that are no multiple of a tile, smaller than one, several tiles per workgroup, a channel slice as one
destination; against the oracle layer by layer, and against the layers' own launches."""
import numpy as np
import pytest

import bench
from oracle import nn
from paper_2502_01277_amd import zoo
from helpers import TOL, rel_err, small_root


def _model(dtype, h, w, n, c0=32, act=zoo.ACT_SILU, first=6):
    B = zoo._Builder("t", dtype, h, w, "classifier", np.random.default_rng(41))
    B.m.in_c = 3
    x = B.conv(B.conv(0, c0, first, 2, 2, act=act), 2 * c0, 3, 2, act=zoo.ACT_SILU)
    a, b = B.conv(x, c0, 1, act=zoo.ACT_SILU), B.conv(x, c0, 1, act=zoo.ACT_SILU)
    c = B.conv(a, 40, 3, 1, act=zoo.ACT_SILU)
    B.m.outputs = [B.fc(B.gap(B.cat([c, b])), 10)]
    B.m.batch_size = n
    return B.m


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("n,h,w", [(1, 64, 64), (2, 70, 102), (3, 38, 130), (4, 2, 6), (2, 33, 34), (1, 31, 400), (150, 60, 66)])
def test_parity(octo, dtype, n, h, w):
    m = _model(dtype, h, w, n)
    x = zoo.round_to_dtype(np.random.default_rng(42).uniform(0, 1, (n, h, w, 3)).astype(np.float32), dtype)
    some = sorted({0, n // 2, n - 1})
    ref = nn.run_model(m, x[some], keep_all=True)
    got = {}
    for keep in (1, 2, 0):                               # every layer on its own; fused, with every buffer kept; fused
        P = octo.Pipeline(zoo.PipelineSpec("t", [small_root(dtype), m], [], 200.0, 32, 32, 1, 1), keep_all_tensors=keep)
        P.run_model_on(1, octo.to_device(x, dtype))
        kids = [int(q) for q in P.layer_info(1)[1][:4]]
        assert (kids == [2100000000, 0, 0, 0]) == (keep != 1), kids
        got[keep] = [P.get_tensor(1, t, n) for t in ((3, 4) if keep else ())] + [P.get_tensor(1, m.outputs[0], n)]
        P.close()
    for k in (1, 2):
        for j, t in enumerate((3, 4)):
            assert rel_err(got[k][j][some], ref[t]) <= TOL[dtype], (k, t)
    # the same roundings at the same places; what differs are sums of at most 288 products in another order, which now and then move a value to its neighbour
    for j in (0, 1):
        step = {"bf16": 2.0 ** -7, "f16": 2.0 ** -10}[dtype] * np.maximum(1.0, np.abs(got[1][j]))
        d = np.abs(got[2][j] - got[1][j])
        assert (d <= 3 * step).all() and (d > step / 2).mean() < 0.05, ((d / step).max(), (d > step / 2).mean())
    assert np.array_equal(got[0][0], got[2][2])


@pytest.mark.gpu
@pytest.mark.parametrize("change", [dict(c0=48), dict(act=zoo.ACT_RELU), dict(first=5)])
def test_other_first_layers_keep_their_launches(octo, change):
    m = _model("bf16", 40, 48, 2, **change)
    P = octo.Pipeline(zoo.PipelineSpec("t", [small_root("bf16"), m], [], 200.0, 32, 32, 1, 1), keep_all_tensors=2)
    x = zoo.round_to_dtype(np.random.default_rng(42).uniform(0, 1, (2, 40, 48, 3)).astype(np.float32), "bf16")
    P.run_model_on(1, octo.to_device(x, "bf16"))
    kids = [int(q) for q in P.layer_info(1)[1][:4]]
    assert 2100000000 not in kids and kids[0] and kids[1] and kids[2], kids
    ref = nn.run_model(m, x, keep_all=True)
    for t in (3, 4):
        assert rel_err(P.get_tensor(1, t, 2), ref[t]) <= TOL["bf16"]
    P.close()


@pytest.mark.gpu
def test_with_every_buffer_kept_the_tensors_inside_are_written(octo):
    m = _model("bf16", 70, 102, 2)
    xs = [zoo.round_to_dtype(np.random.default_rng(seed).uniform(0, 1, (2, 70, 102, 3)).astype(np.float32), "bf16") for seed in (43, 44)]
    got = {}
    for keep in (2, 1):                                  # (the fused form first: its buffers have nothing of the other's)
        P = octo.Pipeline(zoo.PipelineSpec("t", [small_root("bf16"), m], [], 200.0, 32, 32, 1, 1), keep_all_tensors=keep)
        got[keep] = []
        for x in xs:
            P.run_model_on(1, octo.to_device(x, "bf16"))
            assert (int(P.layer_info(1)[1][0]) == 2100000000) == (keep == 2)
            got[keep] += [P.get_tensor(1, t, 2) for t in (1, 2)]
        P.close()
    assert all(np.array_equal(a, b) for a, b in zip(got[1], got[2]))


def test_its_name():
    assert bench.conv_name(2100000000, "f16") == "octo::entry_kernel<_Float16>"
