"""A cross-stage block of 32 channels in one launch (block_kernel): maps that are no multiple of a tile, smaller than one, several tiles per workgroup, with and without the
shortcut; against the oracle and against the layers' own launches."""
import numpy as np
import pytest

import bench
from oracle import nn
from paper_2502_01277_amd import zoo
from helpers import TOL, rel_err, small_root

BLOCK = 2110000000


def _model(dtype, h, w, n, shortcut=True, swap=False, width=32, again=False):
    B = zoo._Builder("t", dtype, h, w, "classifier", np.random.default_rng(51))
    B.ch = [16]
    B.m.in_c = 16
    a, b = B.conv(0, width, 1, act=zoo.ACT_SILU), B.conv(0, width, 1, act=zoo.ACT_SILU)
    c = B.conv(a, width, 1, act=zoo.ACT_SILU)
    d = B.conv(c, width, 3, act=zoo.ACT_SILU, res=a if shortcut else None, res_mode=zoo.RES_AFTER_ACT)
    f = B.conv(B.cat([b, d] if swap else [d, b]), 2 * width, 1, act=zoo.ACT_SILU)
    if again:
        f = B.conv(B.cat([f, d]), 40, 1, act=zoo.ACT_SILU)
    B.m.outputs = [B.fc(B.gap(f), 10)]
    B.m.batch_size = n
    return B.m, c, f


def _run(octo, m, dtype, x, keep, t, n):
    P = octo.Pipeline(zoo.PipelineSpec("t", [small_root(dtype), m], [], 200.0, 32, 32, 1, 1), keep_all_tensors=keep)
    P.run_model_on(1, octo.to_device(x, dtype))
    got = [int(q) for q in P.layer_info(1)[1]], P.get_tensor(1, t, n) if keep else None, P.get_tensor(1, m.outputs[0], n)
    P.close()
    return got


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("n,h,w,shortcut", [(1, 16, 32, True), (2, 9, 17, True), (3, 8, 33, False), (4, 1, 5, True), (2, 47, 15, False), (90, 40, 41, True)])
def test_parity(octo, dtype, n, h, w, shortcut):
    m, c, f = _model(dtype, h, w, n, shortcut)
    x = zoo.round_to_dtype(np.random.default_rng(52).uniform(-1, 1, (n, h, w, 16)).astype(np.float32), dtype)
    some = sorted({0, n // 2, n - 1})
    ref = nn.run_model(m, x[some], keep_all=True)[f]
    one, two, three = (_run(octo, m, dtype, x, keep, f, n) for keep in (1, 2, 0))       # layers on their own; fused with every buffer kept; fused
    assert one[0][c - 1] // 10**7 != 211 and one[0][f - 1]
    for got in (two, three):
        assert got[0][c - 1] == BLOCK + (not shortcut) and not any(got[0][c:f]), got[0]
    for got in (one, two):
        assert rel_err(got[1][some], ref) <= TOL[dtype]
    # the same roundings at the same places; sums that start from the bias now and then move a value to its neighbour
    step = {"bf16": 2.0 ** -7, "f16": 2.0 ** -10}[dtype] * np.maximum(1.0, np.abs(one[1]))
    d = np.abs(two[1] - one[1])
    assert (d <= 3 * step).all() and (d > step / 2).mean() < 0.05, ((d / step).max(), (d > step / 2).mean())
    assert np.array_equal(two[2], three[2])


@pytest.mark.gpu
@pytest.mark.parametrize("change", [dict(swap=True), dict(width=48), dict(again=True)])
def test_other_blocks_keep_their_launches(octo, change):
    m, c, f = _model("bf16", 20, 24, 2, **change)
    x = zoo.round_to_dtype(np.random.default_rng(53).uniform(-1, 1, (2, 20, 24, 16)).astype(np.float32), "bf16")
    kids, got, _ = _run(octo, m, "bf16", x, 2, f, 2)
    assert not any(k // 10**7 == 211 for k in kids) and kids[c - 1] and kids[f - 1], kids
    assert rel_err(got, nn.run_model(m, x, keep_all=True)[f]) <= TOL["bf16"]


@pytest.mark.gpu
@pytest.mark.parametrize("shortcut", [True, False])
def test_with_every_buffer_kept_the_tensors_inside_are_written(octo, shortcut):
    m, c, f = _model("f16", 19, 23, 2, shortcut)
    xs = [zoo.round_to_dtype(np.random.default_rng(seed).uniform(-1, 1, (2, 19, 23, 16)).astype(np.float32), "f16") for seed in (54, 55)]
    inside = (c, c + 1, c + 2)
    got = {}
    for keep in (2, 1):                                  # (the fused form first: its buffers have nothing of the other's)
        P = octo.Pipeline(zoo.PipelineSpec("t", [small_root("f16"), m], [], 200.0, 32, 32, 1, 1), keep_all_tensors=keep)
        got[keep] = []
        for x in xs:
            P.run_model_on(1, octo.to_device(x, "f16"))
            kids = [int(q) for q in P.layer_info(1)[1]]
            assert (kids[c - 1] == BLOCK + (not shortcut) and not any(kids[c:f])) == (keep == 2), kids
            got[keep] += [P.get_tensor(1, t, 2) for t in inside]
        P.close()
    assert f == c + 3 and all(np.array_equal(a, b) for a, b in zip(got[1], got[2]))


def test_its_name():
    assert bench.conv_name(BLOCK, "bf16") == "octo::block_kernel<__bf16, true>"
    assert bench.conv_name(BLOCK + 1, "f16") == "octo::block_kernel<_Float16, false>"
