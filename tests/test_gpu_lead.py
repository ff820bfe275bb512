"""The entry of a cross-stage block in one launch (lead_kernel): pixel counts that are no multiple of a tile, fewer than one, several tiles per workgroup, both channel counts and
input widths, the first layer's output with and without other readers; against the oracle and against the layers' own launches."""
import numpy as np
import pytest

import bench
from oracle import nn
from paper_2502_01277_amd import zoo
from helpers import TOL, rel_err, small_root


def _is_lead(kid):
    return kid // 10**7 == 212


def _model(dtype, h, w, n, cin, c, shortcut, act=zoo.ACT_SILU, swap=False):
    B = zoo._Builder("t", dtype, h, w, "classifier", np.random.default_rng(61))
    B.ch = [cin]
    B.m.in_c = cin
    a, b = B.conv(0, c, 1, act=act), B.conv(0, c, 1, act=act)
    d = B.conv(b if swap else a, c, 1, act=act)
    e = B.conv(d, c, 3, act=act, res=a if shortcut else None, res_mode=zoo.RES_AFTER_ACT)
    f = B.cat([e, b])
    B.m.outputs = [B.fc(B.gap(f), 10)]
    B.m.batch_size = n
    return B.m, a, b, d, f


def _run(octo, m, dtype, x, keep, tensors, n):
    P = octo.Pipeline(zoo.PipelineSpec("t", [small_root(dtype), m], [], 200.0, 32, 32, 1, 1), keep_all_tensors=keep)
    P.run_model_on(1, octo.to_device(x, dtype))
    got = [int(q) for q in P.layer_info(1)[1]], [P.get_tensor(1, t, n) for t in tensors] if keep else None, P.get_tensor(1, m.outputs[0], n)
    P.close()
    return got


FORMS = [(dtype, cin, c, *size) for dtype in ("bf16", "f16") for cin, c in ((128, 64), (256, 64), (256, 128))
         for size in ((1, 3, 5, True), (2, 9, 17, False), (1, 16, 16, True), (5, 37, 89, True))]
FORMS += [("bf16", cin, 64, 9, 121, 123, False) for cin in (128, 256)]      # tiles of 64 pixels, which 64 channels have


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,cin,c,n,h,w,shortcut", FORMS)
def test_parity(octo, dtype, cin, c, n, h, w, shortcut):
    taken = c == 64 or n * h * w >= 64 * octo.device_cu_count()
    m, a, b, d, f = _model(dtype, h, w, n, cin, c, shortcut)
    x = zoo.round_to_dtype(np.random.default_rng(62).uniform(-1, 1, (n, h, w, cin)).astype(np.float32), dtype)
    some = sorted({0, n - 1})
    refs = nn.run_model(m, x[some], keep_all=True)
    want = [a, b, d, f]
    one, two, three = (_run(octo, m, dtype, x, keep, want, n) for keep in (1, 2, 0))    # layers on their own; fused with every buffer kept; fused
    assert not any(map(_is_lead, one[0])) and one[0][d - 1]
    for got in (two, three):
        assert _is_lead(got[0][a - 1]) == taken and not got[0][b - 1] and bool(got[0][d - 1]) != taken, got[0]
    for k, t in enumerate(want):
        for got in (one, two):
            assert rel_err(got[1][k][some], refs[t]) <= TOL[dtype], t
        # the same roundings at the same places; the order of a sum now and then moves a value to its neighbour
        step = {"bf16": 2.0 ** -7, "f16": 2.0 ** -10}[dtype] * np.maximum(1.0, np.abs(one[1][k]))
        q = np.abs(two[1][k] - one[1][k])
        assert (q <= 3 * step).all() and (q > step / 2).mean() < 0.05, (t, (q / step).max(), (q > step / 2).mean())
    assert np.array_equal(two[2], three[2])


@pytest.mark.gpu
@pytest.mark.parametrize("change", [dict(swap=True), dict(act=zoo.ACT_RELU), dict(c=96), dict(cin=192), dict(cin=512, c=128)])
def test_other_entries_keep_their_launches(octo, change):
    m, a, b, d, f = _model("bf16", 11, 13, 2, **dict(dict(cin=128, c=64, shortcut=True), **change))
    x = zoo.round_to_dtype(np.random.default_rng(63).uniform(-1, 1, (2, 11, 13, m.in_c)).astype(np.float32), "bf16")
    kids, got, _ = _run(octo, m, "bf16", x, 2, [d, f], 2)
    assert not any(map(_is_lead, kids)) and kids[a - 1] and kids[d - 1], kids
    refs = nn.run_model(m, x, keep_all=True)
    assert all(rel_err(g, refs[t]) <= TOL["bf16"] for g, t in zip(got, (d, f)))


def test_its_name():
    assert bench.conv_name(2122064256, "bf16") == "octo::lead_kernel<__bf16, 64, 8, 2>"
