"""First layers (3 channels, stride 2) where a wavefront walks down a strip: edges of strips, segments and channels, with and without the
3x3 / stride-2 max-pool behind them."""
import numpy as np
import pytest

from oracle import nn
from paper_2502_01277_amd import zoo
from helpers import TOL, rel_err, small_root

pytestmark = pytest.mark.gpu


def _tensors(octo, m, x, dtype, keep):
    P = octo.Pipeline(zoo.PipelineSpec("t", [small_root(dtype), m], [], 200.0, 32, 32, 1, 1), keep_all_tensors=keep)
    P.run_model_on(1, octo.to_device(x, dtype))
    n = x.shape[0]
    got = [P.get_tensor(1, t, n) for t in (1, 2)], int(P.layer_info(1)[1][0])
    P.close()
    return got


def _model(dtype, h, w, k, pad, cout, act, n, pool):
    B = zoo._Builder("t", dtype, h, w, "classifier", np.random.default_rng(3))
    B.ch = [3]
    B.m.in_c = 3
    a = B.conv(0, cout, k, 2, pad, act=act)
    a = B.conv(B.maxpool(a, 3, 2, 1) if pool else a, 16, 1, 1)
    B.m.outputs = [B.fc(B.gap(a), 10)]
    B.m.batch_size = n
    return B.m


# widths that end a strip of 64 convolution columns exactly, one short and one over; one row; several segments per strip; channel counts
# that end inside a vector, in a block of 32 and at a block's end
CASES = [(6, 2, 30, 126, 32, 2), (6, 2, 32, 128, 64, 2), (6, 2, 33, 130, 20, 3), (6, 2, 2, 260, 44, 1), (6, 2, 260, 64, 32, 9),
         (3, 1, 31, 128, 32, 2), (3, 1, 64, 130, 12, 5), (7, 3, 33, 126, 64, 2), (7, 3, 40, 130, 36, 3)]


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("act", [zoo.ACT_NONE, zoo.ACT_RELU, zoo.ACT_SILU])
@pytest.mark.parametrize("case", CASES)
def test_strips_segments_and_channels(octo, dtype, act, case):
    k, pad, h, w, cout, n = case
    m = _model(dtype, h, w, k, pad, cout, act, n, False)
    x = zoo.round_to_dtype(np.random.default_rng(31).uniform(-1, 1, (n, h, w, 3)).astype(np.float32), dtype)
    got, kid = _tensors(octo, m, x, dtype, 1)
    assert kid // 10000000 == 190, kid
    assert rel_err(got[0], nn.run_model(m, x, keep_all=True)[1]) <= TOL[dtype]


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("act", [zoo.ACT_NONE, zoo.ACT_RELU, zoo.ACT_SILU])
@pytest.mark.parametrize("h,w,cout,n", [(30, 124, 64, 2), (33, 128, 64, 2), (2, 126, 24, 1), (64, 130, 20, 3), (130, 62, 64, 40)])
def test_pooled_rows_and_columns_and_values_that_are_no_numbers(octo, dtype, act, h, w, cout, n):
    """Fused and separate kernels agree bit for bit, also where windows hold infinities and values that are no numbers: an infinite pixel
    makes its outputs infinite, two of opposite sign make NaN, which bias and activation turn into the activation's least value."""
    m = _model(dtype, h, w, 7, 3, cout, act, n, True)
    x = zoo.round_to_dtype(np.random.default_rng(32).uniform(-1, 1, (n, h, w, 3)).astype(np.float32), dtype)
    if act != zoo.ACT_SILU:
        x[0, h // 2, w // 2, 0], x[0, h // 2, w // 2 + 4, 1], x[-1, 0, -1, 2] = np.inf, -np.inf, np.inf
    one, two = _tensors(octo, m, x, dtype, 1), _tensors(octo, m, x, dtype, 2)
    assert two[1] == 1901064074 and one[1] == 1900064074
    assert np.array_equal(one[0][1], two[0][1])
    clean = np.isfinite(one[0][1]).all(axis=-1)
    assert clean.mean() > 0.5 or n == 1
    if act == zoo.ACT_SILU:
        assert rel_err(two[0][1], nn.run_model(m, x, keep_all=True)[2]) <= TOL[dtype]
