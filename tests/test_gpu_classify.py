"""Global average pool, fully connected layer and label in one launch, at edges of channels, outputs and maps."""
import numpy as np
import pytest

from paper_2502_01277_amd import zoo
from helpers import small_root

pytestmark = pytest.mark.gpu


def _model(dtype, h, w, c, n_out, n):
    B = zoo._Builder("t", dtype, h, w, "classifier", np.random.default_rng(11))
    B.ch = [c]
    B.m.in_c = c
    B.m.outputs = [B.fc(B.gap(0), n_out)]
    B.m.batch_size = n
    return B.m


# one vector of channels and one output; 64 vectors of 16-bit and of fp32 channels and matrices of 16 KB, the most that one launch takes, and
# one row more; as many outputs as it takes, and one more; one vector more; channels that are no whole vectors; more items than workgroups
@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("h,w,c,n_out,n", [(1, 1, 8, 1, 3), (7, 7, 512, 16, 5), (7, 7, 512, 17, 3), (4, 4, 256, 16, 3), (4, 4, 256, 17, 3), (3, 5, 8, 128, 4),
                                           (3, 5, 8, 129, 2), (2, 3, 520, 4, 2), (2, 3, 254, 4, 2), (1, 2, 16, 10, 2100)])
def test_classifier_end(octo, dtype, h, w, c, n_out, n):
    m = _model(dtype, h, w, c, n_out, n)
    x = zoo.round_to_dtype(np.random.default_rng(12).uniform(-1, 1, (n, h, w, c)).astype(np.float32), dtype)
    P = octo.Pipeline(zoo.PipelineSpec("t", [small_root(dtype), m], [], 200.0, 32, 32, 1, 1))
    P.run_model_on(1, octo.to_device(x, dtype))
    mean, logits = np.asarray(P.get_tensor(1, 1, n), np.float64).reshape(n, c), np.asarray(P.get_tensor(1, 2, n), np.float64).reshape(n, n_out)
    P.close()
    exact = np.asarray(x, np.float64).mean((1, 2))
    # the mean: fp32 sums of h w values of at most 1, then one rounding to the type
    assert np.abs(mean - exact).max() <= h * w * 2.0 ** -24 + {"f32": 2.0 ** -24, "f16": 2.0 ** -11, "bf16": 2.0 ** -8}[dtype]
    W = np.asarray(m.layers[1].weight, np.float64).reshape(n_out, c)
    want = mean @ W.T + np.asarray(m.layers[1].bias, np.float64)
    # a logit: no chain of sums is longer than c + 8; products of 16-bit values are exact, those of fp32 within a fused rounding
    bound = (c + 8) * 2.0 ** -24 * (np.abs(mean) @ np.abs(W.T) + np.abs(m.layers[1].bias).max())
    assert (np.abs(logits - want) <= bound).all()
