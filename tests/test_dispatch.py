"""The lines between the convolution kernels, on both sides of them, by the ids that launch_conv returns (no GPU: see dispatch.py)."""
import pytest

import dispatch

SPLIT8, SPLIT4, SPLIT4_64 = 1608032032, 1604032032, 1604064032


@pytest.fixture(scope="module")
def ids(tmp_path_factory):
    exe = dispatch.program(tmp_path_factory.mktemp("dispatch"))
    return lambda layers: dispatch.kernel_ids(exe, layers)


def test_fp32_splits_of_eight_stay_splits_of_eight(ids):
    """Layers on which the two sets of estimates differ: sums of eight parts round less than those of four."""
    cases = [(14, 31, 43, 240, 16, 3, 1), (35, 12, 17, 556, 552, 3, 2), (42, 16, 13, 348, 124, 3, 1), (31, 7, 9, 152, 572, 5, 1), (118, 13, 11, 524, 40, 3, 1),
             (98, 14, 14, 84, 20, 5, 1), (19, 7, 8, 60, 472, 5, 1), (1, 112, 147, 272, 28, 3, 1), (2, 80, 119, 508, 48, 5, 1), (1, 80, 59, 680, 240, 3, 1)]
    layers = [dict(zip(("n", "h", "w", "cin", "cout", "k", "stride"), c), dtype="f32") for c in cases]
    assert ids(layers) == [SPLIT8] * len(cases)
    # and where both have four ahead, four it is
    assert ids([dict(dtype="f32", n=30, h=28, w=23, cin=104, cout=9, k=3), dict(dtype="f32", n=1, h=80, w=77, cin=68, cout=44, k=3)]) == [SPLIT4, SPLIT4_64]
