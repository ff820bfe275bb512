"""Layers whose kernel is another one inside a model than on their own (there a layer's input was written by the launch before): each layer
of the model against the single-layer call on the same input, by default bit for bit, since the kernels between which the place chooses
add in one order; where they do not, within the storage type's bar."""
import numpy as np
import pytest

from oracle import nn
from paper_2502_01277_amd import synth, zoo
from helpers import TOL, rel_err, small_root

# (items, h, w, [(cout, kernel, stride, with residual, family in a model, family alone, same order of sums)]); the first layer comes from 16 channels
CASES = [
    (8, 81, 79, [(128, 1, 1, False, None, None, False), (128, 1, 1, False, 13, 12, True), (256, 1, 1, False, 13, 12, True), (64, 1, 1, False, 13, 12, True)]),
    (8, 160, 161, [(32, 1, 1, False, None, None, False), (64, 3, 2, False, 13, 12, True)]),            # steps across taps
    (4, 81, 79, [(96, 1, 1, False, None, None, False), (120, 1, 1, False, 13, 15, True), (120, 1, 1, True, 13, 15, True), (128, 1, 1, False, 13, 15, True)]),          # steps of part of 64 channels
    (13, 41, 40, [(128, 1, 1, False, None, None, False), (128, 3, 1, False, 20, 17, False), (128, 3, 1, True, 20, 17, False)]),      # the whole patch in LDS : slices of 32 channels
    (13, 41, 40, [(128, 1, 1, False, None, None, False), (120, 3, 1, False, 17, 17, False)]),                                          # slices of 64 : 32 channels
    (8, 161, 160, [(64, 1, 1, False, None, None, False), (64, 1, 1, False, 13, 15, True), (64, 1, 1, True, 13, 15, True), (64, 3, 1, False, 18, 18, False),
                    (32, 1, 1, False, 13, 15, True)]),                          # resident weights alone
    (1, 7, 7, [(1024, 1, 1, False, None, None, False), (512, 1, 1, False, None, None, True)]),                                          # split-K or not, in both
    (1, 14, 14, [(128, 1, 1, False, None, None, False), (256, 3, 2, False, None, None, True)]),
]


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("case", CASES)
def test_layers_in_their_place_and_alone(octo, dtype, case):
    import torch
    n, h, w, layers = case
    B = zoo._Builder("t", dtype, h, w, "classifier", np.random.default_rng(97))
    B.ch = [16]
    B.m.in_c = 16
    x = 0
    for cout, k, stride, res, *_ in layers:
        x = B.conv(x, cout, k, stride, act=zoo.ACT_SILU, res=x if res else None, res_mode=nn.RES_AFTER_ACT)
    B.m.outputs = [B.fc(B.gap(x), 10)]
    B.m.batch_size = n
    v = zoo.round_to_dtype(np.random.default_rng(98).uniform(-1, 1, (n, h, w, 16)).astype(np.float32), dtype)
    P = octo.Pipeline(zoo.PipelineSpec("t", [small_root(dtype), B.m], [], 200.0, 32, 32, 1, 1), keep_all_tensors=True)
    P.run_model_on(1, octo.to_device(v, dtype))
    got, kids = [v] + [P.get_tensor(1, q + 1, n) for q in range(len(layers))], [int(q) for q in P.layer_info(1)[1]]
    P.close()
    for q, (cout, k, stride, res, here, alone, same) in enumerate(layers):
        L = B.m.layers[q]
        one = octo.ConvOp(synth.to_storage(L.weight, dtype), L.bias, dtype, stride, k // 2, zoo.ACT_SILU)
        dx = octo.to_device(got[q], dtype)
        dy = torch.empty((n,) + one.out_hw(got[q].shape[1], got[q].shape[2]) + (cout,), dtype=octo.torch_dtype(dtype), device="cuda")
        kid = octo.op_conv(one, dx, dy, dx if res else None, nn.RES_AFTER_ACT if res else nn.RES_NONE)
        torch.cuda.synchronize()
        if here:
            assert (kids[q] // 100000000, kid // 100000000) == (here, alone) and kids[q] != kid, (q, kids[q], kid)
        y = dy.float().cpu().numpy()
        assert np.array_equal(got[q + 1], y) if same else rel_err(got[q + 1], y) <= TOL[dtype], q
