"""Letterbox of frames at three times the size, rows in groups: the last group, borders, alignments that leave the words."""
import numpy as np
import pytest

from oracle import preprocess as pre

pytestmark = pytest.mark.gpu


# destination heights that end inside a group of four rows; borders above, at the sides (142 columns: no group of four pixels is aligned), none;
# rows and frames at odd addresses
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("sh,sw,dh,dw,skip", [(1080, 1920, 363, 640, 0), (1080, 1920, 640, 640, 0), (1920, 1068, 640, 640, 0), (1080, 1920, 361, 640, 1), (1920, 1080, 640, 642, 0)])
def test_rows_in_groups(octo, dtype, sh, sw, dh, dw, skip):
    import torch
    n = 10
    big = torch.randint(0, 256, (n, sh, sw + skip, 3), dtype=torch.uint8, device="cuda", generator=torch.Generator(device="cuda").manual_seed(5))
    frames = [b[:, skip:] for b in big]
    got = octo.op_letterbox(frames, dh, dw, dtype).float().cpu().numpy()
    want = pre.letterbox(np.stack([frames[i].cpu().numpy() for i in (0, n - 1)]), dh, dw, dtype)
    assert np.abs(got[[0, n - 1]] - want).max() <= (2.0 ** -23 if dtype == "f32" else 2.0 ** -8)      # a product of at most 1, rounded to the type


# launches large enough for four rows per lane: a last group of one row, groups that begin or end in the border above and below, borders at
# the sides, frames at odd addresses
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("sh,sw,dh,dw,skip,n", [(1080, 1920, 361, 640, 0, 110), (1080, 1920, 638, 640, 0, 64), (1920, 1056, 640, 640, 0, 64), (1080, 1920, 638, 640, 1, 64)])
def test_rows_in_groups_of_a_large_launch(octo, dtype, sh, sw, dh, dw, skip, n):
    import torch
    few = torch.randint(0, 256, (3, sh, sw + skip, 3), dtype=torch.uint8, device="cuda", generator=torch.Generator(device="cuda").manual_seed(6))
    got = octo.op_letterbox([few[i % 3][:, skip:] for i in range(n)], dh, dw, dtype)
    want = pre.letterbox(few[:, :, skip:].cpu().numpy(), dh, dw, dtype)
    tol = 2.0 ** -23 if dtype == "f32" else 2.0 ** -8                  # a product of at most 1, rounded to the type
    assert np.abs(got[:3].float().cpu().numpy() - want).max() <= tol
    for i in range(3, n):
        assert torch.equal(got[i], got[i % 3]), i
