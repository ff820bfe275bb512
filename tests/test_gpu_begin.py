"""The first launch of a batch: as many frames as one launch's arguments hold, one more, the detector on a few of them at a time; the frames that the letterbox reads, the table that the
crops read, and the counters of the batch before."""
import numpy as np
import pytest

from paper_2502_01277_amd import synth, zoo


@pytest.mark.gpu
@pytest.mark.parametrize("n,bz", [(1, 0), (3, 0), (7, 3), (64, 0), (64, 5), (65, 0), (130, 64)])
def test_frames_and_counters(octo, n, bz):
    import torch
    spec = zoo.tiny_cascade()
    spec.max_frames = n
    spec.models[0].batch_size = n
    spec.models[1].batch_size = n * spec.max_rois_per_frame
    scene = synth.make_scene(np.random.default_rng(71), 2, 320, 320, [6, 5], 16, 96, n_classes=8)
    frames = [torch.from_numpy(np.roll(scene.frames[i % 2], (i, 2 * i), (0, 1))).cuda() for i in range(n)]
    wide = torch.zeros(320, 324, 3, dtype=torch.uint8, device="cuda")
    wide[:, :320] = frames[-1]
    frames[-1] = wide[:, :320]                                   # rows of another pitch
    det = spec.models[0]

    def batch(P, fr):
        P.submit(fr)
        assert P.run() == len(fr)
        got, boxes, _ = P.collect()
        return got["n_boxes"].tolist(), boxes.copy(), P.get_rois(0).copy()

    P = octo.Pipeline(spec, keep_all_tensors=2)
    if bz:
        P.set_detector_batch(bz)
    batch(P, frames[::-1])                                       # leaves other frames, and counters that are not zero
    used = batch(P, frames)
    # the last frame, in the input buffer of the detector's last execution, and the last crop (a copy of 12-byte rows is slow: one item of each)
    at = (n - 1) // bz * bz if 0 < bz < n else 0
    x, crop = P.get_tensor(0, 0, 1, first=n - 1 - at), P.get_tensor(1, 0, 1, first=len(used[2]) - 1)
    P.close()
    Q = octo.Pipeline(spec, keep_all_tensors=2)
    if bz:
        Q.set_detector_batch(bz)
    fresh = batch(Q, frames)
    Q.close()
    assert used[0] == fresh[0] and sum(used[0]) > 0
    for a, b in zip(used[1:], fresh[1:]):
        assert np.array_equal(a, b)
    want = octo.op_letterbox(frames[-1:], det.in_h, det.in_w, det.dtype).float().cpu().numpy()
    assert np.array_equal(x[..., :3].reshape(want.shape), want)
    cls = spec.models[1]
    want = octo.op_crop_resize(frames, used[2], cls.in_h, cls.in_w, cls.dtype, cap=len(used[2]))[-1].float().cpu().numpy()
    assert np.array_equal(crop[..., :3].reshape(want.shape), want)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("h,w", [(1080, 1920), (1920, 1080)])
def test_frames_of_a_launch_with_four_rows_per_lane(octo, dtype, h, w):
    """64 frames at three times the detector's size, where the first launch takes its rows in groups: borders above and below, and at the sides.  The detector's input and the crops against the stage
    calls, which read the frames from a table."""
    import torch
    n = 64
    det = zoo.plain_detector("det", dtype, 640, (8, 8, 8), 8, zoo.SEED0 + 5, batch_size=n, topk=100, max_det=100)
    B = zoo._Builder("child", dtype, 32, 32, "classifier", np.random.default_rng(72))
    B.m.outputs = [B.fc(B.gap(B.conv(0, 16, 3, 2, act=zoo.ACT_RELU)), 4)]
    B.m.batch_size = 4 * n
    spec = zoo.PipelineSpec("rows", [det, B.m], [zoo.Edge(0, 1)], 1000.0, h, w, n, 4)
    few = torch.randint(0, 256, (3, h, w, 3), dtype=torch.uint8, device="cuda", generator=torch.Generator(device="cuda").manual_seed(8))
    frames = [few[(i * i) % 3] for i in range(n)]
    P = octo.Pipeline(spec, keep_all_tensors=2)
    P.submit(frames)
    assert P.run() == n
    P.collect()
    rois = P.get_rois(0).copy()
    at = (0, n - 1)                                      # (a copy of short rows is slow: a few items)
    got = [P.get_tensor(0, 0, 1, first=i) for i in at]
    assert len(rois) > n
    crops = P.get_tensor(1, 0, 6, first=len(rois) - 6)
    P.close()
    want = octo.op_letterbox([frames[i] for i in at], 640, 640, dtype).float().cpu().numpy()
    for k in range(len(at)):
        assert np.array_equal(got[k][..., :3].reshape(want[k].shape), want[k]), at[k]
    want = octo.op_crop_resize(frames, rois, 32, 32, dtype, cap=len(rois))[-6:].float().cpu().numpy()
    assert np.array_equal(crops[..., :3].reshape(want.shape), want)
