"""The launch that selects the boxes of a batch (top-k, NMS, first step of the compaction) against the stage calls, which do it in
launches of their own: candidate counts around the edges of a block of 64, of the two ways to sort and of the list, a truncation inside
a block, and crowds.  Everything is equal, to the last bit."""
import numpy as np
import pytest

from paper_2502_01277_amd import synth, zoo

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("topk,max_det,counts", [
    (1000, 300, [0, 1, 63, 64]),
    (1000, 300, [65, 255, 256, 257]),
    (1000, 300, [999, 1000, 1001, 3000]),
    (1000, 40, [200, 2000, 39, 41]),                 # truncated inside the first block
    (100, 100, [99, 100, 101, 700]),
    (1024, 1024, [1023, 1024, 1025, 4500]),          # as many as there are threads; more than the sort holds at once
    (48, 8, [7, 8, 48, 500]),
])
def test_selection_equals_the_stage_calls(octo, topk, max_det, counts):
    import torch
    spec = zoo.detector_only("f16")
    det = spec.models[0]
    det.topk, det.max_det, det.batch_size, spec.max_frames = topk, max_det, 4, 4
    spec.max_rois_per_frame = max_det
    gen = torch.Generator(device="cuda")
    gen.manual_seed(topk + max_det)
    rng = np.random.default_rng(topk * 7 + max_det)
    A, no = det.n_anchors, 5 + det.n_classes
    heads = []
    n_cell = [g * g * A for g in det.grids]
    first = np.cumsum([0] + n_cell)
    for g in det.grids:
        t = torch.randn((4, g * g * A, no), dtype=torch.float16, device="cuda", generator=gen)
        t[..., 4] = -8.0
        t[..., 5:] -= 6.0
        heads.append(t)
    for f, count in enumerate(counts):
        for s in rng.choice(first[-1], count, replace=False):
            lvl = int(np.searchsorted(first, s, side="right")) - 1
            row = heads[lvl][f, int(s - first[lvl])]
            row[4] = float(rng.uniform(1.0, 4.0))
            row[5 + int(rng.integers(0, 4))] = 4.0           # few classes: many boxes of one class beside each other
            row[2:4] += 1.5                                  # and large ones
    heads = [t.reshape(4, g, g, A * no).contiguous() for t, g in zip(heads, det.grids)]
    P = octo.Pipeline(spec)
    for l, t in enumerate(heads):
        P.set_head(0, l, t)
    P.submit([torch.zeros((spec.src_h, spec.src_w, 3), dtype=torch.uint8, device="cuda") for _ in range(4)])
    assert P.run() == 4
    fr, boxes, st = P.collect()
    assert st == octo.OK
    cand, count = octo.op_decode(det, heads)
    assert count.cpu().tolist() == counts
    top, n_top = octo.op_topk(cand, count, min(topk, det.n_cand()))
    keep, n_keep = octo.op_nms(top, n_top, det.iou_thr, max_det)
    _, _, want, _ = octo.op_compact(top, keep, n_keep, (spec.src_h, spec.src_w), (det.in_h, det.in_w), (1 << 128) - 1, 4 * max_det)
    n_keep = n_keep.cpu().numpy()
    assert fr["n_boxes"].tolist() == n_keep.tolist()
    at = 0
    for f in range(4):
        k = int(n_keep[f])
        for name in ("x1", "y1", "x2", "y2", "score", "cls"):
            assert np.array_equal(boxes[name][at:at + k], want[name][f, :k]), (f, name)
        at += k
    assert counts[0] == 0 or n_keep.max() > 1
    P.close()


@pytest.mark.parametrize("cap,classes", [(100, None), (4, None), (100, (1, 3)), (2, (0, 2, 5)), (1, ())])
def test_a_frame_on_its_own(octo, cap, classes):
    """One frame: the launch writes the ROI table too - the kept boxes of the classes that are routed, in their order, as many as it holds."""
    import torch
    spec = zoo.tiny_cascade()
    spec.max_frames, spec.max_rois_per_frame = 1, cap
    spec.models[0].batch_size, spec.models[1].batch_size = 1, cap
    if classes is not None:
        spec.edges[0].class_mask = sum(1 << c for c in classes)
    scene = synth.make_scene(np.random.default_rng(81), 2, 320, 320, [9, 12], 16, 96, n_classes=8)
    P = octo.Pipeline(spec)
    for frame in scene.frames:                               # the second batch finds the counters of the first
        P.submit([torch.from_numpy(frame).cuda()])
        assert P.run() == 1
        fr, boxes, st = P.collect()
        hit = np.flatnonzero([classes is None or b["cls"] in classes for b in boxes])
        rois = P.get_rois(0)
        assert len(boxes) > 3 and len(rois) == min(len(hit), cap)
        at = hit[:cap]
        assert rois["rank"].tolist() == at.tolist() and not rois["frame"].any() and np.array_equal(rois["cls"], boxes["cls"][at])
        for v in ("x1", "y1", "x2", "y2"):
            assert np.array_equal(rois[v], boxes[v][at])
        assert bool(fr["flags"][0] & 1) == (len(hit) > cap)
        labels = boxes["child_label"][:, 0]
        assert (labels[at] >= 0).all() and (np.delete(labels, at) == -1).all()
    P.close()
