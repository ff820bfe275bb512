"""Stage calls on a stream that is not the current one: their scratch memory and outputs come from the current stream's
allocator, whose pending work must neither reach them late nor be handed their memory early."""
import numpy as np
import pytest

from oracle import preprocess as pre
from paper_2502_01277_amd import synth, zoo

pytestmark = pytest.mark.gpu


def _busy(torch, stream, a, out):
    """Some tens of milliseconds of work on a stream."""
    with torch.cuda.stream(stream):
        for _ in range(6):
            torch.mm(a, a, out=out)


@pytest.fixture()
def work(octo):
    import torch
    a = torch.randn((8192, 8192), device="cuda")
    out = torch.empty_like(a)
    torch.mm(a, a, out=out)
    torch.cuda.synchronize()
    return a, out


def test_a_frame_table_waits_for_earlier_users_of_its_memory(octo, work):
    import torch
    frames = [torch.zeros((8, 8 + i, 3), dtype=torch.uint8, device="cuda") for i in range(5)]
    side, here = torch.cuda.Stream(), torch.cuda.current_stream()
    other = torch.full((2, 5), 77, dtype=torch.int64, device="cuda")
    block = torch.empty((2, 5), dtype=torch.int64, device="cuda")
    at = block.data_ptr()
    torch.cuda.synchronize()
    _busy(torch, here, *work)
    block.copy_(other)                             # pending when the block is given back
    del block
    ptrs, pitches = octo.frame_tables(frames, side)
    torch.cuda.synchronize()
    assert ptrs.data_ptr() == at                    # the allocator's own rule; without it this test shows nothing
    assert ptrs.tolist() == [f.data_ptr() for f in frames] and pitches.tolist() == [f.stride(0) for f in frames]


@pytest.mark.parametrize("raw", [False, True])
def test_stage_calls_on_another_stream_equal_those_on_the_current_one(octo, work, raw):
    """Letterbox, decode, top-k, NMS, compaction and crops, with both streams busy, and memory of the calls' scratch tensors asked
    for again at once (filled with a table of other frames, so that a lost race shows as wrong pixels)."""
    import torch
    det = zoo.traffic_cascade("f16").models[0]
    rng = np.random.default_rng(zoo.SEED0 + 55)
    n, sh, sw = 4, 540, 960
    scene = synth.make_scene(rng, n, sh, sw, [3, 9, 1, 5], 24, 200, log_uniform=True)
    geo = pre.letterbox_geometry(sh, sw, det.in_h, det.in_w)[1:]
    heads = [octo.to_device(h, "f16") for h in synth.planted_heads(rng, det, scene, sh, sw, geo)]
    frames = [torch.from_numpy(f).cuda() for f in scene.frames]
    others = [torch.zeros_like(f) for f in frames]
    table = torch.tensor([[f.data_ptr() for f in others], [f.stride(0) for f in others]], dtype=torch.int64, device="cuda")
    n_cu = octo.device_cu_count()
    side = octo.stream_create_range(0, n_cu) if raw else torch.cuda.Stream()
    there = torch.cuda.ExternalStream(side) if raw else side
    here = torch.cuda.current_stream()

    def passes(stream):
        def hurry():
            if stream is not None:
                _busy(torch, here, *work)
                _busy(torch, there, *work)

        def reuse():                                # takes the memory of the call's frame table if that has been given back
            if stream is not None:
                x = torch.empty_like(table)
                x.copy_(table)
        out = []
        hurry()
        lb = octo.op_letterbox(frames, det.in_h, det.in_w, "f16", stream=stream)
        reuse(); hurry()
        cand, count = octo.op_decode(det, heads, cap=256, stream=stream)
        top, tc = octo.op_topk(cand, count, 100, stream=stream)
        keep, nk = octo.op_nms(top, tc, 0.45, 50, stream=stream)
        hurry()
        rois, roi_of, boxes, flags = octo.op_compact(top, keep, nk, (sh, sw), (det.in_h, det.in_w), (1 << 128) - 1, 64, stream=stream)
        assert len(rois) > 0
        hurry()
        crops = octo.op_crop_resize(frames, rois, 64, 64, "f16", cap=len(rois) + 3, stream=stream)
        reuse()
        torch.cuda.synchronize()
        order = octo.cands_from_device(cand, count)                     # decode writes its candidates in any order
        out += [lb.cpu().numpy(), [np.sort(o["idx"]) for o in order], octo.cands_from_device(top, tc), keep.cpu().numpy(), nk.cpu().numpy(),
                rois, roi_of, boxes, flags, crops.cpu().numpy()]
        return out
    want, got = passes(None), passes(side)
    for w, g in zip(want, got):
        for x, y in zip(w, g) if isinstance(w, list) else [(w, g)]:
            assert x.tobytes() == y.tobytes()
    if raw:
        octo.stream_destroy(side)
