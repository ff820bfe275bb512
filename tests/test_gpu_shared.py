"""Several pipelines with batches in flight at once: their launches are then replayed from recorded graphs.  Every replay
must give what the pipeline gives alone, for frames that change from batch to batch, partial batches and swapped heads."""
import numpy as np
import pytest

from paper_2502_01277_amd import synth, zoo

pytestmark = pytest.mark.gpu


def _spec_and_batches(octo, frames, counts, seed, size=(1080, 1920)):
    """The traffic cascade for up to `frames` frames, and per entry of `counts` (objects per frame) a batch's frames and heads."""
    import torch
    spec = zoo.traffic_cascade("f16", det_batch=frames, max_rois_per_frame=24)
    spec.src_h, spec.src_w = size
    det = spec.models[0]
    rng = np.random.default_rng(zoo.SEED0 + seed)
    sets = []
    for c in counts:
        scene = synth.make_scene(rng, frames, *size, c, 24, 360, log_uniform=True)
        heads = synth.planted_heads(rng, det, scene, *size, octo.letterbox_geometry(*size, det.in_h, det.in_w))
        sets.append(([torch.from_numpy(f).cuda() for f in scene.frames], [octo.to_device(h, det.dtype) for h in heads]))
    return spec, sets


def _plant(P, heads):
    for l, h in enumerate(heads):
        P.set_head(0, l, h)


def test_batches_of_every_size_are_replayed(octo):
    """Batch sizes and object counts that change from batch to batch, as a server's do: after a warm-up nine executions of a model
    in ten are replays, recordings stay few, and every batch gives what it gives alone."""
    spec, [(frames, heads)] = _spec_and_batches(octo, 12, [[0, 9, 1, 4, 14, 2, 7, 0, 3, 20, 6, 5]], 78)
    solo = octo.Pipeline(spec)
    _plant(solo, heads)
    want = {}
    for n in range(1, 13):
        solo.submit(frames[:n])
        assert solo.run() == n
        want[n] = solo.collect()[1].tobytes()
    assert solo.launch_counts() == (12 * 3, 0, 0)          # alone on the GPU: never
    solo.close()
    pipes = [octo.Pipeline(spec) for _ in range(3)]
    for P in pipes:
        _plant(P, heads)
    rng = np.random.default_rng(1)
    before = [None] * 3
    for r in range(150):
        sizes = rng.integers(1, 13, 3)
        if r == 90:
            before = [P.launch_counts() for P in pipes]
        for P, n in zip(pipes, sizes):
            P.submit(frames[:n])
            assert P.run() == n
        for P, n in zip(pipes, sizes):
            assert P.collect()[1].tobytes() == want[n], (r, n)
    for P, (e0, r0, _) in zip(pipes, before):
        e1, r1, rec = P.launch_counts()
        assert e1 - e0 + r1 - r0 == 60 * 3 and r1 - r0 >= 0.9 * 60 * 3, (e1 - e0, r1 - r0)
        assert 12 <= rec <= 12 + 2 * 10, rec                # twelve batch sizes; item counts of two children, rounded
        P.close()


def test_pipelines_of_several_threads(octo):
    """Each pipeline driven by a thread of its own, on its own stream: one records while the others enqueue and replay."""
    import threading
    import torch
    spec, [(frames, heads)] = _spec_and_batches(octo, 6, [[4, 9, 0, 13, 2, 6]], 82)
    solo = octo.Pipeline(spec)
    _plant(solo, heads)
    want = {}
    for n in range(1, 7):
        solo.submit(frames[:n])
        solo.run()
        want[n] = solo.collect()[1].tobytes()
    solo.close()
    n_cu = octo.device_cu_count()
    streams = [octo.stream_create_range(0, n_cu) for _ in range(3)]
    pipes = [octo.Pipeline(spec) for _ in range(3)]
    for P in pipes:
        _plant(P, heads)
    torch.cuda.synchronize()
    wrong = []

    def drive(k):
        rng = np.random.default_rng(k)
        for r in range(40):
            n = int(rng.integers(1, 7))
            pipes[k].submit(frames[:n])
            pipes[k].run(streams[k])
            if pipes[k].collect()[1].tobytes() != want[n]:
                wrong.append((k, r, n))
    threads = [threading.Thread(target=drive, args=(k,)) for k in range(3)]
    for th in threads:
        th.start()
    for th in threads:
        th.join()
    assert not wrong
    assert all(P.launch_counts()[1] > 0 for P in pipes)
    for P in pipes:
        P.close()
    for s in streams:
        octo.stream_destroy(s)


def test_an_uncollected_batch_elsewhere_is_no_work_on_the_gpu(octo):
    import torch
    spec, [(frames, heads)] = _spec_and_batches(octo, 2, [[3, 5]], 79)
    idle, P = octo.Pipeline(spec), octo.Pipeline(spec)
    for q in (idle, P):
        _plant(q, heads)
    idle.submit(frames)
    idle.run()
    torch.cuda.synchronize()
    for _ in range(6):
        P.submit(frames)
        P.run()
        want = P.collect()[1].tobytes()
    assert P.launch_counts() == (18, 0, 0)
    assert idle.collect()[1].tobytes() == want
    idle.close()
    P.close()


def test_layer_info_names_the_kernels_of_a_replayed_batch(octo):
    """A replay enqueues nothing itself; the kernels reported are still those of the batch that ran last."""
    spec, [(frames, heads)] = _spec_and_batches(octo, 16, [[4] * 16], 80)

    def kernels(P):
        return [[int(k) for k in P.layer_info(m)[1]] for m in range(3)]
    solo = octo.Pipeline(spec)
    _plant(solo, heads)
    want = {}
    for n in (16, 1):
        solo.submit(frames[:n])
        solo.run()
        solo.collect()
        want[n] = kernels(solo)[0]
    assert want[16] != want[1]
    solo.close()
    pipes = [octo.Pipeline(spec) for _ in range(2)]
    for P in pipes:
        _plant(P, heads)
    most = [0, 0]                                          # models replayed in one batch
    for r in range(12):
        n = (16, 1)[r % 2]
        counts = [P.launch_counts()[1] for P in pipes]
        for P in pipes:
            P.submit(frames[:n])
            P.run()
        for P in pipes:
            P.collect()
            assert kernels(P)[0] == want[n], (r, n)
        most = [max(m, P.launch_counts()[1] - c) for m, P, c in zip(most, pipes, counts)]
    assert most == [3, 3]                                  # the detector's too
    for P in pipes:
        P.close()


def test_replayed_batches_equal_batches_alone(octo):
    import torch
    spec = zoo.traffic_cascade("f16", det_batch=4, max_rois_per_frame=12)
    det = spec.models[0]
    rng = np.random.default_rng(zoo.SEED0 + 77)
    sets = []
    for k in range(3):
        scene = synth.make_scene(rng, 4, 1080, 1920, [3, 0, 7, 5 + k], 24, 360, log_uniform=True)
        heads = synth.planted_heads(rng, det, scene, 1080, 1920, octo.letterbox_geometry(1080, 1920, det.in_h, det.in_w))
        sets.append(([torch.from_numpy(f).cuda() for f in scene.frames], [octo.to_device(h, det.dtype) for h in heads]))

    def batch(P, s, n, collect=True):
        for l, h in enumerate(sets[s][1]):
            P.set_head(0, l, h)
        P.submit(sets[s][0][:n])
        assert P.run() == n
        return P.collect()[1].tobytes() if collect else None

    solo = octo.Pipeline(spec)
    want = {(s, n): batch(solo, s, n) for s in range(3) for n in (4, 3)}
    solo.close()
    pipes = [octo.Pipeline(spec) for _ in range(2)]
    for r in range(6):
        # the same heads for three rounds: recorded in the second, replayed in the third
        for k, P in enumerate(pipes):
            if r % 3 == 0:
                for l, h in enumerate(sets[(r // 3 + k) % 3][1]):
                    P.set_head(0, l, h)
            for n in (4, 3):
                P.submit(sets[(r // 3 + k) % 3][0][:n])
                assert P.run() == n
        for k, P in enumerate(pipes):
            got = [P.collect(frame_cap=4)[1] for _ in range(2)]
            assert [g.tobytes() for g in got] == [want[(r // 3 + k) % 3, n] for n in (4, 3)], (r, k)
    for P in pipes:
        P.close()
