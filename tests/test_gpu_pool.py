"""Device memory that scenes give back and later scenes take (GPU, through the
C ABI): outlines of scenes opened on recycled memory are those of the same
scenes in a fresh context, whatever was there before and on whichever stream,
and scenes and batches may outlive the context's own use of the memory."""
import numpy as np
import pytest

from paper_2405_00127_amd import scenes as S

pytestmark = pytest.mark.gpu


def _records(ctx, sc, stream=None):
    scene = ctx.encode(sc, stream=stream)
    recs, n, _ = ctx.expand(scene, sc.tolerance, sc.output_mode, stream=stream)
    out = recs.cpu().numpy().copy()
    return scene, out


def _scenes():
    # sizes up and down across the kept blocks' bounds, other kinds between
    return [S.scene_map(1, 30000, 300), S.scene_map(2, 29000, 290), S.scene_c1(3),
            S.with_dashes(S.scene_map(4, 9000, 90), 4, 0.5, 12.0), S.with_fills(S.scene_map(5, 60001, 600)),
            S.scene_map(1, 30000, 300), S.scene_map(6, 12, 1)]


def test_recycled_memory_gives_the_same_outlines():
    import torch

    from paper_2405_00127_amd import binding as B

    torch.cuda.set_device(0)
    ctx = B.Context(0)
    streams = [None, torch.cuda.Stream(), torch.cuda.Stream()]
    for k, sc in enumerate(_scenes()):
        fresh = B.Context(0)
        f_scene, want = _records(fresh, sc)
        scene, got = _records(ctx, sc, streams[k % 3])
        assert np.array_equal(got.view(np.uint32), want.view(np.uint32)), k
        scene.release()
        f_scene.release()
        fresh.close()
    ctx.close()


def test_release_with_work_queued():
    """A scene's memory goes to the next scene only once its work is done."""
    import torch

    from paper_2405_00127_amd import binding as B

    torch.cuda.set_device(0)
    ctx = B.Context(0)
    sc = S.scene_map(7, 40000, 400)
    scene, want = _records(ctx, sc)
    other = torch.cuda.Stream()
    out = torch.empty(want.nbytes, dtype=torch.uint8, device="cuda")
    status = torch.zeros(2, dtype=torch.int64, device="cuda")
    torch.cuda.synchronize()
    for _ in range(20):
        ctx.expand_async(scene, out.data_ptr(), out.numel(), status.data_ptr(), 0.25, 0, stream=other)
    scene.release()
    s2, _ = _records(ctx, S.scene_map(8, 40000, 400))
    torch.cuda.synchronize()
    assert np.array_equal(out.cpu().numpy().view(np.uint32), want.reshape(-1).view(np.uint32))
    s2.release()
    ctx.close()


def test_batch_outlives_its_context():
    import torch

    from paper_2405_00127_amd import binding as B

    torch.cuda.set_device(0)
    ctx = B.Context(0)
    batch = B.Batch(ctx)
    batch.set([ctx.encode(S.scene_map(9, 20000, 200))])
    batch.prepare(0.25, 0)
    ctx.close()
    batch.destroy()


def test_release_while_another_scene_is_captured():
    """A relaxed capture goes on when a scene is released; its graph replays."""
    import torch

    from paper_2405_00127_amd import binding as B

    torch.cuda.set_device(0)
    ctx = B.Context(0)
    sc = S.scene_map(1, 3000, 30)
    scene, want = _records(ctx, sc)
    other, _ = _records(ctx, S.scene_map(2, 3000, 30))
    out = torch.zeros(want.nbytes, dtype=torch.uint8, device="cuda")
    status = torch.zeros(2, dtype=torch.int64, device="cuda")
    torch.cuda.synchronize()
    graph, stream = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    with torch.cuda.stream(stream):
        graph.capture_begin(capture_error_mode="relaxed")
        ctx.expand_async(scene, out.data_ptr(), out.numel(), status.data_ptr(), sc.tolerance, 0, stream=stream)
        other.release()
        graph.capture_end()
    for _ in range(3):
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(out.cpu().numpy().view(np.uint32), want.reshape(-1).view(np.uint32))
    scene.release()
    ctx.close()


def test_release_waits_for_every_stream():
    """Work of a scene that is still queued on a stream other than its last."""
    import torch

    from paper_2405_00127_amd import binding as B

    torch.cuda.set_device(0)
    ctx = B.Context(0)
    scene, want = _records(ctx, S.scene_map(7, 40000, 400))
    busy, last = torch.cuda.Stream(), torch.cuda.Stream()
    out = torch.empty(want.nbytes, dtype=torch.uint8, device="cuda")
    status = torch.zeros(2, dtype=torch.int64, device="cuda")
    work = torch.ones(1 << 28, device="cuda")
    torch.cuda.synchronize()
    with torch.cuda.stream(busy):
        for _ in range(40):
            work.mul_(1.0)
    ctx.expand_async(scene, out.data_ptr(), out.numel(), status.data_ptr(), 0.25, 0, stream=busy)
    done = busy.record_event()
    # (the scene's last stream, with no work queued on it)
    ctx.run_phase(scene, 2, 0.25, 0, stream=last)
    assert not done.query()
    scene.release()
    assert done.query()
    assert np.array_equal(out.cpu().numpy().view(np.uint32), want.reshape(-1).view(np.uint32))
    ctx.close()
