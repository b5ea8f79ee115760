"""The forms of an emission item (GPU, through the C ABI): one unit or two,
with and without its last quarters.  An item's records do not depend on how
many chunks it is cut into, so every chunk size gives the same bytes: 1 (each
item of more than one record in several chunks), 2 to 4 (both forms side by
side; small scenes take at most 4) and, in a scene past 2^17 slots, 255 (no
item in several).  Every join and cap, cusps and loops (split ranges,
evolutes), fills; lines, arcs and exact-density lines."""
import numpy as np
import pytest

import oracle as O
import parity as P
from paper_2405_00127_amd import scenes as S

pytestmark = pytest.mark.gpu


def _scene(copies):
    """Every join x start cap x end cap x width, `copies` times, moved about."""
    rng = np.random.Generator(np.random.PCG64(7))
    b, styles = S.SceneBuilder(), []
    for _ in range(copies):
        for join in (S.JOIN_BEVEL, S.JOIN_MITER, S.JOIN_ROUND):
            for cap in (S.CAP_BUTT, S.CAP_SQUARE, S.CAP_ROUND):
                for w in (0.5, 12.0):
                    at = rng.uniform(50, 900, 2)
                    pts = at + np.array([[0, 0], [30, 5], [40, 60], [70, 10],  # a curve, then a corner
                                         [20, 80], [55, 110], [-40, 110], [15, 80],  # a loop
                                         [16, 20], [60, 90], [60, 90], [90, 91]])  # a line, a degenerate cubic
                    verbs = [S.MOVE, S.CUBIC, S.LINE, S.CUBIC, S.LINE, S.CUBIC]
                    b.add_path(verbs, pts, len(styles), 0)
                    styles.append((w, join, cap))
    st = np.concatenate([S.make_styles([w], j, c, (c + 1) % 3) for w, j, c in styles])
    if copies == 1:
        st["flags"][::5] |= S.STYLE_FILL
    return b.build(st, tolerance=0.1)


@pytest.mark.parametrize("copies,chunks", [(1, (1, 2, 3, 4)), (1500, (1, 16, 255))])
@pytest.mark.parametrize("mode,newton", [(S.OUT_LINES, False), (S.OUT_ARCS, False), (S.OUT_LINES, True)])
def test_chunk_sizes_give_the_same_bytes(copies, chunks, mode, newton):
    import torch

    from paper_2405_00127_amd import binding as B

    sc = _scene(copies)
    sc.output_mode = mode
    ctx = B.Context(0, density=B.DENSITY_NEWTON if newton else B.DENSITY_APPROX)
    try:
        scene, rec, ref = ctx.encode(sc), B.RECORD_BYTES[mode], None
        for k in chunks:
            ctx.set_tuning(chunk_k=k)
            recs, n, buf = ctx.expand(scene, sc.tolerance, mode)
            got = buf[: n * rec].clone()
            assert ref is None or torch.equal(got, ref), k
            ref = got
        if copies == 1 and not newton:
            counts = ctx.counts(scene, sc.tolerance, mode).cpu().numpy().astype(np.uint32)
            rep = P.compare(counts, B.records_to_numpy(recs, mode), O.expand(sc), mode)
            assert rep.ok(), rep
    finally:
        ctx.close()


def _right_angles(n, join=S.JOIN_ROUND):
    """Polylines of right angles with wide joins (18 records each at tolerance
    0.1): more item units per tag than the tile regions hold."""
    b = S.SceneBuilder()
    for k in range(n // 100):
        steps = np.tile([[30.0, 0.0], [0.0, 30.0]], (50, 1))
        pts = np.concatenate([[[0.0, 0.0]], np.cumsum(steps, 0)]) + [20.0 * (k % 97), 20.0 * (k // 97)]
        b.add_path([S.MOVE] + [S.LINE] * 100, pts, 0, 0)
    return b.build(S.make_styles([50.0], join, S.CAP_ROUND), tolerance=0.1)


@pytest.mark.parametrize("n", [8000, 20000, 32000])
@pytest.mark.parametrize("chunk_k", [16, 255])
def test_short_chunks_fit_where_long_ones_did(n, chunk_k):
    """A small scene's chunks of four records take more units than those of
    chunk_k: a fresh scene's workspace still serves an asynchronous expansion
    that it served with them (6 and 4 units a tag of 4 in the regions and 4 in
    the overflow area), with the bytes of a synchronous one of long chunks."""
    import torch

    from paper_2405_00127_amd import binding as B

    sc = _right_angles(n)
    ctx = B.Context(0)
    try:
        ctx.set_tuning(chunk_k=chunk_k)
        scene = ctx.encode(sc)
        out = torch.zeros(scene.n_tags * 24 * B.RECORD_BYTES[0], dtype=torch.uint8, device="cuda")
        status = torch.ones(2, dtype=torch.int64, device="cuda")
        ctx.expand_async(scene, out.data_ptr(), out.numel(), status.data_ptr(), sc.tolerance, S.OUT_LINES)
        torch.cuda.synchronize()
        assert int(status[1]) == 0
        # the same paths among so many that their chunks are chunk_k long
        b = S.SceneBuilder()
        for k in range(sc.n_paths):
            b.add_path(*sc.path(k), 0, 0)
        for k in range(400):
            b.add_path([S.MOVE] + [S.LINE] * 100, np.stack([np.arange(101) * 3.0, np.arange(101) % 2], 1), 0, 0)
        recs, n_rec, buf = ctx.expand(ctx.encode(b.build(sc.styles, tolerance=0.1)), 0.1, S.OUT_LINES)
        m = int(status[0]) * B.RECORD_BYTES[0]
        assert torch.equal(out[:m], buf[:m])
    finally:
        ctx.close()
