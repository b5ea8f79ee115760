"""The bisection, the piece list and the record launch at the edges of their
dispatch (GPU, through the C ABI): scenes at the tag counts where the list
kernel, the record chunks (2^17 slots, four per tag at first), the scans (2^16
and 2^18 tags, 2^17 and 2^20 slots) and the list's turns change, tags with
more pieces than the bisection keeps codes for, and runs of tags without
pieces longer than the list kernel stages.  Against the FP64 oracle at the
parity bars (or bit for bit against the same paths expanded without the empty
ones)."""
import numpy as np
import pytest

import oracle as O
import parity as P
from paper_2405_00127_amd import scenes as S

pytestmark = pytest.mark.gpu

SMALL_TAGS = 4096  # kSmallTags of the list kernels


@pytest.fixture(scope="module")
def ctx():
    import torch

    from paper_2405_00127_amd import binding as B

    torch.cuda.set_device(0)
    c = B.Context(0)
    yield c
    c.close()


def _with_tags(n_tags):
    """A map-shaped scene of exactly n_tags tags: one of 40% fewer segments,
    then open paths of two lines (3 tags) and of one line (2 tags)."""
    base = S.scene_map(11, n_tags * 3 // 5, max(1, n_tags // 125))
    rest = n_tags - len(O.encode(base).tags)
    assert rest >= 3
    b = S.SceneBuilder()
    for k in range(base.n_paths):
        b.add_path(*base.path(k), int(base.style_ix[k]), 0)
    while rest:
        m = 2 if rest % 2 else 1
        x = float(rest % 1000)
        b.add_path([S.MOVE] + [S.LINE] * m, [[x, 5.0], [x + 3.0, 9.0], [x + 7.0, 4.0]][: m + 1], 0, 0)
        rest -= m + 1
    sc = b.build(base.styles, base.xforms, tolerance=0.25)
    assert len(O.encode(sc).tags) == n_tags
    return sc


def _check(ctx, sc):
    from paper_2405_00127_amd import binding as B

    ref = O.expand(sc)
    scene = ctx.encode(sc)
    recs, _, _ = ctx.expand(scene, sc.tolerance, sc.output_mode)
    counts = ctx.counts(scene, sc.tolerance, sc.output_mode).cpu().numpy().astype(np.uint32)
    rep = P.compare(counts, B.records_to_numpy(recs, sc.output_mode), ref, sc.output_mode)
    assert rep.ok(), rep
    scene.release()


@pytest.mark.parametrize("n_tags", [12, 255, 257, SMALL_TAGS, SMALL_TAGS + 1, 16385, 32768, 32769, 65537, 262145])
def test_tag_counts_at_the_edges(ctx, n_tags):
    _check(ctx, _with_tags(n_tags))


@pytest.mark.parametrize("n_cubics,extra", [(6, 0), (6, SMALL_TAGS)])
def test_more_pieces_than_codes_kept(ctx, n_cubics, extra):
    """About 1,400 pieces per cubic (1,024 codes are kept at most): the
    tag's bisection runs again, by its wave (small scenes) or beside the slot
    scan."""
    sc = S.scene_c1(5, n_paths=2, n_cubics=n_cubics, tolerance=1e-5)
    if extra:
        b = S.SceneBuilder()
        for k in range(sc.n_paths):
            b.add_path(*sc.path(k), int(sc.style_ix[k]), 0)
        for j in range(extra // 2):
            b.add_path([S.MOVE, S.LINE], [[j % 997, 1.0], [j % 997 + 2.5, 8.0]], 0, 0)
        sc = b.build(sc.styles, sc.xforms, tolerance=1e-5)
    assert len(O.expand(sc).pieces) > 1024 * n_cubics
    _check(ctx, sc)


@pytest.mark.parametrize("mode", [S.OUT_LINES, S.OUT_ARCS])
@pytest.mark.parametrize("kept,others", [(1008, 31_000), (80, 380_000), (32, 1_050_000)])
def test_codes_kept_do_not_change_the_outline(ctx, kept, others, mode):
    """2,000 stress cubics (cusps, loops, degenerate ones; 10 to 400 pieces
    each), alone, with all their codes kept, and before so many lines that
    `kept` codes are kept per tag: the same records.  A cubic in a thousand
    pieces among them."""
    from paper_2405_00127_amd import binding as B

    few = S.scene_c3(6, n_cubics=2000, output_mode=mode, tolerance=0.02)
    b = S.SceneBuilder()
    for k in range(few.n_paths):
        b.add_path(*few.path(k), int(few.style_ix[k]), 0)
    b.add_path([S.MOVE, S.CUBIC], [[0, 0], [3e6, 1e6], [-2e6, 1e6], [1e6, 0]], 0, 0)
    few = b.build(few.styles, few.xforms, tolerance=few.tolerance, output_mode=mode)
    n = others // 21
    x = np.arange(21 * n, dtype=np.float32).reshape(n, 21)
    lines = np.stack([x % 997, (x % 2) * 9 + x % 13], 2)
    many = b.build(few.styles, few.xforms, tolerance=few.tolerance, output_mode=mode)
    many.verbs = np.concatenate([many.verbs, np.tile(np.uint8([S.MOVE] + [S.LINE] * 20), n)])
    many.verb_off = np.concatenate([many.verb_off, many.verb_off[-1] + 21 * np.arange(1, n + 1, dtype=np.uint32)])
    many.pts = np.concatenate([many.pts, lines.reshape(-1, 2)])
    many.pt_off = np.concatenate([many.pt_off, many.pt_off[-1] + 21 * np.arange(1, n + 1, dtype=np.uint32)])
    many.style_ix = np.concatenate([many.style_ix, np.zeros(n, np.uint32)])
    many.xform_ix = np.concatenate([many.xform_ix, np.zeros(n, np.uint32)])
    got = []
    for sc in (few, many):
        scene = ctx.encode(sc)
        assert sc is few or max(32, (2**25 // (scene.n_tags + 1)) & ~15) == kept, scene.n_tags
        recs, _, _ = ctx.expand(scene, sc.tolerance, mode)
        got.append(B.records_to_numpy(recs, mode).copy())
        scene.release()
    assert len(got[0]) > 300_000
    assert np.array_equal(got[1][: len(got[0])], got[0])
    assert got[1]["path"][len(got[0])] == few.n_paths


def test_long_runs_of_tags_without_pieces(ctx):
    """9,000 paths whose dashes draw nothing (two empty subpaths each) between
    solid ones: a turn of the list kernel spans more tags than it stages."""
    from paper_2405_00127_amd import binding as B

    solid = S.scene_c1(7, n_paths=4, n_cubics=40)
    b = S.SceneBuilder()
    keep = S.SceneBuilder()
    n_st = len(solid.styles)
    for k in range(4):
        b.add_path(*solid.path(k), k, 0)
        keep.add_path(*solid.path(k), k, 0)
        for j in range(2250):
            b.add_path([S.MOVE, S.LINE], [[j, 0.0], [j + 1.0, 3.0]], n_st, 0)
    styles = np.concatenate([solid.styles, solid.styles[:1]])
    sc = b.build(styles, solid.xforms)
    sc.dashes = [None] * n_st + [(np.array([0.0, 10.0], np.float32), 0.0)]
    ref = keep.build(styles, solid.xforms)
    got, n, _ = ctx.expand(ctx.encode(sc), 0.25, S.OUT_LINES)
    want, m, _ = ctx.expand(ctx.encode(ref), 0.25, S.OUT_LINES)
    got, want = (B.records_to_numpy(x, S.OUT_LINES).copy() for x in (got, want))
    assert n == m
    want["path"] *= 2251
    assert np.array_equal(got, want)
