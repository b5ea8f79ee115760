"""Counts of drawings whose decisions are ties (shapes.py) on the GPU, through
the C ABI: those of the oracle, with no margin for the tags whose decisions
are close; the records at the parity bars."""
import numpy as np
import pytest

import oracle as O
import parity as P
import shapes
from paper_2405_00127_amd import scenes as S

pytestmark = pytest.mark.gpu


def _same_as_the_oracle(sc, newton=False):
    import torch

    from paper_2405_00127_amd import binding as B

    torch.cuda.set_device(0)
    ctx = B.Context(0, density=B.DENSITY_NEWTON if newton else B.DENSITY_APPROX)
    try:
        scene = ctx.encode(sc)
        recs, _, _ = ctx.expand(scene, sc.tolerance, sc.output_mode)
        counts = ctx.counts(scene, sc.tolerance, sc.output_mode).cpu().numpy().astype(np.uint32)
        ref = O.expand(sc, fit_mode=O.DENSITY_NEWTON) if newton else O.expand(sc)
        assert np.array_equal(counts, ref.counts), int((counts != ref.counts).sum())
        rep = P.compare(counts, B.records_to_numpy(recs, sc.output_mode), ref, sc.output_mode)
        assert rep.ok(), rep
    finally:
        ctx.close()


@pytest.mark.parametrize("mode,newton", [(S.OUT_LINES, False), (S.OUT_ARCS, False), (S.OUT_LINES, True)])
@pytest.mark.parametrize("name", shapes.SYMMETRIC)
def test_symmetric_shapes_have_the_oracles_counts(name, mode, newton):
    for s in (1.0, 2.0, 1.0 / 3.0):
        sc = shapes.SYMMETRIC[name](shapes.scale(s))
        sc.output_mode = mode
        print("ties", name, mode, newton, s, flush=True)
        _same_as_the_oracle(sc, newton)


@pytest.mark.parametrize("mode", [S.OUT_LINES, S.OUT_ARCS])
@pytest.mark.parametrize("size,w", [(0.25, 1.0), (1.0, 1.0), (0.25, 10.0)])
def test_perpendicular_hodographs_have_the_oracles_counts(size, w, mode):
    """The hodograph test's sum is 0 or rounding alone: the oracle's rounding."""
    for s in (1.0, 1.0 / 3.0, 0.7, np.sqrt(0.5)):
        sc = shapes.connectors(size, w, shapes.scale(s))
        sc.tolerance, sc.output_mode = 1.0, mode
        print("hodographs", size, w, mode, s, flush=True)
        _same_as_the_oracle(sc)


@pytest.mark.parametrize("degrees", [10, 30, 77])
def test_nearly_constant_curvature_in_exact_density(degrees):
    """Turned circles: their curvature changes by rounding alone along a piece,
    and the exact integral over it is that of a constant density (the GPU's
    rounding is its own: at the parity bars)."""
    import torch

    from paper_2405_00127_amd import binding as B

    torch.cuda.set_device(0)
    ctx = B.Context(0, density=B.DENSITY_NEWTON)
    for radius, w, tol in ((1.0, 2.46, 0.0198), (3.0, 1.0, 0.25), (3.0, 2.46, 0.0198), (10.0, 4.0, 0.25)):
        sc = shapes.circles(radius, w, xform=shapes.rotation(degrees))
        sc.tolerance = tol
        scene = ctx.encode(sc)
        recs, _, _ = ctx.expand(scene, tol, 0)
        counts = ctx.counts(scene, tol, 0).cpu().numpy().astype(np.uint32)
        ref = O.expand(sc, fit_mode=O.DENSITY_NEWTON)
        assert np.abs(counts.astype(int) - ref.counts.astype(int)).max() <= 2  # (one a side)
        rep = P.compare(counts, B.records_to_numpy(recs, 0), ref, 0)
        assert rep.ok(), rep
    ctx.close()
