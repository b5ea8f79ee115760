"""Counts of drawings whose decisions are ties (shapes.py) by the device code
compiled for the host: those of the oracle, with no margin for the tags whose
decisions are close.  CPU only."""
import numpy as np
import pytest

import oracle as O
import shapes
from paper_2405_00127_amd import scenes as S
from test_device_code_on_host import _run, dev  # noqa: F401 (a fixture)


@pytest.mark.parametrize("mode,flags", [(S.OUT_LINES, 0), (S.OUT_ARCS, 0), (S.OUT_LINES, 2)])
@pytest.mark.parametrize("name", shapes.SYMMETRIC)
def test_symmetric_shapes_have_the_oracles_counts(dev, name, mode, flags):  # noqa: F811
    for s in (1.0, 2.0, 1.0 / 3.0):
        sc = shapes.SYMMETRIC[name](shapes.scale(s))
        sc.output_mode = mode
        counts, _ = _run(dev, sc, flags)
        ref = O.expand(sc, fit_mode=O.DENSITY_NEWTON) if flags else O.expand(sc)
        assert np.array_equal(counts, ref.counts), (s, int((counts != ref.counts).sum()))


@pytest.mark.parametrize("mode", [S.OUT_LINES, S.OUT_ARCS])
@pytest.mark.parametrize("size,w", [(0.25, 1.0), (1.0, 1.0), (0.25, 10.0)])
def test_perpendicular_hodographs_have_the_oracles_counts(dev, size, w, mode):  # noqa: F811
    """The hodograph test's sum is 0 or rounding alone: the oracle's rounding."""
    for s in (1.0, 1.0 / 3.0, 0.7, np.sqrt(0.5)):
        sc = shapes.connectors(size, w, shapes.scale(s))
        sc.tolerance, sc.output_mode = 1.0, mode
        counts, _ = _run(dev, sc)
        ref = O.expand(sc)
        assert np.array_equal(counts, ref.counts), (s, int((counts != ref.counts).sum()))


@pytest.mark.parametrize("degrees", [10, 30, 77])
def test_nearly_constant_curvature_in_exact_density(dev, degrees):  # noqa: F811
    """Turned circles: their curvature changes by rounding alone along a piece,
    and the exact integral over it is that of a constant density."""
    for radius, w, tol in ((1.0, 2.46, 0.0198), (3.0, 1.0, 0.25), (3.0, 2.46, 0.0198), (10.0, 4.0, 0.25)):
        sc = shapes.circles(radius, w, xform=shapes.rotation(degrees))
        sc.tolerance = tol
        counts, _ = _run(dev, sc, 2)
        ref = O.expand(sc, fit_mode=O.DENSITY_NEWTON)
        assert np.array_equal(counts, ref.counts), (radius, w, int((counts != ref.counts).sum()))
