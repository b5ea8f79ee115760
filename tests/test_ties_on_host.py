"""Counts of drawings whose decisions are ties (shapes.py) by the device code
compiled for the host: those of the oracle, with no margin for the tags whose
decisions are close.  CPU only."""
import numpy as np
import pytest

import oracle as O
import shapes
from paper_2405_00127_amd import scenes as S
from test_device_code_on_host import _run, dev  # noqa: F401 (a fixture)


@pytest.mark.parametrize("name,mode,flags", [(n, m, f) for n in shapes.SYMMETRIC for m, f in
                                             ((S.OUT_LINES, 0), (S.OUT_ARCS, 0), (S.OUT_LINES, 2))
                                             if m == S.OUT_LINES or n not in shapes.LINES_ONLY])
def test_symmetric_shapes_have_the_oracles_counts(dev, name, mode, flags):  # noqa: F811
    for s in (1.0, 2.0, 1.0 / 3.0):
        sc = shapes.SYMMETRIC[name](shapes.scale(s))
        sc.output_mode = mode
        counts, _ = _run(dev, sc, flags)
        ref = O.expand(sc, fit_mode=O.DENSITY_NEWTON) if flags else O.expand(sc)
        assert np.array_equal(counts, ref.counts), (s, int((counts != ref.counts).sum()))
