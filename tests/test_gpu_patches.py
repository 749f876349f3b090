"""Catalogues that fill little of their bounding box: the search grid's cells
follow the occupied area, and the blocks stay those of the oracle.

Tolerance: counts are exact; the estimate within the bars of the precisions
(1e-10, 1e-5 per correlator)."""
import numpy as np
import pytest

import oracle
import synth
from helpers import rel_per_mu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fp():
    import paper_2509_07974_amd as m
    m.lib()
    return m


def catalogue(kind):
    cat = synth.uniform_catalogue(51, 900, 24.0)
    x, y = cat.x.copy(), cat.y.copy()
    if kind == "two":
        x[450:] += 700.0
        y[450:] -= 2000.0
    elif kind == "outlier":
        x[3], y[3] = -3e4, 5e4
    elif kind == "far":              # far from the origin, around multiples of the bitmap's period
        x += 256 * 2.25 * 1000 - 12.0
        y -= 256 * 2.25 * 3 + 12.0
    return synth.Catalogue(x, y, cat.g1, cat.g2, cat.w)


@pytest.mark.parametrize("kind", ["two", "outlier", "far"])
@pytest.mark.parametrize("precision,bar", [("fp64", 1e-10), ("fp16", 1e-5)])
def test_patches(fp, kind, precision, bar):
    cat, edges = catalogue(kind), synth.log_edges(0.5, 18.0, 4)
    cen = np.arange(0, cat.n, 7)
    counts, _, _ = fp.debug_multipoles(*cat.arrays(), edges, 5, precision=precision, centers=cen)
    assert np.array_equal(counts, oracle.multipoles(*cat.arrays(), edges, 5, cen)["counts"])
    got = fp.estimate_4pcf_multipoles(*cat.arrays(), edges, 5, precision=precision, centers=cen)
    assert np.all(rel_per_mu(got, oracle.upsilon(*cat.arrays(), edges, 5, cen)) < bar)
