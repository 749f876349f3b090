"""The register tiles of the 3PCF contraction: bin counts around its tile
sizes (2 to 6 bins, with and without surplus), and centre counts around a wave
and a slice (sums over all neighbours: two galaxies have no distinct pair)."""
import numpy as np
import pytest

import oracle
import synth
from helpers import rel_per_mu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nb", [1, 2, 3, 5, 6, 7, 9, 11, 13, 17])
def test_bins(nb):
    import paper_2509_07974_amd as fp
    cat = synth.uniform_catalogue(nb, 300, 40.0)
    edges = synth.log_edges(0.5, 25.0, nb)
    got = fp.estimate_3pcf_multipoles(*cat.arrays(), edges, 3, precision="fp64")
    assert np.all(rel_per_mu(got, oracle.upsilon3(*cat.arrays(), edges, 3)) < 1e-10)


@pytest.mark.parametrize("n", [2, 63, 64, 65, 1023, 1025])
@pytest.mark.parametrize("precision,bar", [("fp64", 1e-10), ("fp16", 1e-5)])
def test_centres(n, precision, bar):
    import paper_2509_07974_amd as fp
    cat = synth.uniform_catalogue(n, n, 30.0 * np.sqrt(n / 300) + 4.0)
    edges = synth.log_edges(0.5, 20.0, 5)
    got = fp.estimate_3pcf_multipoles(*cat.arrays(), edges, 2, precision=precision, subtract_degenerate=False)
    assert np.all(rel_per_mu(got, oracle.upsilon3(*cat.arrays(), edges, 2, distinct=False)) < bar)
