"""How the work is cut: centre slices of the contraction at small tiles (up to
one per 128 centres; counts around where one is added and where the last would
be empty), and the passes of the binary64 pair kernel (orders at which their
number changes).

Tolerances: the bars of the precisions, 1e-10 and 1e-5 per correlator, on raw
sums; per-centre multipoles in binary64 1e-13 of the sum of the weights of their
bin: order 40 times a few 2^-53 per power, and the sum's roundings."""
import numpy as np
import pytest

import oracle
import synth
from helpers import rel_per_mu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [127, 128, 256, 257, 1030])
@pytest.mark.parametrize("precision,bar", [("fp64", 1e-10), ("fp16", 1e-5), ("bf16", 1e-5)])
def test_slices(n, precision, bar):
    import paper_2509_07974_amd as fp
    cat = synth.uniform_catalogue(n, n, 30.0)
    edges = synth.log_edges(1.0, 18.0, 3)
    got = fp.estimate_4pcf_multipoles(*cat.arrays(), edges, 1, precision=precision, subtract_degenerate=False)
    assert np.all(rel_per_mu(got, oracle.upsilon(*cat.arrays(), edges, 1, distinct=False)) < bar)


@pytest.mark.parametrize("nmax", [2, 3, 4, 5, 8, 10, 12, 13, 16])
def test_binary64_passes(nmax):
    import paper_2509_07974_amd as fp
    cat = synth.uniform_catalogue(nmax, 500, 40.0)
    edges = synth.log_edges(1.0, 18.0, 3)
    cen = np.arange(0, cat.n, 9)
    ref = oracle.multipoles(*cat.arrays(), edges, nmax, cen)
    counts, G, W = fp.debug_multipoles(*cat.arrays(), edges, nmax, precision="fp64", centers=cen)
    assert np.array_equal(counts, ref["counts"])
    r2 = (cat.x[None] - cat.x[cen][:, None]) ** 2 + (cat.y[None] - cat.y[cen][:, None]) ** 2
    e2 = oracle.squared_edges(edges)
    for got, fam, lo in ((G, "G", -2 * nmax - 3), (W, "W", -2 * nmax)):
        want = ref[fam][:, :, lo - ref["ranges"][fam][0]:][:, :, :got.shape[-1]]
        amp = np.abs(cat.w if fam == "W" else cat.w * (cat.g1 + 1j * cat.g2))
        for b in range(3):
            bound = (((r2 >= e2[b]) & (r2 < e2[b + 1])) * amp).sum(1)
            assert np.all(np.abs(got[:, b] - want[:, b]) <= 1e-13 * bound[:, None] + 1e-300), (fam, b)
