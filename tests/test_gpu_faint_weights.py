"""Regions whose weights are far below those of the rest of the catalogue, in
the mixed paths: centres there see only faint neighbours, and their sums of
squares and cubes (the same-galaxy terms) have to keep binary32's relative
accuracy.  The octets of the matrix-core pair kernel hold such weights in too
few bits; the vector kernel serves these catalogues.

Tolerance: the mixed paths' bar of 1e-5 per correlator."""
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


@pytest.mark.parametrize("faint_w,faint_g", [(1e-3, 1.0), (1e-4, 1.0), (1.0, 1e-3), (0.02, 1.0)])
@pytest.mark.parametrize("nmax", [5, 12])
def test_faint_half(fp, faint_w, faint_g, nmax):
    cat = synth.uniform_catalogue(21, 3000, 60.0)
    low = cat.x < 30.0
    cat = synth.Catalogue(cat.x, cat.y, cat.g1 * np.where(low, faint_g, 1.0), cat.g2 * np.where(low, faint_g, 1.0),
                          cat.w * np.where(low, faint_w, 1.0))
    cen = np.flatnonzero((cat.x < 18.0) & (np.abs(cat.y - 30.0) < 15.0))[::8]
    edges = synth.log_edges(0.4, 11.0, 3)
    got = fp.estimate_4pcf_multipoles(*cat.arrays(), edges, nmax, precision="fp16", centers=cen)
    ref = oracle.upsilon(*cat.arrays(), edges, nmax, cen)
    assert np.all(rel_per_mu(got, ref) < 1e-5), rel_per_mu(got, ref)


def test_faint_half_tree(fp):
    """The same on reduced catalogues, against the tree oracle."""
    cat = synth.uniform_catalogue(22, 3000, 60.0)
    w = cat.w * np.where(cat.x < 30.0, 1e-3, 1.0)
    cat = synth.Catalogue(cat.x, cat.y, cat.g1, cat.g2, w)
    cen = np.flatnonzero((cat.x < 18.0) & (np.abs(cat.y - 30.0) < 15.0))[::8]
    edges = synth.log_edges(0.4, 11.0, 4)
    got = fp.estimate_4pcf_multipoles(*cat.arrays(), edges, 5, precision="fp16", centers=cen, tree=(0.25, 2, 4.0))
    ref = oracle.upsilon_tree(*cat.arrays(), edges, 5, 0.25, 2, 4.0, centers=cen)
    assert np.all(rel_per_mu(got, ref) < 1e-5), rel_per_mu(got, ref)


def test_faint_half_3pcf(fp):
    cat = synth.uniform_catalogue(23, 3000, 60.0)
    w = cat.w * np.where(cat.x < 30.0, 1e-4, 1.0)
    cat = synth.Catalogue(cat.x, cat.y, cat.g1, cat.g2, w)
    cen = np.flatnonzero((cat.x < 18.0) & (np.abs(cat.y - 30.0) < 15.0))[::4]
    edges = synth.log_edges(0.4, 11.0, 4)
    got = fp.estimate_3pcf_multipoles(*cat.arrays(), edges, 22, precision="fp16", centers=cen)
    ref = oracle.upsilon3(*cat.arrays(), edges, 22, cen)
    assert np.all(rel_per_mu(got, ref) < 1e-5), rel_per_mu(got, ref)
