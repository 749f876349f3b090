"""The matrix-core pair kernel of stage (a) at the edges of its plan: record
orders where a row block begins or ends, catalogues around a multiple of eight
galaxies (its octets) and of a chunk, sparse and clustered cells, weights of
any scale and unevenness that it takes, and workspaces without room for its operands.

Tolerances: the mixed paths' bar of 1e-5 per correlator; per-centre multipoles
2e-6 of the largest block of their kind and bin, from 2^-22 per operand, a
phase error of order x 2^-24 and binary32 records."""
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


def check_blocks(fp, cat, edges, nmax):
    cen = np.arange(cat.n)[:: max(1, cat.n // 64)]
    ref = oracle.multipoles(*cat.arrays(), edges, nmax, cen)
    counts, G, W = fp.debug_multipoles(*cat.arrays(), edges, nmax, precision="fp16", centers=cen)
    assert np.array_equal(counts, ref["counts"])
    for got, fam, lo in ((G, "G", -2 * nmax - 3), (W, "W", -2 * nmax)):
        want = ref[fam][:, :, lo - ref["ranges"][fam][0]:][:, :, :got.shape[-1]]
        # weights of the bin bound every multipole of it
        amp = np.abs(cat.w if fam == "W" else cat.w * (cat.g1 + 1j * cat.g2))
        e2 = oracle.squared_edges(edges)
        for q, i in enumerate(cen):
            r2 = (cat.x - cat.x[i]) ** 2 + (cat.y - cat.y[i]) ** 2
            for b in range(len(edges) - 1):
                bound = amp[(r2 >= e2[b]) & (r2 < e2[b + 1])].sum()
                assert np.all(np.abs(got[q, b] - want[q, b]) <= 2e-6 * bound + 1e-30), (q, b, fam)


@pytest.mark.parametrize("nmax", [4, 5, 9, 10, 11, 14, 15, 16])
def test_orders(fp, nmax):
    check_blocks(fp, synth.uniform_catalogue(40 + nmax, 700, 40.0), synth.log_edges(1.0, 18.0, 3), nmax)


@pytest.mark.parametrize("n", [2, 7, 8, 9, 63, 64, 65, 129, 1031])
def test_sizes(fp, n):
    check_blocks(fp, synth.uniform_catalogue(n, n, 12.0), synth.log_edges(0.4, 9.0, 2), 5)


@pytest.mark.parametrize("side", [0.0, 3.0, 900.0])
def test_cells(fp, side):
    """All galaxies on a line, in few cells, and far apart."""
    cat = synth.uniform_catalogue(5, 500, 60.0)
    x = cat.x if side == 0.0 else cat.x * (side / 60.0)
    y = np.zeros_like(cat.y) if side == 0.0 else cat.y * (side / 60.0)
    cat = synth.Catalogue(x, y, cat.g1, cat.g2, cat.w)
    check_blocks(fp, cat, synth.log_edges(0.2, 30.0, 4), 6)


@pytest.mark.parametrize("scale_w,scale_g", [(1e-6, 1.0), (3e5, 1.0), (1.0, 1e-5), (1.0, 0.0)])
def test_scales(fp, scale_w, scale_g):
    cat = synth.uniform_catalogue(8, 600, 40.0)
    cat = synth.Catalogue(cat.x, cat.y, cat.g1 * scale_g, cat.g2 * scale_g, cat.w * scale_w)
    check_blocks(fp, cat, synth.log_edges(1.0, 18.0, 3), 5)


@pytest.mark.parametrize("outlier", [5.0, 20.0])
def test_uneven_weights(fp, outlier):
    """An outlier within 2^5 times the rms weight; zero and negative weights."""
    cat = synth.uniform_catalogue(9, 600, 40.0)
    w = cat.w.copy()
    w[17] *= outlier
    w[5:60:7] = 0.0
    w[100:140:9] *= -1.0
    cat = synth.Catalogue(cat.x, cat.y, cat.g1, cat.g2, w)
    edges = synth.log_edges(1.0, 18.0, 3)
    check_blocks(fp, cat, edges, 5)
    got = fp.estimate_4pcf_multipoles(*cat.arrays(), edges, 5, precision="fp16")
    assert np.all(rel_per_mu(got, oracle.upsilon(*cat.arrays(), edges, 5)) < 1e-5)


@pytest.mark.parametrize("m", [13, 14, 16, 22, 24, 26, 32])
def test_3pcf_orders(fp, m):
    """Records of order 7 (vector kernel), 8 (the smallest on the matrix cores),
    11, 12 (vector kernel), 13 and 16."""
    cat = synth.uniform_catalogue(60 + m, 500, 40.0)
    edges = synth.log_edges(1.0, 18.0, 4)
    got = fp.estimate_3pcf_multipoles(*cat.arrays(), edges, m, precision="fp16")
    ref = oracle.upsilon3(*cat.arrays(), edges, m)
    assert np.all(rel_per_mu(got, ref) < 1e-5)


def test_workspace_without_operands(fp):
    """A workspace that holds everything but the operands still serves."""
    import torch
    cat = synth.uniform_catalogue(3, 900, 40.0)
    edges = synth.log_edges(1.0, 18.0, 3)
    ref = fp.estimate_4pcf_multipoles(*cat.arrays(), edges, 5, precision="fp16")
    need, _ = fp.plan(cat.n, edges, 5, "fp16")
    least, _ = fp.plan(cat.n, edges, 5, "fp16", smallest=True)
    assert least < need
    ws = torch.empty(least, dtype=torch.uint8, device="cuda")
    r = fp.Request(*cat.arrays(), edges, 5, precision="fp16", workspace=ws)
    while r.step():
        pass
    got = r.finalize()
    r.close()
    assert np.all(rel_per_mu(got, ref) < 4e-6)
    with pytest.raises(fp.Fpcf4Error):
        fp.Request(*cat.arrays(), edges, 5, precision="fp16",
                   workspace=torch.empty(least - 256, dtype=torch.uint8, device="cuda"))


@pytest.mark.parametrize("precision,nmax", [("fp16", 6), ("fp16", 2), ("fp64", 3)])
@pytest.mark.parametrize("n", [1, 65, 700])
def test_listed_centres(fp, precision, nmax, n):
    """Listed centres are worked off in another order; blocks come as listed,
    those of the whole catalogue bit for bit."""
    cat = synth.uniform_catalogue(17, 700, 40.0)
    edges = synth.log_edges(1.0, 18.0, 3)
    cen = np.random.default_rng(n).permutation(700)[:n]
    whole = fp.debug_multipoles(*cat.arrays(), edges, nmax, precision=precision)
    got = fp.debug_multipoles(*cat.arrays(), edges, nmax, precision=precision, centers=cen)
    for a, b in zip(got, whole):
        assert np.array_equal(a, b[cen])
