"""The folded sums of the natural components at the edges of their plan: one
angular bin, odd and even counts (the middle bin is its own mirror), counts
around a wave of 64 bins and their mirrors, the smallest and largest nmax.

Tolerance, relative to the sum of |Upsilon| over the multipoles times the area
of an angular bin, which bounds the result: 64 roundings of the sums, and the
angular integrals, differences of sines of phases up to 2 pi nmax divided by m,
whose error of a few 2^-53 x 2 pi is 8 nphi roundings of a bin's width."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nmax,nphi", [(0, 1), (1, 2), (2, 3), (16, 7), (5, 127), (3, 128), (10, 129), (4, 256),
                                       (1, 259)])
@pytest.mark.parametrize("everything", [False, True])
def test_angular_bins(nmax, nphi, everything):
    import paper_2509_07974_amd as fp
    rng = np.random.default_rng(nmax * 1000 + nphi)
    nb, nn = 3, 2 * nmax + 1
    u = rng.standard_normal((9, nb, nb, nb, nn, nn)) + 1j * rng.standard_normal((9, nb, nb, nb, nn, nn))
    if everything:
        if nphi > 128:
            pytest.skip("the whole tensor at one size of each kind")
        trip = np.array([(a, b, c) for a in range(nb) for b in range(nb) for c in range(nb)], dtype=np.int32)
        g, n = fp.to_natural(u, nphi)
        g, n = np.asarray(g).reshape(8, len(trip), nphi, nphi), np.asarray(n).reshape(len(trip), nphi, nphi)
    else:
        trip = np.array([(2, 0, 1), (1, 1, 1), (0, 2, 2), (2, 0, 1), (0, 0, 0)], dtype=np.int32)
        g, n = fp.to_natural_triplets(u, nphi, trip)
    rg, rn = oracle.natural_components_triplets(u, nphi, trip)
    ub = np.abs(u)[:, trip[:, 0], trip[:, 1], trip[:, 2]].sum((-1, -2))[..., None, None] / nphi**2
    tol = (64 + 8 * nphi) * 2.0**-53
    assert g.shape == rg.shape and n.shape == rn.shape
    assert np.all(np.abs(n - rn) <= tol * ub[8])
    assert np.all(np.abs(g * n - rg * rn) <= 2 * tol * ub[:8])
