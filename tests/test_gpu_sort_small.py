"""The sort of few pairs (up to 16384: every element's rank counted in one
launch), at its last size and the first of the radix passes, around a
workgroup's sixteen elements, with duplicates that only stability orders.
Results are exact."""
import numpy as np
import pytest

from helpers import ensure_built
from test_gpu_sort import _check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 15, 16, 17, 2000, 16383, 16384, 16385])
@pytest.mark.parametrize("bits,nbytes", [(3, 4), (16, 4), (32, 4), (5, 8), (64, 8)])
def test_sort_few_pairs(n, bits, nbytes):
    ensure_built()
    keys = np.random.default_rng(n * 100 + bits).integers(0, 2 ** bits - 1, n, dtype=np.uint64, endpoint=True)
    _check(keys, bits, nbytes)
