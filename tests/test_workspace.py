"""Workspace sizes: what a plan reserves, and what an estimate falls back to
when the device has no room for it (host logic, no GPU)."""
import os
import shutil
import subprocess

import numpy as np
import pytest

from helpers import ROOT, ensure_built

EDGES = np.geomspace(1.0, 50.0, 5)


@pytest.fixture(scope="module")
def fp():
    ensure_built()
    import paper_2509_07974_amd as m
    return m


def extra(fp, n, nmax, precision, **kw):
    return fp.plan(n, EDGES, nmax, precision, **kw)[0] - fp.plan(n, EDGES, nmax, precision, smallest=True, **kw)[0]


def test_operands_reserved_where_they_serve(fp):
    """96 bytes per galaxy for the matrix-core pair kernel, which takes
    catalogues of fewer than 2^25 galaxies."""
    kw = {"tile_centers": 64}     # one slice of the contraction
    below, above = 2 ** 25 - 8, 2 ** 25
    assert abs(extra(fp, below, 8, "fp16", **kw) - 96 * below) < 4096
    assert extra(fp, above, 8, "fp16", **kw) < 4096
    assert extra(fp, below, 8, "fp64", **kw) < 4096


def test_extra_slices_reserved_once(fp):
    """One slice of the contraction at least; two fill the chip at 256 centres,
    three at 384, and the first is not reserved again for them."""
    one, two = (extra(fp, n, 3, "fp64") for n in (256, 384))
    assert one > 0 and abs(two - 2 * one) <= 1024


# (n, nbins, nmax, precision, centres): bytes planned before there were smallest sizes
SAVED = [((0, 1, 0, "fp64", None), 290048), ((1, 1, 0, "fp16", None), 287744), ((100, 4, 3, "fp64", 7), 1868288),
         ((2000, 4, 3, "fp16", None), 9961984), ((2000, 12, 10, "fp16", 7), 165670400),
         ((30000, 12, 8, "fp64", None), 1826300160), ((1000000, 12, 10, "fp64", None), 68465752064)]


@pytest.mark.parametrize("case,saved", SAVED)
def test_saved_sizes_still_serve(fp, case, saved):
    """A program that keeps a workspace of a size planned earlier."""
    n, nb, nmax, precision, cen = case
    least, _ = fp.plan(n, np.geomspace(1, 50, nb + 1), nmax, precision, ncenters=cen, smallest=True)
    assert least <= saved


PROGRAM = """
#include <cstdio>
#include "workspace.hpp"
int main() {
  // bytes that the device has, status 2 = no memory, 5 = another failure
  struct Case { std::size_t have; int other; } cases[] = {{100, 0}, {60, 0}, {10, 0}, {100, 5}};
  for (auto c : cases) {
    std::size_t bytes = 0;
    int asked = 0;
    int st = fpcf4::reserve(std::size_t(80), std::size_t(50), 2, [&](std::size_t b) {
      ++asked;
      return c.other ? c.other : b <= c.have ? 0 : 2;
    }, &bytes);
    std::printf("%d %zu %d\\n", st, bytes, asked);
  }
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host compiler")
def test_smallest_size_where_the_planned_one_does_not_fit(tmp_path):
    src = tmp_path / "t.cpp"
    src.write_text(PROGRAM)
    exe = tmp_path / "t"
    subprocess.run(["g++", "-std=c++17", "-I", os.path.join(ROOT, "paper_2509_07974_amd", "csrc"), str(src), "-o",
                    str(exe)], check=True)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.split("\n")[:-1]
    assert out == ["0 80 1", "0 50 2", "2 50 2", "5 80 1"]


@pytest.mark.gpu
def test_parts_of_a_workspace(fp):
    """Bytes between the smallest and the planned size serve what fits them: a
    workspace without room for the centre order still holds the operands of
    the pair kernel (the same records, bit for bit), the smallest one does not."""
    import torch
    import synth
    cat = synth.uniform_catalogue(31, 700, 40.0)
    edges = synth.log_edges(1.0, 18.0, 3)
    cen = np.random.default_rng(1).permutation(700)[:200]

    def run(take_off):
        need, _ = fp.plan(cat.n, edges, 6, "fp16", ncenters=200)
        least, _ = fp.plan(cat.n, edges, 6, "fp16", ncenters=200, smallest=True)
        ws = torch.empty(least if take_off is None else need - take_off, dtype=torch.uint8, device="cuda")
        r = fp.Request(*cat.arrays(), edges, 6, precision="fp16", centers=cen, workspace=ws)
        while r.step():
            pass
        out = r.finalize()
        r.close()
        return out

    whole = run(0)
    assert np.array_equal(run(512), whole)
    assert not np.array_equal(run(None), whole)
