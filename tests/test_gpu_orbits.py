"""Intermediate field by orbits of sources that mirror one another.

A tile holds as many leaf groups of one parity class as its columns (48 or 64)
and its bound on the distinct refined fathers of their sources (200 or 240)
allow.  The cases end tiles in each way: a uniform grid in order (full tiles and a remainder;
every father shared with neighbouring columns), the same grid shuffled (the bound
on fathers), and a graded grid at the box's edge (missing and leaf sources, both
element types of a mixed plan).  Splits 3 and 21 cut the phases of 7 orbits
unevenly.  Every order and both forms against the FP64 oracle, at the gates of
the two forms; whole and split sums differ by rounding only.
"""
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from gpu_util import compare, gate  # noqa: E402

from synth import cell_masses, plummer, shuffle_order  # noqa: E402
from synth.hierarchy import build_graded, refine_sphere, unigrid  # noqa: E402

GRIDS = {"columns": unigrid(5), "fathers": shuffle_order(unigrid(5), 5),
         "edges": shuffle_order(build_graded(4, 6, refine_sphere((0.05, 0.1, 0.9), {4: 0.2, 5: 0.1})), 7)}


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("p", list(range(1, 9)))
@pytest.mark.parametrize("grid,split", [("columns", 0), ("fathers", 3), ("edges", 21)])
def test_tiles_and_splits(grid, split, p, precision):
    h = GRIDS[grid]
    m = cell_masses(h, plummer(1.0, 0.1), 0.01, 200 + p)
    compare(h, m, p, precision, gate(precision), tap_split=split, fp64_levels=4 if grid == "edges" else 2)
