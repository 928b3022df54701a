"""M2L by orbits of sources that mirror one another (from p = 5).

A tile holds 32 (FP32 to p = 6) or 16 groups of one parity class.  The uniform grid
fills tiles; the shuffled graded grid leaves a remainder in every class and has missing and
leaf sources in one orbit; the small grid gives tiles of a single column.  fp64_levels
2 and 3 put the first levels on either form.  Splits 1 (sums in place), 5 and 21 (ranges of 11
and 2 or 3 orbits, an odd and an even number for the two LDS buffers) against the FP64
oracle at the gates of the two forms, and a batch against its members' own plans bit
by bit (their tiles differ).
"""
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

import paper_2607_19489_amd as A  # noqa: E402
from gpu_util import compare, gate  # noqa: E402

from synth import cell_masses, plummer, shuffle_order  # noqa: E402
from synth.hierarchy import build_graded, refine_sphere, unigrid  # noqa: E402

GRIDS = {"full": unigrid(5), "small": unigrid(4),
         "graded": shuffle_order(build_graded(4, 6, refine_sphere((0.1, 0.2, 0.85), {4: 0.25, 5: 0.12})), 11)}


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("p", [4, 5, 6, 7, 8])
@pytest.mark.parametrize("grid,split,levels", [("full", 1, 2), ("small", 21, 2), ("graded", 5, 3)])
def test_tiles_and_splits(grid, split, levels, p, precision):
    h = GRIDS[grid]
    m = cell_masses(h, plummer(1.0, 0.1), 0.01, 300 + p)
    compare(h, m, p, precision, gate(precision), tap_split=split, fp64_levels=levels)


@pytest.mark.parametrize("p", [5, 8])
def test_batch_has_the_bits_of_its_plans(p):
    hs = [GRIDS["graded"], GRIDS["small"]]
    ms = [cell_masses(h, plummer(1.0, 0.1), 0.01, 400 + i) for i, h in enumerate(hs)]
    plans = [A.Plan(h, p=p, precision="fp32", tap_split=3, fp64_levels=2) for h in hs]
    masses = [torch.from_numpy(m).cuda() for m in ms]
    ind = [q.solve(mt) for q, mt in zip(plans, masses)]
    batch = A.Batch(plans)
    phis, accs = batch.solve(masses)
    torch.cuda.synchronize()
    for h, (p0, a0), p1, a1 in zip(hs, ind, phis, accs):
        leaf = torch.from_numpy(h.leaf_mask()).cuda()
        assert torch.equal(p0[leaf], p1[leaf]) and torch.equal(a0[leaf], a1[leaf])
