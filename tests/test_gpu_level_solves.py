"""Solves of one level by their own chain of local expansions.

Where M2L runs 32 groups per tile (FP32, p = 5 and 6) a chain of few tiles takes
tiles of 16.  A column's sum does not depend on its tile, so the leaves of a level solve
have the bits of the full solve's; those agree with the FP64 oracle.  p = 4 and 7 have one
width.  The splits are the automatic one, none and three ranges.
"""
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

import oracle  # noqa: E402
import paper_2607_19489_amd as A  # noqa: E402
from gpu_util import check_errors  # noqa: E402

from synth import cell_masses, plummer, shuffle_order  # noqa: E402
from synth.hierarchy import build_graded, refine_sphere  # noqa: E402

H = shuffle_order(build_graded(4, 7, refine_sphere((0.45, 0.5, 0.4), {4: 0.3, 5: 0.15, 6: 0.07})), 13)


@pytest.mark.parametrize("p", [4, 5, 6, 7])
@pytest.mark.parametrize("split", [0, 1, 3])
def test_level_solve_has_the_bits_of_the_full_solve(p, split):
    m = cell_masses(H, plummer(1.0, 0.1), 0.01, 700 + p)
    plan = A.Plan(H, p=p, precision="fp32", tap_split=split, fp64_levels=2)
    mt = torch.from_numpy(m).cuda()
    phi, acc = plan.solve(mt)
    po, ao = oracle.Oracle(H, p).solve_all(m)
    leaf = H.leaf_mask()
    check_errors(phi.cpu().numpy()[leaf], acc.cpu().numpy()[leaf], po[leaf], ao[leaf], "fp32", what=f"p={p} split={split}")
    level = torch.from_numpy(H.level_of()).cuda()
    for lev in range(H.levelmin + 1, H.levelmax + 1):
        at = torch.from_numpy(leaf).cuda() & (level == lev)
        p1, a1 = plan.solve(mt, level=lev)
        assert at.any() and torch.equal(p1[at], phi[at]) and torch.equal(a1[at], acc[at]), lev
    plan.close()
