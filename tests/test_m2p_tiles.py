"""Tiles of the intermediate field for groups near to and far from each other.

A staged tile takes groups of one parity class until its columns (48 or 64) or its
distinct refined fathers (200 or 240) run out; a level whose groups lie so far
apart that its staged tiles outnumber full ones 1.5 (2) times takes direct tiles of
16 to 64 columns.  replay() is that rule in a few lines.  On the CPU it shows that the
geometries reach what they are here for: tiles that end by fathers, with their table
close to full, in a level that stays staged (32^3 with 55% of its cells refined), and
direct tiles of one quad per wave and of several (16^3 and 32^3 with 10%).  On the GPU every
order and both forms agree with the FP64 oracle there; splits 3 and 21 begin
ranges of orbits inside a phase of 7 and inside a pass.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
import paper_2607_19489_amd as A  # noqa: E402
from gpu_util import check_errors, compare, gate, gpu_solve  # noqa: E402

from synth import cell_masses, plummer  # noqa: E402
from synth.hierarchy import build_graded  # noqa: E402


def scattered(base, share):
    on = np.random.default_rng(base).random((1 << base,) * 3) < share
    return build_graded(base, base + 1, lambda lev, ijk, h: on[tuple(ijk.T)] if lev == base else np.zeros(len(ijk), bool))


GRIDS = {"bound": scattered(5, 0.55), "narrow": scattered(4, 0.1), "wide": scattered(5, 0.1)}


def replay(h, columns, fathers):
    """Fathers of every staged tile of the finest level that ended by them, the number of staged tiles and of full ones."""
    c = h.ijk[0][h.refined[0].astype(bool)].astype(np.int64)
    bits = np.arange(h.levelmin)
    key = sum((((c[:, d, None] >> bits) & 1) << (3 * bits + d)).sum(1) for d in range(3))
    c = c[np.argsort(key)]
    top = (1 << (h.levelmin - 1)) - 1
    ended, staged, full = [], 0, 0
    for octant in range(8):
        cls = c[((c & 1) * [1, 2, 4]).sum(1) == octant] >> 1  # the groups' fathers; every cell of their level is refined
        full += -(-len(cls) // columns)
        n, have = 0, set()
        for g in cls:
            lo, hi = np.maximum(g - 1, 0), np.minimum(g + 1, top)
            near = {(x, y, z) for x in range(lo[0], hi[0] + 1) for y in range(lo[1], hi[1] + 1) for z in range(lo[2], hi[2] + 1)}
            if n == columns or len(have | near) > fathers:
                if n < columns:
                    ended.append(len(have))
                staged, n, have = staged + 1, 0, set()
            n, have = n + 1, have | near
        staged += n > 0
    return ended, staged, full


@pytest.mark.parametrize("columns,fathers,line", [(48, 200, 1.5), (64, 240, 2.0)])
def test_the_geometries_reach_their_tiles(columns, fathers, line):
    ended, staged, full = replay(GRIDS["bound"], columns, fathers)
    assert staged <= line * full and len(ended) > 100 and max(ended) >= fathers - 2
    for name, quads in (("narrow", 1), ("wide", 2)):
        ended, staged, full = replay(GRIDS[name], columns, fathers)
        assert staged > line * full, (name, staged, full)
        assert min(columns // 16, max(1, int(GRIDS[name].refined[0].sum()) // (6 * 256))) == quads


@pytest.mark.gpu
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("p", list(range(1, 9)))
@pytest.mark.parametrize("grid,split", [("bound", 3), ("narrow", 21), ("narrow", 0), ("wide", 3)])
def test_against_oracle(grid, split, p, precision):
    h = GRIDS[grid]
    m = cell_masses(h, plummer(1.0, 0.1), 0.01, 500 + p)
    compare(h, m, p, precision, gate(precision), sample=400, tap_split=split, fp64_levels=2)


@pytest.mark.gpu
@pytest.mark.parametrize("periodic", [False, True])
@pytest.mark.parametrize("p", [3, 4, 6, 7])
def test_direct_tiles_have_the_bits_of_staged_ones(p, periodic):
    # far apart alone, the first plan's groups take direct tiles; beside the groups of a dense grid,
    # in a batch, the level is staged: one sum, in one order
    hs = [GRIDS["narrow"], scattered(4, 1.0)]
    ms = [cell_masses(h, plummer(1.0, 0.1), 0.01, 600 + i) for i, h in enumerate(hs)]
    plans = [A.Plan(h, p=p, precision="fp32", tap_split=2, fp64_levels=2, periodic=periodic) for h in hs]
    masses = [torch.from_numpy(m).cuda() for m in ms]
    ind = [q.solve(mt) for q, mt in zip(plans, masses)]
    phis, accs = A.Batch(plans).solve(masses)
    torch.cuda.synchronize()
    for h, (p0, a0), p1, a1 in zip(hs, ind, phis, accs):
        leaf = torch.from_numpy(h.leaf_mask()).cuda()
        assert torch.equal(p0[leaf], p1[leaf]) and torch.equal(a0[leaf], a1[leaf])


@pytest.mark.gpu
@pytest.mark.parametrize("p", [3, 6, 8])
def test_direct_tiles_of_a_periodic_box(p):
    # neighbours and their children wrap round the box.  FP64: the potential of nearly even
    # masses is a hundredth of a monopole's, so the mixed form's gate says little here; its bits are above
    h = GRIDS["narrow"]
    m = np.random.default_rng(p).uniform(0.2, 1.0, h.total) / 8.0 ** (h.level_of() - h.levelmin)
    o = oracle.Oracle(h, p, periodic=True)
    po, ao = o.solve_all(m)
    o.close()
    leaf = h.leaf_mask()
    phi, acc, plan = gpu_solve(h, m, p, "fp64", periodic=True, tap_split=2)
    plan.close()
    check_errors(phi[leaf], acc[leaf], po[leaf], ao[leaf], "fp64", what=f"periodic p={p}")
