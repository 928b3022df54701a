"""max_device_bytes: what a plan does in little memory.

The sets of partial sums of the automatic splits are the part of a plan that can be
smaller: a cap that holds the plan without splits holds the plan, and one that holds the
automatic splits leaves them as they are.  An adjoint that does not fit leaves the plan
as it was, however often it is asked for.
"""
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

import oracle  # noqa: E402
import paper_2607_19489_amd as A  # noqa: E402
from gpu_util import check_errors, gpu_solve  # noqa: E402

from synth import cell_masses, plummer  # noqa: E402
from synth.hierarchy import build_graded, refine_sphere, unigrid  # noqa: E402

GRIDS = {"uniform": unigrid(5), "graded": build_graded(4, 6, refine_sphere((0.45, 0.5, 0.55), {4: 0.25, 5: 0.12}))}


def need(h, p, precision, **kw):
    plan = A.Plan(h, p=p, precision=precision, **kw)
    n = plan.info()["device_bytes"]
    plan.close()
    return n


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("p", [1, 4, 5, 8])
@pytest.mark.parametrize("grid", list(GRIDS))
def test_fewer_sets_rather_than_no_plan(grid, p, precision):
    h = GRIDS[grid]
    m = cell_masses(h, plummer(1.0, 0.1), 0.01, 800 + p)
    least, full = need(h, p, precision, tap_split=1), need(h, p, precision)
    assert least < full
    po, ao = oracle.Oracle(h, p).solve_all(m)
    leaf = h.leaf_mask()
    free, _, _ = gpu_solve(h, m, p, precision)
    for cap in (least, (least + full) // 2, full):
        plan = A.Plan(h, p=p, precision=precision, max_device_bytes=cap)
        assert plan.info()["device_bytes"] <= cap
        phi, acc, _ = gpu_solve(h, m, p, plan=plan)
        check_errors(phi[leaf], acc[leaf], po[leaf], ao[leaf], precision, what=f"{grid} p={p} cap {cap}")
        if cap == full:
            assert (phi[leaf] == free[leaf]).all() and plan.info()["device_bytes"] == full
        plan.close()
    # (the tile lists of level solves depend a little on the splits, so `least` is not the last byte)
    with pytest.raises(A.AfmmError, match="max_device_bytes"):
        A.Plan(h, p=p, precision=precision, max_device_bytes=least // 2)


# the FP32 copy of the adjoint's D~ rows fits the first cap, both copies and the source tiles fit the second,
# which the bars exceed
@pytest.mark.parametrize("more", [2 << 20, 4 << 20])
def test_a_refused_adjoint_leaves_the_plan_as_it_was(more):
    h, p = unigrid(6), 6
    m = cell_masses(h, plummer(1.0, 0.1), 0.01, 900)
    plan = A.Plan(h, p=p, precision="fp32", max_device_bytes=need(h, p, "fp32") + more)
    mt = torch.from_numpy(m).cuda()
    phi, acc = plan.solve(mt)
    before = plan.info()["device_bytes"]
    for _ in range(3):
        with pytest.raises(A.AfmmError, match="max_device_bytes"):
            plan.solve_adjoint(phi, acc)
        assert plan.info()["device_bytes"] == before
    again, _ = plan.solve(mt)
    torch.cuda.synchronize()
    assert torch.equal(again, phi)
    plan.close()
