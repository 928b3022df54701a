"""The mixed form's mass bars against the FP64 form's, leaf by leaf.

A single inner product hides an error in the FP32 rows, stages or first accumulators of
high orders under the size of its other terms; the relative L2 norm over the leaves
does not.  Every order on a graded grid, whose levels split their taps, and the 128^3 grid,
whose 16384 source tiles do not.  The bound is the forward pass's own for the
mixed form.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

import paper_2607_19489_amd as A  # noqa: E402
from gpu_util import FP32_REGRESSION  # noqa: E402

from synth import cell_masses, plummer, shuffle_order  # noqa: E402
from synth.hierarchy import build_graded, refine_sphere, unigrid  # noqa: E402

GRADED = shuffle_order(build_graded(4, 6, refine_sphere((0.2, 0.15, 0.8), {4: 0.25, 5: 0.12})), 9)


def check(h, p, seed):
    rng = np.random.default_rng(seed)
    leaf = torch.from_numpy(h.leaf_mask()).cuda()
    m = torch.from_numpy(cell_masses(h, plummer(1.0, 0.1), 0.01, seed)).cuda()
    tp = torch.from_numpy(rng.standard_normal(h.total)).cuda() * leaf
    ta = torch.from_numpy(rng.standard_normal((h.total, 3))).cuda() * leaf[:, None]
    bars = {}
    for precision in ("fp64", "fp32"):
        plan = A.Plan(h, p=p, precision=precision, fp64_levels=2)
        plan.solve(m)
        bars[precision] = plan.solve_adjoint(tp, ta)[leaf]
        torch.cuda.synchronize()
        plan.close()
    err = float((bars["fp32"] - bars["fp64"]).norm() / bars["fp64"].norm())
    print(f"{h.levelmin}..{h.levelmax} p={p}: {err:.1e}", flush=True)
    assert 0 < err <= FP32_REGRESSION


@pytest.mark.parametrize("p", list(range(1, 9)))
def test_split_levels(p):
    check(GRADED, p, 1000 + p)


@pytest.mark.parametrize("p", [5, 6, 8])
def test_a_level_without_split(p):
    check(unigrid(7), p, 1100 + p)
