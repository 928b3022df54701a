"""Transposed M2L and M2P on the independent (folded) coefficients: the rows of the others
follow by the harmonic relation, in the partial sets' sum where the taps are split and in
the translation itself where a level has so many source tiles that they are not (the
128^3 grid; its sources make 16384 tiles).  <t, A m> = <A^T t, m> for random t and m at
every order and in both forms.  Both sides are the plan's own, so the forms' truncation cancels:
what is left is the rounding of sums of N random terms, below sqrt(N) unit roundoffs of the
terms' norm times a factor of 100 for the depth of the sums.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

import paper_2607_19489_amd as A  # noqa: E402

from synth import shuffle_order  # noqa: E402
from synth.hierarchy import build_graded, refine_sphere, unigrid  # noqa: E402

GRADED = shuffle_order(build_graded(4, 6, refine_sphere((0.2, 0.15, 0.8), {4: 0.25, 5: 0.12})), 9)


def check(h, p, precision):
    plan = A.Plan(h, p=p, precision=precision, fp64_levels=2)
    rng = np.random.default_rng(p)
    leaf = torch.from_numpy(h.leaf_mask()).cuda()
    m = torch.from_numpy(rng.random(h.total)).cuda() * leaf
    tp = torch.from_numpy(rng.standard_normal(h.total)).cuda() * leaf
    ta = torch.from_numpy(rng.standard_normal((h.total, 3))).cuda() * leaf[:, None]
    phi, acc = plan.solve(m)
    phi, acc = phi * leaf, acc * leaf[:, None]
    mbar = plan.solve_adjoint(tp, ta)
    torch.cuda.synchronize()
    lhs = float((tp * phi).sum() + (ta * acc).sum())
    rhs = float((mbar * m).sum())
    scale = float(tp.norm() * phi.norm() + ta.norm() * acc.norm())
    eps = 2.2e-16 if precision == "fp64" else 1.2e-7
    plan.close()
    assert abs(lhs - rhs) <= 100 * eps * scale, (lhs, rhs, scale)


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("p", list(range(1, 9)))
def test_split_levels(p, precision):
    check(GRADED, p, precision)


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("p", [2, 5])
def test_a_level_without_split(p, precision):
    check(unigrid(7), p, precision)
