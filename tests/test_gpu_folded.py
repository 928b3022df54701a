"""Folded (harmonic) expansions: M2L forms the (p + 1)^2 coefficients with c <= 1
and the completion kernel the others, in place in the rows of L when the taps
are not split (also at the first level, which has no father's expansion to
add), or from the partial sets.  Every order and both forms against the FP64
oracle, at the gates of the two forms.
"""
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from gpu_util import compare, gate  # noqa: E402

from synth import cell_masses, plummer, shuffle_order  # noqa: E402
from synth.hierarchy import build_graded, refine_sphere  # noqa: E402

H = shuffle_order(build_graded(3, 6, refine_sphere((0.45, 0.5, 0.55), {3: 0.4, 4: 0.25, 5: 0.12})), 3)


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("p", list(range(1, 9)))
@pytest.mark.parametrize("split", [1, 21])
def test_every_order_in_place_and_split(p, precision, split):
    m = cell_masses(H, plummer(1.0, 0.1), 0.01, 100 + p)
    # fp64_levels = 2: the FP32 kernels run from the first level with expansions
    compare(H, m, p, precision, gate(precision), tap_split=split, fp64_levels=2)
