"""The reverse of a sub-stepped source, which runs as a kernel of its own
between the two that reverse the rest of a step: the dot-product identity of
test_gpu_adjoint_dot.py (same tolerance) in 3-D, with several reactions and
with none, and with a box whose cells end inside a block of threads."""
import pytest

from paper_2304_05657_amd import workloads as W

from .gpu_util import say
from .test_gpu_adjoint_dot import _dot_case

pytestmark = pytest.mark.gpu


def _reactions(n):
    return [W.Reaction([0, 1], 1e10 * 300.0 ** -(0.1 * j), 0.1 * j, 15000.0 + 500.0 * j, [-1.0, -4.0, 5.0, 0.0], 3.0e4)
            for j in range(n)]


@pytest.mark.parametrize("n_rx", [0, 1, 3])
@pytest.mark.parametrize("objective", ["wall_q", "flame_x"])
def test_dot_product_3d(n_rx, objective):
    prob = W.porous_3d(nx=21, ny=11, nz=9, porosity=0.9, radius=3.0, margin=4, front_x=10.0)
    prob = prob.replace(faces=("periodic",) * 6, reactions=_reactions(n_rx), chem_substeps_max=8)
    say("3-D, %d reactions, up to 8 sub-steps, %s" % (n_rx, objective))
    _dot_case(prob, objective, 6, seed=21 + n_rx)


def test_dot_product_2d():
    prob = W.channel_flame(nx=61, ny=15, front_x=20.0).replace(reactions=_reactions(2), chem_substeps_max=8)
    say("2-D, 2 reactions, up to 8 sub-steps")
    _dot_case(prob, "wall_q", 10, seed=31)
