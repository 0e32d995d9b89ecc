"""The reverse sweep's reading of the cells' codes (pull sources, stencil
points, ghost images, walls) at the geometries where it can go wrong: boxes
of one to five cells along an axis, wrapped and walled, single-cell solids,
inlets in front of solid mirror cells.  Against the forward-mode step, which
classifies every neighbour on the fly: <J dx, lam> = <dx, J^T lam>.

Tolerance: both sides are sums of products whose factors carry the rounding
of some hundred FP64 operations: 1e-12 of the sum of the products'
magnitudes."""
import numpy as np
import pytest

from .gpu_util import need_gpu, say
from .test_gpu_adjoint_dot import _blocks_in
from .test_gpu_tiles2d import _box as box2
from .test_gpu_tiles3d import _box as box3

pytestmark = pytest.mark.gpu

PERIODIC = ("periodic",) * 6
CLOSED2 = ("wall", "wall", "wall_adiabatic", "wall", "periodic", "periodic")
CLOSED3 = ("wall", "wall", "wall_adiabatic", "wall", "wall", "wall_adiabatic")
INLET = ("inflow", "wall", "periodic", "periodic", "periodic", "periodic")
INLETS = ("wall", "inflow", "inflow", "wall_adiabatic", "periodic", "periodic")


@pytest.mark.parametrize("nx,ny,nz,faces", [
    (65, 9, 1, PERIODIC), (2, 2, 1, PERIODIC), (67, 5, 1, CLOSED2), (5, 1, 1, CLOSED2), (1, 6, 1, CLOSED2),
    (66, 7, 1, INLET), (9, 4, 1, INLETS),
    (17, 5, 3, PERIODIC), (2, 2, 2, PERIODIC), (18, 4, 5, CLOSED3), (5, 1, 2, CLOSED3), (19, 3, 4, INLET),
    (9, 6, 5, INLETS),
])
@pytest.mark.parametrize("objective", ["wall_q", "flame_x"])
def test_dot_product(nx, ny, nz, faces, objective):
    from paper_2304_05657_amd.lbfd import Solver
    need_gpu()
    p = box2(nx, ny, faces) if nz == 1 else box3(nx, ny, nz, faces)
    say("case dot product %dx%dx%d %s %s" % (nx, ny, nz, faces, objective))
    s = Solver(p)
    s.set_objective(objective)
    s.step(2)
    Q, N, nsp = p.lattice, s.N, p.n_species
    rng = np.random.default_rng(5)
    fluid = p.mask.ravel() == 0
    lp, ls = rng.standard_normal((Q, N)) * fluid, rng.standard_normal((1 + nsp, N)) * fluid
    wq = float(rng.standard_normal())
    adj = s.step_adjoint(lp, ls, wq)
    for name, block in _blocks_in(rng, p, Q, N, nsp).items():
        po, so, dq = s.step_tangent(*block)
        out = [po * lp, so * ls, np.array([wq * dq])]
        inn = [d * g for d, g in zip(block, adj) if d is not None]
        lhs, rhs = (sum(float(t.sum()) for t in v) for v in (out, inn))
        scale = max(sum(float(np.abs(t).sum()) for t in v) for v in (out, inn))
        assert abs(lhs - rhs) <= 1e-12 * scale, (name, lhs, rhs, scale)
