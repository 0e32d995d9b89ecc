"""Outflow faces of boxes one cell wide in x: no cell has an inner neighbour,
so the outlet sets no population and the outflow face acts as a wall for the
populations.  Heights below, at and past a tile of the 2-D step, every kind of
opposite face, 2-D and 3-D, with and without diagnostics, against the oracle
(FP64; the tolerance of test_gpu_tiles2d.py: the two sides differ by rounding
order only)."""
import numpy as np
import pytest

from paper_2304_05657_amd import workloads as W

from .gpu_util import compare_fields, need_gpu, oracle_threads, say

pytestmark = pytest.mark.gpu


def _column(ny, nz, xfaces):
    base = W.channel_flame(nx=40, ny=8) if nz == 1 else W.porous_3d(nx=40, ny=4, nz=4)
    shape = (nz, ny, 1)
    rng = np.random.default_rng(5)
    mask = rng.choice([0, 1, 2], size=shape, p=[0.9, 0.07, 0.03]).astype(np.uint8)
    mask[0, 0, 0] = mask[-1, -1, 0] = 0  # the first and the last cell of the box are fluid
    th = rng.uniform(0.0, 1.0, shape)
    Y0 = np.stack([(1.0 - 0.5 * th) * a + 0.5 * th * b for a, b in zip(base.Y_in, W.Y_BURNT_STOICH)])
    u0 = np.where(mask == 0, rng.uniform(-0.01, 0.01, (3,) + shape), 0.0)
    if nz == 1:
        u0[2] = 0.0
    return base.replace(nx=1, ny=ny, nz=nz, faces=xfaces + ("wall", "wall_adiabatic") + (
        ("periodic",) * 2 if nz == 1 else ("wall_adiabatic", "wall")), face_T=(510.0, 520.0, 530.0, 540.0, 550.0, 560.0),
        mask=mask, wall_T=np.full(shape, 500.0), T0=600.0 + 200.0 * th, Y0=Y0, u0=u0, T_in=600.0, u_in=(0.01, 0.0, 0.0),
        notes={})


@pytest.mark.parametrize("xfaces", [("inflow", "outflow"), ("outflow", "inflow"), ("wall", "outflow"),
                                    ("outflow", "wall_adiabatic"), ("outflow", "outflow")])
@pytest.mark.parametrize("ny,nz", [(1, 1), (6, 1), (16, 1), (33, 1), (5, 3)])
def test_outflow_without_inner_cell(ny, nz, xfaces):
    import oracle
    from paper_2304_05657_amd.lbfd import Solver
    need_gpu()
    p = _column(ny, nz, xfaces)
    say("1x%dx%d %s | %s" % (ny, nz, *xfaces))
    g, o = Solver(p, check_every=2), oracle.Oracle(p, threads=oracle_threads())
    g.step(5)
    o.step(5)
    g.sync()
    e = compare_fields(g.fields(), o.fields(), p)
    assert max(e.values()) <= 1e-10, e
    g.close()
