"""The tiles of thin boxes (64 x 4 cells in 2-D, 8 x 8 x 4 in 3-D) at the sizes
where their indexing can go wrong: one cell short of, at and past a tile in
each axis, boxes thinner than the stencil, several bands of the 3-D tile order
with a ragged last one, every face kind, single-cell solids; and the switch of
a thin box to the ordinary tiles and back when curved walls are set and
cleared.  Sizes are past the line from which such a box takes these tiles
(lbfd_api.hip).  Against the oracle; tolerances as in test_gpu_tiles2d.py."""
import numpy as np
import pytest

from paper_2304_05657_amd import workloads as W

from .gpu_util import compare_fields, need_gpu, oracle_threads, say
from .test_gpu_tiles2d import CLOSED, DUCT, INLETS, PERIODIC, TUBE, _box as box2d
from .test_gpu_tiles3d import CLOSED as CLOSED3, DUCT as DUCT3, INLETS as INLETS3, _box as box3d

pytestmark = pytest.mark.gpu

TOL = {"fp64": 1e-10, "fp32": 5e-3, "fp16": 5e-2}


def _compare(p, precision, steps, what):
    import oracle
    from paper_2304_05657_amd.lbfd import Solver
    say("%s %dx%dx%d" % (what, p.nx, p.ny, p.nz))
    tol = TOL[precision]
    g, o = Solver(p, precision=precision, check_every=2), oracle.Oracle(p, threads=oracle_threads())
    g.step(steps)
    o.step(steps)
    g.sync()
    keys = ("u", "T", "Y", "Ph", "rho") if precision == "fp64" else ("u", "T", "Y", "rho")
    e = compare_fields(g.fields(), o.fields(), p, keys=keys)
    assert max(e.values()) <= tol, e
    dg, do = g.diagnostics(), o.diagnostics()
    for k in ("sum_theta", "wall_q", "fuel_rate"):
        assert abs(dg[k] - do[k]) <= tol * max(abs(do[k]), 1e-12), (k, dg[k], do[k])
    g.close()


@pytest.mark.parametrize("nx,ny,faces", [
    (12321, 1, DUCT), (12353, 2, PERIODIC), (12415, 3, TUBE), (12351, 4, CLOSED), (12417, 5, INLETS),
    (6271, 17, PERIODIC), (6273, 18, DUCT), (6337, 20, INLETS), (6272, 19, CLOSED),
])
@pytest.mark.parametrize("precision", ["fp64", "fp32", "fp16"])
def test_2d(nx, ny, faces, precision):
    need_gpu()
    _compare(box2d(nx, ny, faces), precision, 4, "2-D %s" % precision)


@pytest.mark.parametrize("nx,ny,nz,faces", [
    (1, 9, 13, CLOSED3), (2, 15, 5, PERIODIC), (4, 16, 12, DUCT3), (5, 17, 9, INLETS3), (7, 33, 4, PERIODIC),
    (8, 131, 11, PERIODIC), (9, 137, 131, DUCT3), (31, 72, 63, INLETS3),
])
@pytest.mark.parametrize("precision", ["fp64", "fp16"])
def test_3d(nx, ny, nz, faces, precision):
    need_gpu()
    _compare(box3d(nx, ny, nz, faces), precision, 4, "3-D %s" % precision)


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_3d_mechanism(precision):
    need_gpu()
    _compare(box3d(5, 18, 13, DUCT3, mech=True), precision, 4, "3-D 9 species %s" % precision)


def test_mixture_transport():
    need_gpu()
    _compare(W.mixture_transport(box2d(12353, 3, CLOSED)), "fp64", 4, "2-D mixture transport")
    _compare(W.mixture_transport(box3d(6, 17, 9, DUCT3)), "fp64", 4, "3-D mixture transport")


def test_curved_walls_set_and_cleared():
    """Links at their half-way distance (1/2) change no value: the box with
    them (ordinary tiles), with them cleared again and without them agree to
    rounding, states and reductions."""
    need_gpu()
    from paper_2304_05657_amd.lbfd import Solver
    p = box3d(7, 33, 13, PERIODIC)
    links = _half_links(p)
    a, b = Solver(p), Solver(p)
    b.set_wall_links(*links)
    for s in (a, b):
        s.step(3)
    d = [s.diagnostics() for s in (a, b)]
    b.set_wall_links()
    for s in (a, b):
        s.step(3)
    d += [s.diagnostics() for s in (a, b)]
    e = compare_fields(b.fields(), a.fields(), p)
    assert max(e.values()) <= 1e-12, e
    for x, y in ((d[0], d[1]), (d[2], d[3])):
        for k in ("sum_theta", "wall_q", "fuel_rate", "sum_g"):
            assert abs(x[k] - y[k]) <= 1e-12 * max(abs(x[k]), 1e-12), (k, x[k], y[k])


def _half_links(p):
    """Every link of a fluid cell to a solid one, met half-way."""
    cell, direction = [], []
    mask = p.mask
    for z, y, x in np.argwhere(mask == 0):
        for d in range(27):
            c = (d % 3 - 1, d // 3 % 3 - 1, d // 9 - 1)
            if mask[(z + c[2]) % p.nz, (y + c[1]) % p.ny, (x + c[0]) % p.nx] != 0:
                cell.append((z * p.ny + y) * p.nx + x)
                direction.append(d)
    return np.array(cell, dtype=np.int64), np.array(direction, dtype=np.int32), np.full(len(cell), 0.5)
