"""Seams between tiles that the tile tests' boxes do not reach: 2-D boxes of
several 16 x 16 tiles in both axes (one cell short of, at and past a tile), so
that halos, wraps, inlet ghosts and single-cell solids lie on seams in y; 3-D
boxes whose tile order has several bands in y with a ragged last one, with the
diagnostics' sums, which a skipped or doubled tile would change; and lists of
curved-wall links and image points that name some ghosts of a wave and not
others.  Against the oracle; tolerances as in test_gpu_tiles2d.py (FP64:
rounding order only)."""
import numpy as np
import pytest

from paper_2304_05657_amd import workloads as W

from .gpu_util import compare_fields, need_gpu, oracle_threads, say
from .test_gpu_tiles2d import CLOSED, DUCT, INLETS, PERIODIC, _box as box2d
from .test_gpu_tiles3d import CLOSED as CLOSED3, DUCT as DUCT3, _box as box3d

pytestmark = pytest.mark.gpu

TOL = {"fp64": 1e-10, "fp32": 5e-3, "fp16": 5e-2}


def _compare(p, precision, steps, links=None, images=None):
    import oracle
    from paper_2304_05657_amd.lbfd import Solver
    tol = TOL[precision]
    g, o = Solver(p, precision=precision, check_every=2), oracle.Oracle(p, threads=oracle_threads())
    if links is not None:
        g.set_wall_links(*links)
        o.set_wall_links(links[0], links[1], links[2].astype(np.float32).astype(np.float64))
    if images is not None:
        g.set_image_points(*images)
        o.set_image_points(*images)
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


@pytest.mark.parametrize("faces", [PERIODIC, DUCT, CLOSED, INLETS], ids=["periodic", "duct", "closed", "inlets"])
@pytest.mark.parametrize("nx,ny", [(15, 33), (16, 17), (17, 16), (33, 15), (31, 32), (32, 47), (49, 34)])
def test_2d(nx, ny, faces):
    need_gpu()
    say("2-D seams %dx%d %s" % (nx, ny, faces))
    _compare(box2d(nx, ny, faces, seed=nx * ny), "fp64", 6)


@pytest.mark.parametrize("precision", ["fp32", "fp16"])
@pytest.mark.parametrize("nx,ny,faces", [(33, 47, DUCT), (17, 33, INLETS)])
def test_2d_mixed(nx, ny, faces, precision):
    need_gpu()
    say("2-D seams %dx%d %s" % (nx, ny, precision))
    _compare(box2d(nx, ny, faces), precision, 6)


@pytest.mark.parametrize("nx,ny,nz,faces", [(65, 71, 3, PERIODIC), (65, 33, 5, CLOSED3), (40, 67, 4, DUCT3)])
def test_3d_bands(nx, ny, nz, faces):
    need_gpu()
    say("3-D bands %dx%dx%d" % (nx, ny, nz))
    _compare(box3d(nx, ny, nz, faces), "fp64", 4)


@pytest.mark.parametrize("kind", ["2d", "3d", "3d-9-species", "3d-mixture"])
@pytest.mark.parametrize("part", [0.05, 0.5])
def test_partial_lists(kind, part):
    need_gpu()
    if kind == "2d":
        p = W.cylinder_burner(nx=200, ny=64, radius=9.0, pitch=32, x_begin=40, x_end=160, front_x=100.0)
    elif kind == "3d-9-species":
        p = W.porous_3d_mech(nx=100, ny=20, nz=18, porosity=0.85, radius=(3.0, 5.0), margin=8)
    else:
        p = W.porous_3d(nx=100, ny=20, nz=18, porosity=0.85, radius=4.0, margin=8, seed=7)
        if kind == "3d-mixture":
            p = W.mixture_transport(p)
    rng = np.random.default_rng(11)
    lk, im = W.wall_links(p), W.image_points(p)
    a, b = rng.random(len(lk[0])) < part, rng.random(len(im[0])) < part
    say("%s: %d of %d links, %d of %d image points" % (kind, a.sum(), a.size, b.sum(), b.size))
    _compare(p, "fp64", 5, tuple(v[a] for v in lk), tuple(v[b] for v in im))
