"""3-D tiles of the step (64 x 2 x 2 cells, every fluid cell in its tile) at
the sizes where their indexing can go wrong: boxes one cell short of, at and
past a tile in each axis, boxes thinner than the +-2 stencil, every face
kind next to ragged tiles, single-cell solids against faces.  FP64 against the oracle.

Tolerance: the two sides differ by rounding order only (see
test_gpu_parity.py): 1e-10 of each field's largest magnitude.  The mixed
forms: u is a difference of stored populations, so their rounding (2^-24,
2^-11) reaches it amplified by the populations' pressure part over u, some
1e4 for single and 1e2 for half (whose scale is the pressure) here: 5e-3 and
5e-2 over six steps."""
import numpy as np
import pytest

from paper_2304_05657_amd import workloads as W

from .gpu_util import compare_fields, need_gpu, oracle_threads, say

pytestmark = pytest.mark.gpu

PERIODIC = ("periodic",) * 6
DUCT = ("inflow", "outflow", "wall", "wall_adiabatic", "periodic", "periodic")
CLOSED = ("wall", "wall", "wall_adiabatic", "wall", "wall", "wall_adiabatic")
INLETS = ("outflow", "wall", "periodic", "periodic", "inflow", "wall")


def _box(nx, ny, nz, faces, mech=False, seed=3):
    """Single solid cells (7 %, isothermal and adiabatic) in warm gas with a
    smooth temperature and composition and a random velocity."""
    base = W.porous_3d_mech(nx=40, ny=4, nz=4) if mech else W.porous_3d(nx=40, ny=4, nz=4)
    rng = np.random.default_rng(seed)
    shape = (nz, ny, nx)
    mask = rng.choice([0, 1, 2], size=shape, p=[0.93, 0.05, 0.02]).astype(np.uint8)
    mask[0, 0, 0] = 0
    z, y, x = np.meshgrid(np.arange(nz), np.arange(ny), np.arange(nx), indexing="ij")
    th = 0.5 + 0.5 * np.sin(2 * np.pi * (x / nx + y / ny + z / nz) + 0.3)
    T0 = 600.0 + 200.0 * th
    burnt = np.array(W.Y_BURNT_STOICH if not mech else (0.0, 0.0, 0.05, 0.05, 0.05, 0.05, 0.0, 0.05, 0.75))
    Y0 = np.stack([(1.0 - 0.5 * th) * a + 0.5 * th * b for a, b in zip(base.Y_in, burnt)])
    u0 = np.where(mask == 0, rng.uniform(-0.01, 0.01, (3,) + shape), 0.0)
    return base.replace(nx=nx, ny=ny, nz=nz, faces=faces, face_T=(510.0, 520.0, 530.0, 540.0, 550.0, 560.0),
                        mask=mask, wall_T=np.full(shape, 500.0), T0=T0, Y0=Y0, u0=u0, T_in=600.0, notes={})


@pytest.mark.parametrize("nx,ny,nz,faces", [
    (63, 2, 2, PERIODIC), (64, 3, 5, PERIODIC), (65, 5, 3, PERIODIC), (130, 4, 2, PERIODIC), (2, 2, 2, PERIODIC),
    (65, 5, 7, DUCT), (64, 2, 3, DUCT), (3, 6, 5, DUCT), (129, 3, 4, DUCT),
    (65, 3, 3, CLOSED), (5, 1, 1, CLOSED), (63, 4, 5, CLOSED),
    (66, 7, 4, INLETS),
])
def test_tiles_fp64(nx, ny, nz, faces):
    import oracle
    from paper_2304_05657_amd.lbfd import Solver
    need_gpu()
    p = _box(nx, ny, nz, faces)
    g, o = Solver(p, check_every=2), oracle.Oracle(p, threads=oracle_threads())
    g.step(5)
    o.step(5)
    g.sync()
    e = compare_fields(g.fields(), o.fields(), p)
    say("tiles %dx%dx%d %s: %s" % (nx, ny, nz, faces, " ".join("%s=%.1e" % kv for kv in e.items())))
    assert max(e.values()) <= 1e-10, e
    dg, do = g.diagnostics(), o.diagnostics()
    for k in ("sum_theta", "wall_q", "fuel_rate"):
        assert abs(dg[k] - do[k]) <= 1e-10 * max(abs(do[k]), 1e-12), (k, dg[k], do[k])


@pytest.mark.parametrize("nx,ny,nz,faces", [(65, 5, 3, PERIODIC), (63, 4, 5, DUCT)])
@pytest.mark.parametrize("precision,tol", [("fp64", 1e-10), ("fp32", 5e-3), ("fp16", 5e-2)])
def test_tiles_mechanism(nx, ny, nz, faces, precision, tol):
    import oracle
    from paper_2304_05657_amd.lbfd import Solver
    need_gpu()
    p = _box(nx, ny, nz, faces, mech=True)
    g, o = Solver(p, precision=precision), oracle.Oracle(p, threads=oracle_threads())
    g.step(6)
    o.step(6)
    e = compare_fields(g.fields(), o.fields(), p, keys=("u", "T", "Y", "rho"))
    say("mechanism %s %dx%dx%d: %s" % (precision, nx, ny, nz, " ".join("%s=%.1e" % kv for kv in e.items())))
    assert max(e.values()) <= tol, e
