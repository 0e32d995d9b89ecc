"""2-D tiles of the step (16 x 16 cells, every fluid cell in its tile, scalars
staged with a 2-cell halo) at the sizes where their indexing can go wrong:
boxes one cell short of, at and past a tile in x (test_gpu_tile_seams.py: in
y), boxes thinner than the halo, every face kind next to ragged tiles, single-cell solids against
faces and behind an inlet's first cell.  Against the oracle.

Tolerance: in FP64 the two sides differ by rounding order only (see
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
TUBE = ("outflow", "inflow", "periodic", "periodic", "periodic", "periodic")
CLOSED = ("wall", "wall", "wall_adiabatic", "wall", "periodic", "periodic")
INLETS = ("outflow", "wall", "inflow", "inflow", "periodic", "periodic")


def _box(nx, ny, faces, seed=3):
    """Single solid cells (7 %, isothermal and adiabatic) in warm gas with a
    smooth temperature and composition and a random velocity."""
    base = W.channel_flame(nx=40, ny=8)
    rng = np.random.default_rng(seed)
    shape = (1, ny, nx)
    mask = rng.choice([0, 1, 2], size=shape, p=[0.93, 0.05, 0.02]).astype(np.uint8)
    mask[0, 0, 0] = 0
    if nx > 2 and ny > 2:  # the mirror cells of the second ghost are solid
        mask[0, 1, [0, 1, nx - 2, nx - 1]] = [0, 1, 2, 0]
    x, y = np.meshgrid(np.arange(nx), np.arange(ny), indexing="xy")
    th = (0.5 + 0.5 * np.sin(2 * np.pi * (x / nx + y / ny) + 0.3))[None]
    T0 = 600.0 + 200.0 * th
    Y0 = np.stack([(1.0 - 0.5 * th) * a + 0.5 * th * b for a, b in zip(base.Y_in, W.Y_BURNT_STOICH)])
    u0 = np.where(mask == 0, rng.uniform(-0.01, 0.01, (3,) + shape), 0.0)
    u0[2] = 0.0
    return base.replace(nx=nx, ny=ny, faces=faces, face_T=(510.0, 520.0, 530.0, 540.0, 550.0, 560.0), mask=mask,
                        wall_T=np.full(shape, 500.0), T0=T0, Y0=Y0, u0=u0, T_in=600.0, u_in=(0.01, 0.0, 0.0),
                        notes={})


@pytest.mark.parametrize("precision,tol", [("fp64", 1e-10), ("fp32", 5e-3), ("fp16", 5e-2)])
@pytest.mark.parametrize("nx,ny,faces", [
    (63, 3, PERIODIC), (64, 4, PERIODIC), (65, 5, PERIODIC), (130, 9, PERIODIC), (2, 2, PERIODIC),
    (65, 7, DUCT), (64, 8, DUCT), (3, 6, DUCT), (129, 11, DUCT), (67, 2, TUBE), (62, 9, TUBE),
    (66, 13, CLOSED), (5, 1, CLOSED), (1, 6, CLOSED), (66, 6, INLETS), (4, 9, INLETS),
])
def test_tiles(nx, ny, faces, precision, tol):
    import oracle
    from paper_2304_05657_amd.lbfd import Solver
    need_gpu()
    p = _box(nx, ny, faces)
    g, o = Solver(p, precision=precision, check_every=2), oracle.Oracle(p, threads=oracle_threads())
    g.step(6)
    o.step(6)
    g.sync()
    e = compare_fields(g.fields(), o.fields(), p, keys=("u", "T", "Y", "rho"))
    say("tiles %s %dx%d %s: %s" % (precision, nx, ny, faces, " ".join("%s=%.1e" % kv for kv in e.items())))
    assert max(e.values()) <= tol, e
    dg, do = g.diagnostics(), o.diagnostics()
    for k in ("sum_theta", "wall_q", "fuel_rate"):
        assert abs(dg[k] - do[k]) <= tol * max(abs(do[k]), 1e-12), (k, dg[k], do[k])
