"""lbfd_read_fields_dev: the fields launch writes the caller's device buffers
itself, each optional.  Every subset of outputs gives the values of a full
host read (the same kernel arithmetic: equal bits), solid cells included,
and leaves the context's state and the buffers not asked for alone."""
import ctypes as C

import numpy as np
import pytest

from paper_2304_05657_amd import workloads as W

from .gpu_util import need_gpu, say

pytestmark = pytest.mark.gpu

KEYS = ("rho", "u", "T", "Y", "Ph")


def _problem(dim, nsp):
    if dim == 2:
        return W.cylinder_burner(nx=131, ny=64, radius=8.0, pitch=32, x_begin=32, x_end=96, front_x=64.0)
    if nsp == 9:
        return W.porous_3d_mech(nx=34, ny=11, nz=9, porosity=0.9, radius=(2.0, 3.0), margin=6)
    return W.porous_3d(nx=66, ny=11, nz=9, porosity=0.9, radius=2.5, margin=6)


@pytest.mark.parametrize("dim,nsp,precision", [(2, 4, "fp64"), (2, 4, "fp16"), (3, 4, "fp64"), (3, 4, "fp16"),
                                               (3, 9, "fp32")])
def test_subsets_of_outputs(dim, nsp, precision):
    torch = need_gpu()
    from paper_2304_05657_amd.lbfd import Solver
    p = _problem(dim, nsp)
    s = Solver(p, precision=precision)
    s.step(3)
    state = s.save_state()
    host = s.fields()
    host["u"] = host["u"][:dim]
    size = {"rho": p.N, "u": dim * p.N, "T": p.N, "Y": len(p.W) * p.N, "Ph": p.N}
    for asked in (KEYS, ("T",), ("Y",), ("rho", "Ph"), ("u",), ()):
        say("%dd %d species %s: %s" % (dim, nsp, precision, ",".join(asked) or "nothing"))
        buf = {k: torch.full((size[k] + 2,), -7.0, dtype=torch.float64, device="cuda") for k in KEYS}
        rc = s._lib.lbfd_read_fields_dev(s._h, *(C.c_void_p(buf[k][1:].data_ptr()) if k in asked else None
                                                 for k in KEYS))
        assert rc == 0
        for k in KEYS:
            b = buf[k].cpu().numpy()
            assert b[0] == -7.0 and b[-1] == -7.0
            if k in asked:
                assert np.array_equal(b[1:-1], host[k].reshape(-1)), k
            else:
                assert np.all(b == -7.0), k
    assert s.save_state() == state
    s.close()
