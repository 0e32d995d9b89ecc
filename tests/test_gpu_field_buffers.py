"""Device buffers of lbfd_read_fields_dev that the fields launch must not write
by itself: one whose allocation ends before its field does (filled by a copy,
which the runtime refuses; the refused buffers hold half their field, so that
no rounding of an allocation's size hides it), buffers that overlap, or that lie
off the alignment of a double (filled by copies in the order rho, u, P_h, T,
Y)."""
import ctypes as C

import numpy as np
import pytest

from paper_2304_05657_amd import workloads as W

from .gpu_util import need_gpu, say

pytestmark = pytest.mark.gpu

KEYS = ("rho", "u", "T", "Y", "Ph")


def _solver(dim, precision):
    from paper_2304_05657_amd.lbfd import Solver
    p = W.cylinder_burner(nx=256, ny=64, radius=8.0, pitch=32, x_begin=32, x_end=96, front_x=64.0) if dim == 2 \
        else W.porous_3d(nx=66, ny=16, nz=16, porosity=0.9, radius=2.5, margin=6)
    s = Solver(p, precision=precision)
    s.step(3)
    host = s.fields()
    host["u"] = host["u"][:dim]
    return s, p, host, {"rho": p.N, "u": dim * p.N, "T": p.N, "Y": len(p.W) * p.N, "Ph": p.N}


@pytest.mark.parametrize("dim", [2, 3])
@pytest.mark.parametrize("small", KEYS)
def test_too_small_is_refused(dim, small):
    torch = need_gpu()
    s, p, host, size = _solver(dim, "fp64")
    hip = s._lib  # (its symbols include those of the HIP runtime it is linked to)
    raw = C.c_void_p()
    assert hip.hipMalloc(C.byref(raw), C.c_size_t(size[small] * 4)) == 0
    say("%dd %s: %d bytes for %d doubles" % (dim, small, size[small] * 4, size[small]))
    buf = {k: torch.full((size[k],), -7.0, dtype=torch.float64, device="cuda") for k in KEYS}
    rc = s._lib.lbfd_read_fields_dev(s._h, *(raw if k == small else C.c_void_p(buf[k].data_ptr()) for k in KEYS))
    assert rc == -3 and b"copy of a field" in s._lib.lbfd_last_error()
    # the context still reads and steps
    assert s._lib.lbfd_read_fields_dev(s._h, *(C.c_void_p(buf[k].data_ptr()) for k in KEYS)) == 0
    for k in KEYS:
        assert np.array_equal(buf[k].cpu().numpy(), host[k].reshape(-1)), k
    s.step(1)
    s.sync()
    assert hip.hipFree(raw) == 0
    s.close()


@pytest.mark.parametrize("dim,precision", [(2, "fp64"), (3, "fp64"), (3, "fp16")])
def test_overlapping_and_odd_buffers(dim, precision):
    torch = need_gpu()
    s, p, host, size = _solver(dim, precision)
    # rho and P_h in one buffer, T overlapping the end of u
    one = torch.full((p.N,), -7.0, dtype=torch.float64, device="cuda")
    both = torch.full((size["u"] + p.N // 2,), -7.0, dtype=torch.float64, device="cuda")
    T = both[size["u"] - p.N // 2:]
    rc = s._lib.lbfd_read_fields_dev(s._h, C.c_void_p(one.data_ptr()), C.c_void_p(both.data_ptr()),
                                     C.c_void_p(T.data_ptr()), None, C.c_void_p(one.data_ptr()))
    assert rc == 0
    assert np.array_equal(one.cpu().numpy(), host["Ph"].reshape(-1))
    assert np.array_equal(T.cpu().numpy(), host["T"].reshape(-1))
    assert np.array_equal(both.cpu().numpy()[:size["u"] - p.N // 2], host["u"].reshape(-1)[:size["u"] - p.N // 2])
    # four bytes off the alignment of a double
    odd = torch.zeros(2 * p.N + 2, dtype=torch.float32, device="cuda")
    rc = s._lib.lbfd_read_fields_dev(s._h, C.c_void_p(odd.data_ptr() + 4), None, None, None, None)
    assert rc == 0
    got = np.frombuffer(odd.cpu().numpy().tobytes()[4:4 + 8 * p.N], dtype=np.float64)
    assert np.array_equal(got, host["rho"].reshape(-1))
    s.close()
