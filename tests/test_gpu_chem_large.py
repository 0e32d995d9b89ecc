"""A mechanism whose specialised chemistry does not fit the registers of four
waves per SIMD (32 reactions, 9 species: compiled again for three) against the
generic kernel: the same bits, as for the smaller mechanisms of
test_gpu_chem_specialised.py."""
import numpy as np
import pytest

from paper_2304_05657_amd import workloads as W

from .gpu_util import need_gpu, say
from .test_gpu_chem_specialised import _run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_rx", [26, 32])
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_large_mechanism_equals_generic(precision, n_rx):
    need_gpu()
    prob = W.porous_3d_mech(nx=48, ny=24, nz=24, margin=6).replace(reactions=W.synthetic_mechanism(9, n_rx, 2305))
    say("%d reactions, %s" % (n_rx, precision))
    spec, note, fj = _run(prob, precision, True, 5)
    assert spec, note
    gen, _, fg = _run(prob, precision, False, 5)
    assert not gen
    for key in ("T", "Y"):
        assert np.all(np.isfinite(np.asarray(fj[key])))
        assert np.array_equal(np.asarray(fj[key]), np.asarray(fg[key])), key
