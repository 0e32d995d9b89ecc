"""The specialised chemistry text of the largest mechanisms (32 reactions, two
to four reactants each, 9 species), on the CPU: its register budget is an
argument, everything else the same text; compiled at three waves per SIMD it
takes no private memory (where a kernel's spilled registers go), which is what
the library falls back to when four waves spill.  The private memory is read
from the metadata of the code object just built."""
import os
import shutil
import subprocess
import tempfile

import pytest

from paper_2304_05657_amd import workloads as W

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2304_05657_amd")
HIPCC = "/opt/rocm/bin/hipcc"

HARNESS = r'''
#include <hip/hip_runtime.h>
#include <hip/hiprtc.h>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <cstdlib>
#include <fstream>
#include <sstream>
#include <string>
#include <vector>
#include "lbfd_internal.h"
struct R { double adt, b, Ta, q; int n; int react[4]; double nu[9]; };
static const R rs[] = { %(rows)s };
// h f64|f32 waves text header code
int main(int, char **argv) {
    const int n = sizeof(rs) / sizeof(rs[0]);
    std::vector<lbfd::ChemRx> h(n);
    memset(h.data(), 0, sizeof(lbfd::ChemRx) * n);
    const double c = 0x1.71547652b82fep+8;
    for (int j = 0; j < n; ++j) {
        h[j].adt = rs[j].adt; h[j].b = rs[j].b; h[j].ta = rs[j].Ta; h[j].q = rs[j].q; h[j].n_react = rs[j].n;
        h[j].bs = h[j].b * c; h[j].tas = h[j].ta * c; h[j].lnadts = std::log(h[j].adt) * c;
        for (int m = 0; m < 4; ++m) h[j].react[m] = rs[j].react[m];
        for (int k = 0; k < 9; ++k) h[j].nu[k] = rs[j].nu[k];
    }
    const bool fp64 = strcmp(argv[1], "f64") == 0;
    const int waves = atoi(argv[2]);
    const std::string src = waves ? lbfd::chem_jit_source(h.data(), n, 9, fp64, waves)
                                  : lbfd::chem_jit_source(h.data(), n, 9, fp64);
    std::ofstream(argv[3]) << src;
    std::ifstream hf(argv[4]);
    std::stringstream hs; hs << hf.rdbuf();
    const std::string hdr = hs.str();
    hiprtcProgram p;
    const char *hd[] = {hdr.c_str()};
    const char *hn[] = {"lbfd_math.h"};
    if (hiprtcCreateProgram(&p, src.c_str(), "chem.hip", 1, hd, hn) != HIPRTC_SUCCESS) return 3;
    const char *o[] = {"--offload-arch=gfx950", "-O3", "-std=c++17", "-Xclang", "-target-feature", "-Xclang",
                       "-packed-fp32-ops"};
    if (hiprtcCompileProgram(p, 7, o) != HIPRTC_SUCCESS) return 2;
    size_t cs = 0;
    hiprtcGetCodeSize(p, &cs);
    std::vector<char> code(cs);
    hiprtcGetCode(p, code.data());
    std::ofstream(argv[5], std::ios::binary).write(code.data(), cs);
    return 0;
}
'''


def _private_bytes(path):
    """.private_segment_fixed_size of the code object's kernel (a MessagePack
    integer after its key)."""
    d = open(path, "rb").read()
    key = b".private_segment_fixed_size"
    assert d.count(key) == 1
    at = d.index(key) + len(key)
    t = d[at]
    if t < 0x80:
        return t
    width = {0xcc: 1, 0xcd: 2, 0xce: 4}[t]
    return int.from_bytes(d[at + 1:at + 1 + width], "big")


@pytest.fixture(scope="module", params=[2, 4])
def harness(request):
    lib = os.path.join(PKG, "liblbfd.so")
    if not (os.path.exists(HIPCC) and os.path.exists(lib)):
        pytest.skip("hipcc or the built library is missing")
    rows = []
    for i, r in enumerate(W.synthetic_mechanism(9, 32, 2305)):
        re_ = list(r.reactants) + [i % 8, (3 * i) % 8][:request.param - 2]
        rows.append("{ %r, %r, %r, %r, %d, {%s}, {%s} }" % (
            r.A * 1e-6, r.b, r.Ta, r.q, len(re_), ",".join(map(str, re_ + [9] * (4 - len(re_)))),
            ", ".join(repr(float(x)) for x in r.nu)))
    d = tempfile.mkdtemp(prefix="lbfd_chem_large_")
    src = os.path.join(d, "h.hip")
    with open(src, "w") as f:
        f.write(HARNESS % {"rows": ",\n".join(rows)})
    exe = os.path.join(d, "h")
    subprocess.run([HIPCC, "-std=c++17", "-I", os.path.join(PKG, "csrc"), src, "-o", exe, "-L" + PKG, "-llbfd",
                    "-L/opt/rocm/lib", "-lhiprtc", "-Wl,-rpath," + PKG + ":/opt/rocm/lib"],
                   check=True, capture_output=True)
    yield exe, d
    shutil.rmtree(d, ignore_errors=True)


@pytest.mark.parametrize("kind", ["f64", "f32"])
def test_register_budget(harness, kind):
    exe, d = harness
    text, spill = {}, {}
    for waves in (0, 4, 3):
        t, c = os.path.join(d, "%s_%d.hip" % (kind, waves)), os.path.join(d, "%s_%d.co" % (kind, waves))
        r = subprocess.run([exe, kind, str(waves), t, os.path.join(PKG, "csrc", "lbfd_math.h"), c], cwd=d,
                           capture_output=True, text=True, timeout=300)
        assert r.returncode == 0, r.stdout + r.stderr
        text[waves], spill[waves] = open(t).read(), _private_bytes(c)
    assert text[0] == text[4]
    assert text[4].replace("amdgpu_waves_per_eu(4)", "amdgpu_waves_per_eu(3)") == text[3] != text[4]
    assert spill[3] == 0, spill
