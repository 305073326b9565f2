"""The platform FFT may overwrite the input of a complex transform even where the
output is another buffer (rocFFT's own header says so), and the imagers' grids
are read only: for sides they hand to the library, the transform runs in place
in the scratch.  The library's entry points are replaced by recording stubs in a
process without a device (the kernels around the transform cannot launch there,
which the calls report at their end)."""
import os
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

STUBS = r"""
#include <cstdio>
extern "C" {
int hipfftPlanMany(void **plan, int, int *, int *, int, int, int *, int, int, int, int) {
    *plan = reinterpret_cast<void *>(8);
    return 0;
}
int hipfftSetStream(void *, void *) { return 0; }
int hipfftDestroy(void *) { return 0; }
int hipfftExecC2C(void *, void *in, void *out, int) {
    std::printf("C2C %p %p\n", in, out);
    std::fflush(stdout);
    return 0;
}
}
"""

CHILD = """
import ctypes as C, sys
C.CDLL(sys.argv[2], mode=C.RTLD_GLOBAL)     # found before the library's own
hip = C.CDLL("libamdhip64.so")
n = C.c_int(0)
if hip.hipGetDeviceCount(C.byref(n)) == 0 and n.value > 0:
    sys.exit(77)                    # a device is visible: nothing is launched
L = C.CDLL(sys.argv[1])
vp = C.c_void_p
L.mg_imager_exec.argtypes = [vp] * 6 + [C.c_int32, C.c_int32, vp]
L.mg_wstack_imager_exec.argtypes = [vp] * 6 + [C.c_double] * 3 + [vp]
GRID, WORK, IMAGE, CORR = 0x10000, 0x20000, 0x30000, 0x40000
h = vp()
assert L.mg_imager_create(C.byref(h), 2, 6, 10) == 0
L.mg_imager_exec(h, GRID, WORK, IMAGE, CORR, CORR, 0, 10, None)
L.mg_imager_exec(h, GRID, WORK, WORK, CORR, CORR, 0, 10, None)
assert L.mg_wstack_imager_create(C.byref(h), 1, 3, 6, 10) == 0
L.mg_wstack_imager_exec(h, GRID, WORK, IMAGE, CORR, CORR, 0.1, 0.1, 1.0, None)
"""


def test_library_transforms_run_in_the_scratch(tmp_path):
    lib = os.path.join(ROOT, "paper_2111_04141_amd", "libmigrid.so")
    if not os.path.exists(lib) or shutil.which("g++") is None:
        pytest.skip("needs the built library and a host compiler")
    src, so = tmp_path / "stubs.cpp", tmp_path / "stubs.so"
    src.write_text(STUBS)
    subprocess.run(["g++", "-shared", "-fPIC", "-o", str(so), str(src)], check=True)
    env = dict(os.environ, HIP_VISIBLE_DEVICES="-1")
    r = subprocess.run([sys.executable, "-c", CHILD, lib, str(so)], env=env, capture_output=True,
                       text=True, timeout=120)
    if r.returncode == 77:
        pytest.skip("a device is visible")
    assert r.returncode == 0, r.stderr
    calls = [line.split()[1:] for line in r.stdout.splitlines() if line.startswith("C2C")]
    assert calls == [["0x20000", "0x20000"]] * 3
