"""Mode lists with components at the ends of the 32-bit range, given to the layout of dense
lists in a build of the host code that traps on undefined behaviour (the absolute
value of -2^31 is one)."""
import os
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CODE = """
import ctypes as C, sys
import numpy as np
L = C.CDLL(sys.argv[1], mode=0x1)       # RTLD_LAZY: the kernels' launchers are not linked
f = L.rbe_plan_columns
f.argtypes = [C.c_void_p, C.c_int32, C.c_int64, C.c_int32, C.c_int64, C.c_void_p]
f.restype = None
ax = np.arange(-6, 7)
m = np.stack(np.meshgrid(ax, ax, ax, indexing="ij")).reshape(3, -1).astype(np.int32)
m = np.ascontiguousarray(m[:, (m != 0).any(0)])
out = np.zeros(5, np.int32)
for d in range(3):
    for v in (2 ** 31 - 1, -2 ** 31 + 1, -2 ** 31):
        k = m.copy()
        k[d, 700] = v
        f(k.ctypes.data, k.shape[1], 5000, 1, 1 << 40, out.ctypes.data)
        assert out[0] == 0, (d, v, out)
print("mode range: ok")
"""


@pytest.mark.skipif(shutil.which("hipcc") is None and not os.path.exists("/opt/rocm/bin/hipcc"),
                    reason="hipcc not available")
def test_modes_at_the_ends_of_the_range(tmp_path):
    from paper_2010_01559_amd import build as B
    so = str(tmp_path / "api.so")
    cmd = [B.hipcc(), "-O1", "-std=c++17", "-fPIC", "--offload-arch=gfx950", "-Xclang", "-target-feature", "-Xclang",
           "-packed-fp32-ops", "-Xarch_host", "-fsanitize=undefined", "-Xarch_host", "-fsanitize-trap=undefined",
           "-I", os.path.join(ROOT, "include"), "-I", B.CSRC, "-shared", "-Wl,--unresolved-symbols=ignore-all",
           "-x", "hip", os.path.join(B.CSRC, "rbe_api.cpp"), "-o", so]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([sys.executable, "-c", CODE, so], capture_output=True, text=True)
    assert r.returncode == 0 and "mode range: ok" in r.stdout, (r.returncode, r.stderr[-2000:])
