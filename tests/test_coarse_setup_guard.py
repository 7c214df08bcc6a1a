"""A coarsest level of more unknowns than its kernels have room for (512), or of
none, is refused before anything is launched.  No GPU: a preloaded stand-in for
the first call of a launch counts them."""
import os
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
STUB = "int launches = 0;\nint __hipPushCallConfiguration() { ++launches; return 1; }\n"      # 1: go no further
CODE = """
import ctypes, sys
sys.path.insert(0, %r)
from paper_1910_12979_amd import macproj as M
lib = M.lib()
# mg::launch_coarse_setup(const Shape&, h, bx, by, bz, minv, scratch, stream, bnd, singular)
f = lib["_ZN2mg19launch_coarse_setupERKNS_5ShapeEdPKdS4_S4_PdS5_P12ihipStream_tPKNS_3BndIdEEi"]
f.restype = ctypes.c_int
vp = ctypes.c_void_p
f.argtypes = [vp, ctypes.c_double] + [vp] * 7 + [ctypes.c_int]
shape = (ctypes.c_int * 3)(*%r)
rc = f(ctypes.addressof(shape), 1.0, None, None, None, None, None, None, None, 1)
print(rc, ctypes.c_int.in_dll(ctypes.CDLL(%r), "launches").value)
"""


@pytest.mark.parametrize("n,refused", [((9, 8, 8), True), ((8, 8, 9), True), ((0, 8, 8), True), ((8, 8, 8), False),
                                       ((4, 4, 4), False)])
def test_refused_before_any_launch(tmp_path, n, refused):
    from paper_1910_12979_amd import build, macproj
    cc = shutil.which("gcc")
    if cc is None:
        pytest.skip("gcc not installed")
    if not os.path.exists(macproj.LIB_PATH):
        build.build()
    stub = str(tmp_path / "stub.so")
    (tmp_path / "stub.c").write_text(STUB)
    subprocess.run([cc, "-shared", "-fPIC", str(tmp_path / "stub.c"), "-o", stub], check=True)
    pre = " ".join(p for p in (os.environ.get("LD_PRELOAD"), stub) if p)
    r = subprocess.run([sys.executable, "-c", CODE % (ROOT, n, stub)], capture_output=True, text=True, timeout=300,
                       env=dict(os.environ, HIP_VISIBLE_DEVICES="", ROCR_VISIBLE_DEVICES="", LD_PRELOAD=pre))
    assert r.returncode == 0, r.stderr
    rc, launches = (int(x) for x in r.stdout.split()[-2:])
    assert (rc == 1 and launches == 0) if refused else launches >= 1       # hipErrorInvalidValue
