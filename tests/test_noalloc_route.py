"""The allocation-free sort takes the same route as the sort with a workspace at
every size it accepts: its fixed scratch holds the digit passes' counts.  Seen
from the launches each enqueues, on a stand-in for the runtime."""
import os
import subprocess
import sys

import pytest

import paper_2409_03970_amd as hv
from test_failed_launch import STAND_IN

pytestmark = pytest.mark.skipif(not os.path.exists(hv.LIB_PATH), reason="libhvms.so not built")

RUN = r"""
import ctypes, sys
shim = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
L = ctypes.CDLL(sys.argv[2])
V, I = ctypes.c_void_p, ctypes.c_int64
L.hvms_sort_workspace_bytes.restype = I
for n in (1000, 32768, 32769, 65536, 131073, 1 << 20, 3670015, 3670016, 3840000, 3850241, 4000001,
          (1 << 22) - 1, 1 << 22):
    need = L.hvms_sort_workspace_bytes(I(n), 0, None)
    shim.begin(0)
    assert L.hvms_sort_i32(V(1 << 40), V(2 << 40), I(n), V(3 << 40), ctypes.c_size_t(need), None,
                           None) == 0
    with_ws = shim.attempted()
    shim.begin(0)
    assert L.hvms_sort_i32_noalloc(V(1 << 40), V(2 << 40), I(n), None, None) == 0
    assert shim.attempted() == with_ws, (n, shim.attempted(), with_ws)
print("ok")
"""


def test_the_same_launches_with_and_without_a_workspace(tmp_path):
    src, so, run = tmp_path / "shim.c", tmp_path / "shim.so", tmp_path / "run.py"
    src.write_text(STAND_IN + "int hipGetSymbolAddress(void **p, const void *s)"
                              "{ *p = (void *)(4ul << 40); return 0; }\n")
    run.write_text(RUN)
    subprocess.run(["gcc", "-shared", "-fPIC", "-w", str(src), "-o", str(so)], check=True)
    r = subprocess.run([sys.executable, str(run), str(so), hv.LIB_PATH], capture_output=True,
                       text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout + r.stderr
