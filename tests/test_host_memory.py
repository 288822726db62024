"""Host allocations that fail inside the C entry points give a status, never an
exception through the C boundary (which would end the process).  Each call runs
in a child whose address space is limited; no device is touched."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CHILD = """
import ctypes, resource, sys
import numpy as np
import paper_2606_00079_amd as bm
entry, B, nnz, more = sys.argv[1], int(sys.argv[2]), int(sys.argv[3]), int(sys.argv[4])
L = bm.lib()
fake = ctypes.c_void_p(0x1000)  # never dereferenced: the tables come first
p = lambda a: a.ctypes.data_as(ctypes.c_void_p)
off = np.array([0, nnz], np.int64)
tok = np.zeros(nnz, np.int32)   # every entry is token 0's: B x nnz entry lists
w = np.ones(nnz, np.float32)
used = int(open("/proc/self/statm").read().split()[0]) * resource.getpagesize()
resource.setrlimit(resource.RLIMIT_AS, (used + more, used + more))
st = getattr(L, entry)(fake, fake, fake, fake, 10, 1, 8, 128, 64, fake, 64, fake, B, p(off), p(tok), p(w),
                       fake, ctypes.c_void_p(0))
print("status", st, bm.last_error())
"""


# the entry lists do not fit (34 GB); they fit (537 MB), and their copy for the device does not
@pytest.mark.parametrize("entry,B,nnz,more", [
    ("bitsmoe_moe_decode", 65535, 65535, 1 << 31),
    ("bitsmoe_moe_decode_in", 65535, 65535, 1 << 31),
    ("bitsmoe_moe_decode_in", 1024, 65535, 800 << 20),
])
def test_decode_routing_tables_without_memory(entry, B, nnz, more):
    from paper_2606_00079_amd import LIB_PATH
    if not os.path.exists(LIB_PATH):
        pytest.skip("libbitsmoe.so not built")
    r = subprocess.run([sys.executable, "-c", CHILD, entry, str(B), str(nnz), str(more)], cwd=ROOT,
                       capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr[-2000:]
    assert r.stdout.startswith("status 5 ") and "host allocation" in r.stdout, r.stdout


def test_device_cus_allocates_nothing(tmp_path):
    """The number of compute units is looked up once per device, on the path of
    the decode that promises to allocate nothing (any device index works)."""
    from paper_2606_00079_amd import build as b
    exe = str(tmp_path / "device_cus_check")
    subprocess.run(["g++", *b.CXX_FLAGS, f"-I{b.INCLUDE}", f"-I{b.CSRC}", "-o", exe,
                    os.path.join(ROOT, "tests", "device_cus_check.cpp"), os.path.join(b.CSRC, "api.cpp"),
                    f"-L{b.ROCM}/lib", f"-Wl,-rpath,{b.ROCM}/lib", "-lamdhip64", "-ldl"], check=True)
    out = subprocess.run([exe], capture_output=True, text=True, timeout=60, check=True).stdout.split()
    assert out[:5] == ["100", "103", "103", "100", "170"]
    assert out[5] == "3" and out[6] == "0", out
