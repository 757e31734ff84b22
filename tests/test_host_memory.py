"""Host allocations that fail: every entry that plans or runs returns
MAFAT_ENOMEM (or what it returns anyway), and no exception leaves the library.
In a process of its own, whose operator new fails on demand (host code, no GPU:
the run calls end at their argument checks)."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SHIM = """
#include <cstdlib>
#include <new>
static long left = -1;  // allocations until one fails; -1: none does
extern "C" void fail_after(long n) { left = n; }
void* operator new(std::size_t n) {
  if (left == 0) throw std::bad_alloc();
  if (left > 0) --left;
  if (void* p = std::malloc(n ? n : 1)) return p;
  throw std::bad_alloc();
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, std::size_t) noexcept { std::free(p); }
"""

SCRIPT = """
import ctypes, sys
shim = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
shim.fail_after.argtypes = [ctypes.c_long]
from paper_2107_06960_amd import mafat as M
from paper_2107_06960_amd import workloads as W
lib, name = M.lib(), sys.argv[2]
seen = set()
for k in range(200):
    plan = M.Plan(W.YOLOV2_16, (608, 608, 3), "5x5/8/2x2", row_reuse=True)
    out = (ctypes.c_size_t if name == "workspace_size" else ctypes.c_int64)()
    fn, args = {
        "workspace_size": (lib.mafat_workspace_size, (plan.handle, 1, M.MAFAT_BF16, ctypes.byref(out))),
        "predict_mem": (lib.mafat_predict_mem, (plan.handle, 0, 1, M.MAFAT_BF16, ctypes.byref(out))),
        "run_group": (lib.mafat_run_group, (plan.handle, 0, 1, M.MAFAT_BF16) + (None,) * 6 + (0, None)),
        "run_network": (lib.mafat_run_network, (plan.handle, 1, M.MAFAT_BF16) + (None,) * 7 + (0, None)),
    }[name]
    shim.fail_after(k)
    rc = fn(*args)
    shim.fail_after(-1)
    seen.add(rc)
    if rc != -6 and k > 20:
        break
print(sorted(seen))
"""


@pytest.fixture(scope="module")
def shim(tmp_path_factory):
    d = tmp_path_factory.mktemp("shim")
    (d / "shim.cpp").write_text(SHIM)
    subprocess.check_call(["g++", "-O1", "-shared", "-fPIC", "-o", str(d / "shim.so"), str(d / "shim.cpp")])
    return str(d / "shim.so")


@pytest.mark.parametrize("entry,status", [("workspace_size", 0), ("predict_mem", 0), ("run_group", -4), ("run_network", -1)])
def test_failed_allocation_is_a_status(shim, entry, status):
    env = dict(os.environ, PYTHONPATH=ROOT)
    env["LD_PRELOAD"] = " ".join(v for v in (shim, env.get("LD_PRELOAD")) if v)
    r = subprocess.run([sys.executable, "-c", SCRIPT, shim, entry], cwd=ROOT, env=env, capture_output=True, text=True,
                       timeout=120)
    assert r.returncode == 0, r.stderr[-2000:]
    assert r.stdout.strip() == str(sorted({-6, status})), r.stdout
