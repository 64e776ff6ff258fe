"""Host allocations that fail, in serial code and in threads: a status, never the end
of the process."""
import os
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# operator new that, once armed, refuses the n-th request of at least 4 KiB from the
# solver library, whichever thread makes it
SHIM = r"""
#include <dlfcn.h>
#include <atomic>
#include <cstdlib>
#include <cstring>
#include <new>
static std::atomic<long> left{-1};
static std::atomic<int> hit{0};
extern "C" void shim_arm(long n) { hit = 0; left = n; }
extern "C" int shim_hit() { return hit; }
static bool from_solver(void* caller) {
  Dl_info i;
  return dladdr(caller, &i) && i.dli_fname && std::strstr(i.dli_fname, "libhelm.so");
}
void* operator new(std::size_t n) {
  if (left >= 0 && n >= 4096 && from_solver(__builtin_return_address(0)) && left-- == 0) {
    hit = 1;
    throw std::bad_alloc();
  }
  void* p = std::malloc(n ? n : 1);
  if (!p) throw std::bad_alloc();
  return p;
}
"""

CHILD = """
import ctypes, os, sys
sys.path.insert(0, sys.argv[1])
from paper_2004_06309_amd import helm, workloads as wl
shim = ctypes.CDLL(sys.argv[2])
ws = [wl.small_box(n=(8, 8, 6), order=2, n_parts=(3, 2, 1), overlap=2), wl.tiny(nx=8)]
helm.load()
refused = 0
for name, w in enumerate(ws):
    for k in range(100000):
        pid = os.fork()
        if pid == 0:
            code = 3
            try:
                h = helm.Helm(-1)
                shim.shim_arm(ctypes.c_long(k))
                try:
                    h.assemble(w.xyz, w.tets, w.order, w.c_tet, w.omega)
                    h.precond_setup(w.part, w.n_sub, w.overlap, w.coarse_xyz, w.coarse_tets)
                    code = 0
                except helm.HelmError as e:
                    code = 0 if e.code == helm.HELM_ENOMEM else 4
                if code == 0 and not shim.shim_hit():
                    code = 1  # the run makes fewer requests
            finally:
                os._exit(code)
        _, status = os.waitpid(pid, 0)
        if os.WIFSIGNALED(status) or os.WEXITSTATUS(status) > 1:
            sys.exit(f"request {k} of workload {name}: wait status {status}")
        if os.WEXITSTATUS(status) == 1:
            break
        refused += 1
print("refused", refused, flush=True)
sys.exit(0 if refused > 100 else "too few requests")
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs a host compiler")
def test_a_refused_allocation_is_a_status(tmp_path):
    """Assembly and setup on the host (two threads), one process per refused request:
    HELM_ENOMEM, or HELM_OK where the request had another way."""
    src, lib = tmp_path / "shim.cpp", tmp_path / "shim.so"
    src.write_text(SHIM)
    subprocess.run(["g++", "-O1", "-shared", "-fPIC", "-o", str(lib), str(src), "-ldl"], check=True)
    env = dict(os.environ, OMP_NUM_THREADS="2", LD_PRELOAD=str(lib))
    out = subprocess.run([sys.executable, "-c", CHILD, ROOT, str(lib)], env=env, capture_output=True, text=True,
                         timeout=600)
    assert out.returncode == 0, out.stdout + out.stderr
