"""Host memory of an assembly over threads."""
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CHILD = """
import resource, sys
sys.path.insert(0, sys.argv[1])
from paper_2004_06309_amd import helm, workloads as wl
w = wl.tiny(nx=60)
h = helm.Helm(-1)
n = h.assemble(w.xyz, w.tets, w.order, w.c_tet, w.omega)
print(n, resource.getrusage(resource.RUSAGE_SELF).ru_maxrss * 1024)
"""

DIGEST = """
import hashlib, sys
sys.path.insert(0, sys.argv[1])
import numpy as np
from paper_2004_06309_amd import helm, workloads as wl
for w in (wl.tiny(nx=60), wl.small_box(n=(36, 36, 20), order=2, n_parts=(1, 1, 1), coarse=False)):
    h = helm.Helm(-1)
    n = h.assemble(w.xyz, w.tets, w.order, w.c_tet, w.omega)
    assert 160 * 8 * n > 256 << 20
    print(n, hashlib.sha256(b"".join(np.ascontiguousarray(x).tobytes() for x in h.matrix_csr())).hexdigest())
"""


def _peak(threads):
    env = dict(os.environ, OMP_NUM_THREADS=str(threads))
    out = subprocess.run([sys.executable, "-c", CHILD, ROOT], env=env, capture_output=True, text=True, check=True)
    return (int(v) for v in out.stdout.split())


def test_assembly_memory_does_not_grow_by_the_unknowns_of_every_thread():
    """160 threads against one: marks of 8 bytes per unknown and thread would be 290
    MB, beyond the 256 MB they may take; stacks, allocator arenas and tables over the
    columns of a row are far below half of that."""
    n, one = _peak(1)
    _, many = _peak(160)
    assert 160 * 8 * n > 256 << 20
    assert many - one <= 159 * 8 * n / 2


def test_marks_and_tables_assemble_the_same_matrix():
    """The matrix over one thread (marks) and over 160 (tables), bit for bit."""
    a, b = (subprocess.run([sys.executable, "-c", DIGEST, ROOT], env=dict(os.environ, OMP_NUM_THREADS=t),
                           capture_output=True, text=True, check=True).stdout for t in ("1", "160"))
    assert a and a == b
