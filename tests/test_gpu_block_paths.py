"""Level solves and products of 2 to 16 right-hand sides advanced together against
one right-hand side at a time, on operators that reach every branch: levels of more
tiles than get four waves each, rows without, with some and with only imaginary
parts, and a coarse stage."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2004_06309_amd import helm  # noqa: E402
from paper_2004_06309_amd import workloads as wl  # noqa: E402


def _one_step(h, nrhs, block, seed):
    """One Arnoldi step from zero, u = y M^{-1} b with y from the dots of
    A M^{-1} b: no stopping test decides anything, and both sides apply the same
    panels and entries in FP64 (the local solves of the two agree to 1e-12, y to
    the same)."""
    B = torch.stack([torch.from_numpy(wl.random_vector(h.n, seed + k)) for k in range(nrhs)]).to("cuda")
    U, V = torch.zeros_like(B), torch.zeros_like(B)
    h.solve(B, U, tol=1e-14, restart=1, maxit=1, block=block)
    for k in range(nrhs):
        h.solve(B[k].contiguous(), V[k], tol=1e-14, restart=1, maxit=1)
        assert float((U[k] - V[k]).norm() / V[k].norm()) <= 1e-11


# Leaves of four unknowns: forward levels of 6,187 and 3,911 tiles (a remainder of
# three on the groups of four), backward ones of 2,302 (216 of them wide), 4,360 and
# 3,120, so a wave takes a narrow tile of its own from 2,049 tiles on.
@pytest.mark.parametrize("c64", [0, 1, 2])
@pytest.mark.parametrize("nrhs", [2, 4, 7])
def test_narrow_blocks_on_levels_of_many_tiles(nrhs, c64):
    w = wl.small_box(n=(22, 18, 14), order=2, n_parts=(3, 3, 1), overlap=1, coarse=False)
    h = helm.from_workload(w, c64=c64, leaf_size=4, batches=1)
    # the first forward level holds every leaf, at least half of the supernodes of
    # binary trees
    assert h.stats()["n_supernodes"] > 2 * 2048
    print(f"[many tiles] c64={c64} nrhs={nrhs}", flush=True)
    _one_step(h, nrhs, 8, 60)


# Rows of every kind: with real velocities real rows of many entries (and those of
# the absorbing faces, with a few imaginary parts), with attenuation only complex
# ones; even counts of cells, so a coarse stage takes part.
@pytest.mark.parametrize("nrhs", [2, 4, 7, 9, 16])
@pytest.mark.parametrize("attenuation", [0.0, 0.02])
def test_products_and_coarse_stage_of_a_block(attenuation, nrhs):
    w = wl.small_box(n=(6, 6, 4), order=2, n_parts=(2, 2, 1), overlap=2, attenuation=attenuation)
    h = helm.from_workload(w)
    assert h.stats()["n_coarse"] > 0
    ptr, _, val = h.matrix_csr()
    length = np.diff(ptr)
    imag = np.add.reduceat((val.imag != 0).astype(np.int64), ptr[:-1])
    assert bool(((imag == 0) & (length > 16)).any()) == (attenuation == 0.0)
    assert bool(((imag > 0) & (imag < length)).any()) == (attenuation == 0.0)
    print(f"[products] attenuation={attenuation} nrhs={nrhs}", flush=True)
    _one_step(h, nrhs, 16, 90)
