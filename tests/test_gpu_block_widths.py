"""Level solves of 2 to 8 right-hand sides advanced together (FP64 MFMA, real
and imaginary parts side by side) against one right-hand side at a time."""
import dataclasses

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2004_06309_amd import helm  # noqa: E402
from paper_2004_06309_amd import workloads as wl  # noqa: E402

# ragged: levels of a few tiles, their rows split over workgroups; one tree:
# tiles wider than a staging pass; mid/4: levels of up to 1,570 tiles over both
# batches, four waves each, and the coarse level's 16-row tiles (levels of more than
# 2,048 tiles, a wave per narrow tile: test_gpu_block_paths.py)
SHAPES = {
    "ragged_p2": lambda: wl.small_box(n=(5, 3, 4), order=2, n_parts=(3, 2, 1), overlap=1, coarse=False),
    "one_tree_p2": lambda: wl.small_box(n=(14, 13, 12), order=2, n_parts=(1, 1, 1), overlap=1, coarse=False),
    "mid_quarter_2lvl": lambda: wl.mid(scale=4, n_parts=(4, 4, 1)),
}


# One Arnoldi step from zero, u = y M^{-1} b with y from the dots of A M^{-1} b:
# no stopping test decides anything, and both sides apply the same panels in
# FP64 (the local solves of the two agree to 1e-12, y to the same).
@pytest.mark.parametrize("nrhs", [2, 3, 5, 8])
@pytest.mark.parametrize("name,c64", [("ragged_p2", 0), ("ragged_p2", 1), ("one_tree_p2", 0), ("mid_quarter_2lvl", 0),
                                      ("mid_quarter_2lvl", 2)])
def test_narrow_blocks_match_single_solves(name, c64, nrhs):
    w = SHAPES[name]()
    h = helm.from_workload(w, c64=c64)
    print(f"[widths] {name} c64={c64} nrhs={nrhs}", flush=True)
    B = torch.stack([torch.from_numpy(wl.random_vector(h.n, 50 + k)) for k in range(nrhs)]).to("cuda")
    U, V = torch.zeros_like(B), torch.zeros_like(B)
    h.solve(B, U, tol=1e-14, restart=1, maxit=1, block=8)
    for k in range(nrhs):
        h.solve(B[k].contiguous(), V[k], tol=1e-14, restart=1, maxit=1)
        assert float((U[k] - V[k]).norm() / V[k].norm()) <= 1e-11


# The sparse kernels of a one-level block step (products, prolongation) over every
# width.  The box is attenuated in either case, so its rows are complex apart from the
# identity rows of the free surface (real and mixed rows, and a coarse stage:
# test_gpu_block_paths.py).  One step as above.
@pytest.mark.parametrize("nrhs", [2, 4, 7, 9, 16])
@pytest.mark.parametrize("attenuation", [0.0, 0.02])
def test_block_products_match_single_solves(attenuation, nrhs):
    w = wl.small_box(n=(6, 5, 4), order=2, n_parts=(2, 2, 1), overlap=2)
    w = dataclasses.replace(w, c_tet=w.c_tet * (1 - 1j * attenuation))
    h = helm.from_workload(w)
    print(f"[products] attenuation={attenuation} nrhs={nrhs}", flush=True)
    B = torch.stack([torch.from_numpy(wl.random_vector(h.n, 80 + k)) for k in range(nrhs)]).to("cuda")
    U, V = torch.zeros_like(B), torch.zeros_like(B)
    h.solve(B, U, tol=1e-14, restart=1, maxit=1, block=16)
    for k in range(nrhs):
        h.solve(B[k].contiguous(), V[k], tol=1e-14, restart=1, maxit=1)
        assert float((U[k] - V[k]).norm() / V[k].norm()) <= 1e-11
