"""Both single-vector sweeps in one launch (workgroups that wait for the tiles
they depend on) against one launch per level (which a sn_jobs_min of the caller's
own asks for), and under graph capture."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2004_06309_amd import helm  # noqa: E402
from paper_2004_06309_amd import workloads as wl  # noqa: E402

SHAPES = {
    # one leaf: a root without children, nothing to wait for
    "one_leaf_p1": lambda: wl.small_box(n=(2, 1, 1), order=1, n_parts=(1, 1, 1), overlap=1, coarse=False),
    # subdomains of a few leaves, remainders of every tile height
    "ragged_p2": lambda: wl.small_box(n=(5, 3, 4), order=2, n_parts=(3, 2, 1), overlap=1, coarse=False),
    "small_p2_2lvl": lambda: wl.small_box(n=(6, 6, 4), order=2, n_parts=(2, 2, 1), overlap=2),
    # one deep tree: tiles of up to 998 columns split over row ranges (wider than an
    # LDS pass: test_gpu_flow_passes.py)
    "one_tree_p2": lambda: wl.small_box(n=(14, 13, 12), order=2, n_parts=(1, 1, 1), overlap=1, coarse=False),
    "mid_quarter_2lvl": lambda: wl.mid(scale=4, n_parts=(4, 4, 1)),
}


def _vec(n, seed):
    return torch.from_numpy(wl.random_vector(n, seed)).to("cuda")


# The two forms sum the same products in another order: a row has at most a
# few thousand terms per level and about 20 levels, 2e4 x 2^-53 = 2e-12 at
# worst and its square root in practice; the levels' own forms agree to 1e-12.
@pytest.mark.parametrize("c64", [0, 1, 2])
@pytest.mark.parametrize("name", list(SHAPES))
def test_flow_matches_level_launches(name, c64):
    w = SHAPES[name]()
    print(f"[flow] {name} c64={c64}", flush=True)
    hf = helm.from_workload(w, c64=c64)
    hl = helm.from_workload(w, c64=c64, sn_jobs_min=1 << 30)
    zf, zl = (torch.empty(hf.n, dtype=torch.complex128, device="cuda") for _ in range(2))
    for seed in (1, 2):
        r = _vec(hf.n, seed)
        hf.apply_oras(r, zf)
        hl.apply_oras(r, zl)
        assert float((zf - zl).norm() / zl.norm()) <= 1e-12
        # repeated, and with kernel timing on (the sweeps launched apart): bit for bit
        hf.apply_oras(r, zl)
        assert torch.equal(zf, zl)
        hf.profile(True)
        hf.apply_oras(r, zl)
        hf.profile(False)
        assert torch.equal(zf, zl)


@pytest.mark.parametrize("tile_rows", [16, 32])
def test_flow_other_tile_heights(tile_rows):
    w = SHAPES["ragged_p2"]()
    hf = helm.from_workload(w, tile_rows=tile_rows)
    hl = helm.from_workload(w, tile_rows=tile_rows, sn_jobs_min=1 << 30)
    r = _vec(hf.n, 3)
    zf, zl = torch.empty_like(r), torch.empty_like(r)
    hf.apply_oras(r, zf)
    hl.apply_oras(r, zl)
    assert float((zf - zl).norm() / zl.norm()) <= 1e-12


def test_flow_replays_from_a_graph():
    """Every sweep finds its counters clear, so captured and eager applications may
    alternate."""
    w = SHAPES["small_p2_2lvl"]()
    h = helm.from_workload(w)
    r = _vec(h.n, 4)
    z, ref = torch.empty_like(r), torch.empty_like(r)
    h.apply_precond(r, z)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        h.apply_precond(r, z)
    for seed in (5, 6, 7):
        r.copy_(_vec(h.n, seed))
        h.apply_precond(r, ref)
        z.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(z, ref)
        g.replay()
        h.apply_precond(r, ref)
        torch.cuda.synchronize()
        assert np.array_equal(z.cpu().numpy(), ref.cpu().numpy())
