"""Both sweeps in one launch where a tile is wider than the LDS input buffer and is
taken in several passes, against one launch per level."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2004_06309_amd import helm  # noqa: E402
from paper_2004_06309_amd import workloads as wl  # noqa: E402


# One subdomain whose first separator is a plane of 49 x 25 P2 unknowns: forward
# tiles of up to 1,225 columns, backward ones of up to 1,776, buffers of 1,024.
# The two forms sum the same products in another order: a row has at most a few
# thousand terms per level and about 20 levels, 2e4 x 2^-53 = 2e-12 at worst and its
# square root in practice; the levels' own forms agree to 1e-12.
@pytest.mark.parametrize("c64", [0, 1, 2])
def test_tiles_wider_than_a_pass(c64):
    w = wl.small_box(n=(24, 24, 12), order=2, n_parts=(1, 1, 1), overlap=1, coarse=False)
    hf = helm.from_workload(w, c64=c64)
    hl = helm.from_workload(w, c64=c64, sn_jobs_min=1 << 30)
    assert hf.stats()["max_front"] > 1024 and hf.stats()["factor_entries"] <= 3e8
    print(f"[flow] passes c64={c64}", flush=True)
    zf, zl = (torch.empty(hf.n, dtype=torch.complex128, device="cuda") for _ in range(2))
    for seed in (1, 2):
        r = torch.from_numpy(wl.random_vector(hf.n, seed)).to("cuda")
        hf.apply_oras(r, zf)
        hl.apply_oras(r, zl)
        assert float((zf - zl).norm() / zl.norm()) <= 1e-12
        hf.apply_oras(r, zl)
        assert torch.equal(zf, zl)
