"""Which form the single-vector sweeps take, one launch or one per level, and the
launches per level themselves: subdomain batches on their own streams."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2004_06309_amd import helm  # noqa: E402
from paper_2004_06309_amd import workloads as wl  # noqa: E402

SHAPES = {
    "ragged_p2": lambda: wl.small_box(n=(5, 3, 4), order=2, n_parts=(3, 2, 1), overlap=1, coarse=False),
    "mid_quarter_2lvl": lambda: wl.mid(scale=4, n_parts=(4, 4, 1)),
}


def _forward_launches(h, r, z):
    h.profile(True)
    h.apply_oras(r, z)
    torch.cuda.synchronize()
    k = h.profile_read()["trsv_fwd"]["launches"]
    h.profile(False)
    return k


@pytest.mark.parametrize("value,one", [(0, True), (6144, True), (-1, True), (1, False), (1 << 30, False)])
def test_the_line_of_one_wave_jobs_chooses_the_form(value, one):
    """The default of sn_jobs_min, given or not, leaves a small operator with one
    launch; a line of the caller's own asks for level launches."""
    h = helm.from_workload(SHAPES["ragged_p2"](), sn_jobs_min=value)
    r = torch.from_numpy(wl.random_vector(h.n, 5)).to("cuda")
    n = _forward_launches(h, r, torch.empty_like(r))
    assert (n == 1) if one else (n > h.stats()["batches"])
