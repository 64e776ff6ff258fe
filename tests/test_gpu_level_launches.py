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


@pytest.mark.parametrize("nb", [2, 3, 4])
@pytest.mark.parametrize("c64", [0, 1, 2])
@pytest.mark.parametrize("name", list(SHAPES))
def test_batches_on_level_launches(name, c64, nb):
    """Two, three and four batches, each on a stream of its own, against one: the
    same tiles and sums, so bit for bit, also with kernel timing on (the batches
    one after the other), repeated, and on another input."""
    w = SHAPES[name]()
    h1 = helm.from_workload(w, c64=c64, batches=1, sn_jobs_min=1 << 30)
    hk = helm.from_workload(w, c64=c64, batches=nb, sn_jobs_min=1 << 30)
    assert hk.stats()["batches"] == nb and h1.stats()["batches"] == 1
    print(f"[batches] {name} c64={c64} x{nb}", flush=True)
    for seed in (6, 7):
        r = torch.from_numpy(wl.random_vector(h1.n, seed)).to("cuda")
        z1, zk = torch.empty_like(r), torch.empty_like(r)
        h1.apply_oras(r, z1)
        for _ in range(2):
            hk.apply_oras(r, zk)
            assert torch.equal(zk, z1)
        zk.zero_()
        assert _forward_launches(hk, r, zk) > nb
        assert torch.equal(zk, z1)
