"""The kernels between two preconditioner applications of a GMRES step on both
sides of their size lines: delayed against classical Gram-Schmidt, and a step
enqueued ahead of the host's decision against one that is not."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2004_06309_amd import helm  # noqa: E402
from paper_2004_06309_amd import workloads as wl  # noqa: E402

SHAPES = {
    "one_tile": lambda: wl.small_box(n=(3, 3, 2), order=1, n_parts=(2, 1, 1), overlap=1, coarse=False),
    "two_level": lambda: wl.small_box(n=(6, 6, 4), order=2, n_parts=(2, 2, 1), overlap=2),
    # 16,384 unknowns: 256 tiles of 64 rows, the most of one launch; 16,896: 264
    "tiles_256": lambda: wl.small_box(n=(31, 31, 15), order=1, n_parts=(3, 3, 1), overlap=1, coarse=False),
    "tiles_264": lambda: wl.small_box(n=(32, 31, 15), order=1, n_parts=(3, 3, 1), overlap=1, coarse=False),
}


# Twelve steps with a restart after eight: both orthogonalisations are exact to
# a few eps, and a least-squares problem of eight preconditioned columns has a
# condition far below 1e4, so the two solutions agree to 1e-12 times that.
@pytest.mark.parametrize("nrhs", [1, 3])
@pytest.mark.parametrize("name", list(SHAPES))
def test_delayed_and_classical_steps_agree(name, nrhs):
    h = helm.from_workload(SHAPES[name]())
    print(f"[steps] {name} n={h.n} nrhs={nrhs}", flush=True)
    B = torch.stack([torch.from_numpy(wl.random_vector(h.n, 20 + k)) for k in range(nrhs)]).to("cuda")
    U, V = torch.zeros_like(B), torch.zeros_like(B)
    kw = dict(tol=1e-14, restart=8, maxit=12, block=nrhs)
    h.solve(B, U, **kw)
    h.solve(B, V, classic_cgs2=True, **kw)
    assert float((U - V).norm() / V.norm()) <= 1e-8


# Kernel timing turns the early enqueueing off (with two levels it is off on both
# sides): the same kernels, bit for bit,
# also where the cycle ends at the restart length, at maxit or by convergence.
@pytest.mark.parametrize("kw", [dict(tol=1e-14, restart=4, maxit=9), dict(tol=1e-3, restart=50, maxit=60)])
@pytest.mark.parametrize("name", ["one_tile", "two_level", "tiles_256"])
def test_steps_ahead_change_nothing(name, kw):
    h = helm.from_workload(SHAPES[name]())
    print(f"[steps] {name} {kw}", flush=True)
    b = torch.from_numpy(wl.random_vector(h.n, 40)).to("cuda")
    u, v = torch.zeros_like(b), torch.zeros_like(b)
    h.solve(b, u, **kw)
    h.profile(True)
    h.solve(b, v, **kw)
    h.profile(False)
    assert torch.equal(u, v)
