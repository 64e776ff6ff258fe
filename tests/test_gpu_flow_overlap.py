"""Applications of one context on two streams without an order between them: what
they return is undefined, but the context has to give the same results as before
afterwards."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2004_06309_amd import helm  # noqa: E402
from paper_2004_06309_amd import workloads as wl  # noqa: E402


CALLS = {
    "oras": lambda h, r, z: h.apply_oras(r, z),
    "coarse": lambda h, r, z: h.apply_coarse(r, z),
    "precond": lambda h, r, z: h.apply_precond(r, z),
    "coarse_noalloc": lambda h, r, z: h.apply_coarse_noalloc(r, z),
}


@pytest.mark.parametrize("name", list(CALLS))
def test_a_context_survives_overlapping_applications(name):
    h = helm.from_workload(wl.small_box(n=(10, 10, 6), order=2, n_parts=(3, 2, 1), overlap=2))
    call = CALLS[name]
    r = torch.from_numpy(wl.random_vector(h.n, 11)).to("cuda")
    z, ref = torch.empty_like(r), torch.empty_like(r)
    call(h, r, ref)
    torch.cuda.synchronize()
    assert bool(torch.isfinite(torch.view_as_real(ref)).all())
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    outs = [torch.empty_like(r) for _ in streams]
    for rep in range(4):
        for _ in range(10):
            for s, o in zip(streams, outs):
                with torch.cuda.stream(s):
                    call(h, r, o)
        torch.cuda.synchronize()
        print(f"[overlap] {name} {rep}: spoilt {sum(not torch.equal(o, ref) for o in outs)} of 2", flush=True)
        for _ in range(3):
            call(h, r, z)
            torch.cuda.synchronize()
            assert torch.equal(z, ref)
