"""Applications of the preconditioner that a solve enqueues ahead of the host's
decision: none of them is wasted where convergence is steady."""
import time

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2004_06309_amd import helm  # noqa: E402
from paper_2004_06309_amd import workloads as wl  # noqa: E402


@pytest.mark.parametrize("classic", [False, True])
@pytest.mark.parametrize("nx", [8, 16, 24])
def test_short_solves_apply_the_preconditioner_once_per_step(nx, classic):
    from torch.profiler import ProfilerActivity, profile

    w = wl.tiny(nx=nx)
    h = helm.from_workload(w)
    b = torch.from_numpy(h.point_source((500.0, 500.0, 100.0))).to("cuda")
    u = torch.zeros_like(b)
    for tol in (0.5, 1e-1, 1e-2, 1e-3, 1e-4, 1e-6):
        with profile(activities=[ProfilerActivity.CUDA]) as prof:
            time.sleep(0.05)  # the profiler drops kernels at the ends of its window
            rc, info = h.solve(b, u, tol=tol, restart=50, classic_cgs2=classic)
            torch.cuda.synchronize()
            time.sleep(0.05)
        sweeps = sum(e.count for e in prof.key_averages() if "flow_kernel" in e.key)
        if not sweeps:
            pytest.skip("the profiler reported no kernels")
        print(f"[ahead] n={h.n} classic={classic} tol={tol}: {info[0]['iterations']} steps, {sweeps} sweeps", flush=True)
        assert rc == helm.HELM_OK and sweeps <= info[0]["iterations"]
