"""Steps recorded in a HIP graph of the host program's own.  Every launch
exchanges the two population buffers, so a graph whose call takes an even number
of one- and two-step launches (3, 4, 7, 8, 11, 12, ... steps) goes on from its own
result when it is replayed; each replay, with unrelated eager work and
synchronizations in between, equals as many single steps taken eagerly."""
import pytest
import torch

from paper_2003_07968_amd import lbm
from paper_2003_07968_amd import workloads as W

from .gpu_common import gpu_lattice, require_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batched", [False, True])
@pytest.mark.parametrize("size", [(64, 64), (700, 640)], ids=["block", "deep"])
@pytest.mark.parametrize("n", [3, 4, 7, 8, 12, 20])
def test_replays_of_a_captured_call_go_on(n, size, batched):
    require_gpu()
    nx, ny = size
    p = W.params(nx, ny, tr=0.8)
    rg, rl = W.unit_cs_coexistence(0.8)
    rho0 = W.smooth_random(nx, ny, 77, mean=0.5 * (rg + rl), amplitude=0.4 * (rl - rg))
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        ref = gpu_lattice(p, rho0, launch=(256, 8))
        lat = gpu_lattice(p, rho0)
        target = lat
        if batched:
            target = lbm.Batch(1)
            target.add(lat)
        form = target.get_pass()[1]   # (writes a batch's table before the capture)
        assert form == (lbm.LBM_PASS_BLOCK if nx == 64 else lbm.LBM_PASS_DEEP)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            target.step(n)
        f = torch.empty((9, ny, nx), dtype=torch.float64, device="cuda")
        for k in range(3):
            graph.replay()
            _ = torch.zeros(4, device="cuda").sum().item()
            ref.step(n)
            lbm.lbm_get_populations(lat.handle, f)
            assert torch.equal(f, ref.populations()), k
        lat.sync()
