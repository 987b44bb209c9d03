"""Batches in the two-step pass (a launch shape that is set keeps the longer
passes away): eager launches and replays of the captured eight-step graphs,
against lattices stepped alone and against the oracle; on the legacy null stream,
which cannot be captured, eager launches alone."""
import pytest
import torch

from paper_2003_07968_amd import lbm
from paper_2003_07968_amd import workloads as W

from .gpu_common import PARITY_TOL, assert_parity, gpu_lattice, gpu_state, oracle_state, require_gpu
from .helpers import oracle_params

pytestmark = pytest.mark.gpu


def _two_step_batch(lats):
    batch = lbm.Batch(len(lats))
    for lat in lats:
        batch.add(lat)
    batch.set_launch(2, 256, 0)
    assert batch.get_pass()[:2] == (2, lbm.LBM_PASS_SHORT)
    return batch


@pytest.mark.parametrize("null_stream", [False, True])
@pytest.mark.parametrize("storage", ["f64", "f32", "f16", "f16l"])
def test_two_step_batch_equals_alone(storage, null_stream):
    require_gpu()
    stream = torch.cuda.default_stream() if null_stream else torch.cuda.Stream()
    with torch.cuda.stream(stream):
        cases = W.batch_case(count=6, seed=3, storage=storage, side_range=(24, 160))
        solo = [gpu_lattice(p, r, launch=(256, 8)) for p, r in cases]
        mates = [gpu_lattice(p, r) for p, r in cases]
        batch = _two_step_batch(mates)
        done = 0
        for n in (3, 8, 8, 1, 16, 5, 2):
            batch.step(n)
            for s in solo:
                s.step(n)
            done += n
            _ = torch.zeros(4, device="cuda").sum().item()  # unrelated eager work
            for k, (s, m) in enumerate(zip(solo, mates)):
                assert m.t == s.t == done
                assert torch.equal(s.populations(), m.populations()), (storage, k, done)
        for m in mates:
            m.sync()


@pytest.mark.parametrize("collision", ["bgk", "mrt"])
def test_two_step_graph_replays_match_oracle(oracle, collision):
    require_gpu()
    with torch.cuda.stream(torch.cuda.Stream()):
        cases = W.batch_case(count=3, seed=21, storage="f64", side_range=(20, 72))
        for p, _ in cases:
            if collision == "mrt":
                p.update(collision=W.COLLISION["mrt"], tau_e=0.9, tau_zeta=1.1, tau_q=1.2)
        lats = [gpu_lattice(p, r) for p, r in cases]
        batch = _two_step_batch(lats)
        refs = [(oracle_params(oracle, p), oracle.init(oracle_params(oracle, p), r))
                for p, r in cases]
        done = 0
        for n in (8, 32):
            batch.step(n)
            done += n
            for (p, _), lat, (P, f) in zip(cases, lats, refs):
                oracle.step(P, f, n)
                lat.sync()
                assert lat.t == done
                assert_parity(gpu_state(lat), oracle_state(oracle, P, f), PARITY_TOL,
                              f"{p['nx']}x{p['ny']} {collision} t={done}")
