"""The path that the library takes by itself at the sizes of the benchmark and
above, element by element: the four 2048 x 2048 slabs as one batch through the
deep pass (a launch of four steps and one of three) against the oracle, in every
storage mode, and 8192 x 8192 against single steps."""
import pytest
import torch

from paper_2003_07968_amd import lbm
from paper_2003_07968_amd import workloads as W

from .gpu_common import (PARITY_TOL, assert_parity, gpu_lattice, gpu_state, log, oracle_state,
                         require_gpu)
from .helpers import oracle_params
from .test_gpu_storage import EMULATED_TOL

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("storage,collision", [("f64", "bgk"), ("f64", "mrt"), ("f32", "bgk"),
                                               ("f16", "bgk"), ("f16l", "bgk")])
def test_full_size_batch_in_the_default_pass(oracle, storage, collision):
    require_gpu()
    import bench
    tol = PARITY_TOL if storage == "f64" else EMULATED_TOL[storage]
    with torch.cuda.stream(torch.cuda.Stream()):
        cases = []
        for tr in bench.TEMPS:
            p, rho0 = W.slab_case(n=bench.N, tr=tr)
            p["storage"] = W.STORAGE[storage]
            p["rho_ref"] = W.shift_reference(rho0, storage)
            p["collision"] = W.COLLISION[collision]
            cases.append((p, rho0))
        lats = [gpu_lattice(p, rho0) for p, rho0 in cases]
        batch = lbm.Batch(len(lats))
        for lat in lats:
            batch.add(lat)
        used = batch.get_pass()
        log(f"case four 2048x2048 slabs as one batch, {storage} {collision}, pass {used}")
        assert used[:2] == (4, lbm.LBM_PASS_DEEP)
        refs = []
        for p, rho0 in cases:
            P = oracle_params(oracle, p)
            refs.append((P, oracle.init(P, rho0)))
        for n, t in ((4, 4), (3, 7)):
            batch.step(n)
            torch.cuda.synchronize()
            for lat, (P, f), tr in zip(lats, refs, bench.TEMPS):
                oracle.step(P, f, n)
                assert lat.t == t
                assert_parity(gpu_state(lat), oracle_state(oracle, P, f), tol,
                              f"T_r={tr} t={t}")
        for lat in lats:
            lat.sync()


@pytest.mark.parametrize("storage", ["f64", "f32"])
def test_8192_bitwise_equal_single_steps(storage):
    require_gpu()
    n = 8192
    rg, rl = W.unit_cs_coexistence(0.8)
    rho0 = W.smooth_random(n, n, 61, mean=0.5 * (rg + rl), amplitude=0.45 * (rl - rg), modes=6)
    rho0 += W.noise((n, n), 62)
    p = W.params(n, n, tr=0.8, storage=storage)
    p["rho_ref"] = W.shift_reference(rho0, storage)
    lat = gpu_lattice(p, rho0)
    assert lat.get_pass()[:2] == (4, lbm.LBM_PASS_DEEP)
    lat.step(11)   # two launches of four steps and one of three
    lat.sync()
    f = lat.populations()
    lat.close()
    del lat
    ref = gpu_lattice(p, rho0, launch=(0, 0))   # single steps, default shape
    ref.step(11)
    assert torch.equal(f, ref.populations())
