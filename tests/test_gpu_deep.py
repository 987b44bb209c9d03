"""The passes of more than two steps per launch that the library takes by
itself (no launch shape set): bitwise equal to single steps in every storage
mode with either collision, from tiny lattices that wrap inside one tile to
several strips, and for step counts with every remainder, alone and batched
(launched directly, without graphs); and the first domain error is the oracle's
step and cell whichever step of a block pass it falls in.  (The library takes
the block pass at these sizes but for the two largest and two of the batches;
the other forms have their own tests in test_gpu_pass_forms.py.)  Every comparison is exact: each step runs the single step's routines on
the same values, rounded to the storage type in between."""
import numpy as np
import pytest
import torch

from paper_2003_07968_amd import lbm
from paper_2003_07968_amd import workloads as W

from .gpu_common import gpu_lattice, log, require_gpu
from .helpers import oracle_params

pytestmark = pytest.mark.gpu

# tiny and wrapping; one and several columns of blocks (18 cells wide), odd row
# counts; the last two in the deep pass
SIZES = [(3, 3), (5, 19), (17, 9), (50, 33), (51, 16), (64, 64), (114, 7), (115, 40), (242, 31),
         (243, 77), (18, 18), (19, 37), (200, 200), (301, 203), (640, 640), (1030, 517)]


def _case(nx, ny, storage, collision, seed=31, alt=False):
    p = W.params(nx, ny, tr=0.8, storage=storage, collision=collision, m2_trace_alt=alt,
                 mrt=(1.0, 0.9, 1.1, 1.0, 1.2))
    rg, rl = W.unit_cs_coexistence(0.8)
    rho0 = W.smooth_random(nx, ny, seed, mean=0.5 * (rg + rl), amplitude=0.5 * (rl - rg))
    p["rho_ref"] = W.shift_reference(rho0, storage)
    return p, rho0


@pytest.mark.parametrize("collision", ["bgk", "mrt"])
@pytest.mark.parametrize("storage", ["f64", "f32", "f16", "f16l"])
def test_default_steps_bitwise_equal_single_steps(storage, collision):
    require_gpu()
    for k, (nx, ny) in enumerate(SIZES):
        p, rho0 = _case(nx, ny, storage, collision, seed=31 + k, alt=k % 4 == 0)
        ref = gpu_lattice(p, rho0, launch=(256, 8))
        lat = gpu_lattice(p, rho0)
        for n in (8, 7, 13):  # passes from even and odd times, each remainder
            ref.step(n)
            lat.step(n)
            lat.sync()
            assert torch.equal(lat.populations(), ref.populations()), (nx, ny, n)


@pytest.mark.parametrize("collision", ["bgk", "mrt"])
@pytest.mark.parametrize("storage", ["f64", "f32", "f16", "f16l"])
@pytest.mark.parametrize("sizes", [SIZES, SIZES[:-2], [(24, 20)], [(1500, 700), (3, 3)]],
                         ids=["all", "small", "one", "large"])
def test_default_batch_bitwise_equal_single_steps(storage, collision, sizes):
    # sets of lattices that the library advances in either form of long pass
    require_gpu()
    with torch.cuda.stream(torch.cuda.Stream()):
        cases = [_case(nx, ny, storage, collision, seed=70 + k)
                 for k, (nx, ny) in enumerate(sizes)]
        solo = [gpu_lattice(p, r, launch=(256, 8)) for p, r in cases]
        mates = [gpu_lattice(p, r) for p, r in cases]
        batch = lbm.Batch(len(cases))
        for lat in mates:
            batch.add(lat)
        for n in (7, 16, 3, 24, 4):
            batch.step(n)
            _ = torch.zeros(4, device="cuda").sum().item()  # unrelated work between replays
            for s, m, size in zip(solo, mates, sizes):
                s.step(n)
                assert m.t == s.t
                assert torch.equal(s.populations(), m.populations()), (size, n)
        for m in mates:
            m.sync()


def test_a_set_shape_is_kept():
    # an explicit two-step shape, and back to the library's choice
    require_gpu()
    p, rho0 = _case(300, 257, "f64", "bgk")
    ref = gpu_lattice(p, rho0, launch=(256, 8))
    ref.step(22)
    lat = gpu_lattice(p, rho0, fusion=(2, 128, 9))
    assert lat.launch()[:2] == (128, 9)
    lat.step(10)
    lat.set_fusion(2)
    lat.step(12)
    assert torch.equal(lat.populations(), ref.populations())


@pytest.mark.parametrize("batched", [False, True])
@pytest.mark.parametrize("lead", [0, 1, 2])
@pytest.mark.parametrize("disk,step", [((4, 0.35, 0.2), 2), ((5, 0.35, 0.2), 3),
                                       ((6, 0.35, 0.2), 4), ((7, 0.35, 0.2), 5)])
def test_domain_error_same_step_and_cell(oracle, disk, step, lead, batched):
    # a disk whose rim moves inward leaves the EOS domain at a known later
    # step: with `lead` steps taken first, every step of a pass is covered
    require_gpu()
    radius, rho_disk, speed = disk
    yy, xx = np.mgrid[0:20, 0:24]
    dx, dy = xx - 11, yy - 9
    r = np.hypot(dx, dy)
    rho0 = np.where(r <= radius, rho_disk, 0.2)
    ring = (r <= radius) & (r > radius - 2.2)
    ux = np.where(ring, -speed * dx / np.maximum(r, 1), 0.0)
    uy = np.where(ring, -speed * dy / np.maximum(r, 1), 0.0)
    p = W.params(24, 20, tr=0.8)
    P = oracle_params(oracle, p)
    with pytest.raises(oracle.OracleError) as ref:
        oracle.step(P, oracle.init(P, rho0, ux, uy), 12)
    assert ref.value.fault.step == step
    with torch.cuda.stream(torch.cuda.Stream()):
        lat = gpu_lattice(p, rho0, ux, uy)
        if batched:
            batch = lbm.Batch(1)
            batch.add(lat)
        (batch if batched else lat).step(lead)
        (batch if batched else lat).step(16)
        with pytest.raises(lbm.LbmError) as e:
            lat.sync()
        assert e.value.status == lbm.LBM_ERR_DOMAIN
        msg = lbm.lbm_last_error(lat.handle)
    log(f"  {msg}")
    assert f"step {step}," in msg and f"cell {ref.value.fault.cell} " in msg
