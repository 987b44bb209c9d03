"""The autotuners leave the lattice's error word alone: their timed launches
check the EOS at steps that are not taken (up to three past t), and a lattice
that would leave its domain there is still valid after tuning.  Once it is
stepped, the first error is the oracle's step and cell."""
import numpy as np
import pytest
import torch

from paper_2003_07968_amd import lbm
from paper_2003_07968_amd import workloads as W

from .gpu_common import gpu_lattice, log, require_gpu
from .helpers import oracle_params

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batched", [False, True])
@pytest.mark.parametrize("disk,step,lead", [((4, 0.35, 0.2), 2, 1), ((4, 0.35, 0.2), 2, 0),
                                            ((5, 0.35, 0.2), 3, 0)])
def test_autotune_records_no_error_of_steps_not_taken(oracle, disk, step, lead, batched):
    # a disk whose rim moves inward leaves the domain at `step`; tuned at
    # t = lead, one to three steps earlier
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
        target = lat
        if batched:
            target = lbm.Batch(1)
            target.add(lat)
        target.step(lead)
        target.autotune()
        assert lat.t == lead
        lat.sync()
        target.step(16)
        with pytest.raises(lbm.LbmError) as e:
            lat.sync()
        assert e.value.status == lbm.LBM_ERR_DOMAIN
        msg = lbm.lbm_last_error(lat.handle)
    log(f"  {msg}")
    assert f"step {step}," in msg and f"cell {ref.value.fault.cell} " in msg
