"""The calls that wait report the lattice's own status: an error that the
host program's own HIP calls have left in the runtime is not theirs."""
import ctypes

import pytest
import torch

from paper_2003_07968_amd import lbm
from paper_2003_07968_amd import workloads as W

from .gpu_common import gpu_lattice, require_gpu

pytestmark = pytest.mark.gpu


def _hip():
    with open("/proc/self/maps") as maps:
        path = next(line.split()[-1] for line in maps if "libamdhip64" in line)
    return ctypes.CDLL(path)


def test_sync_after_a_failed_call_of_the_host_program():
    require_gpu()
    hip = _hip()
    p, rho0 = W.droplet_64(seed=5)
    lat = gpu_lattice(p, rho0)
    lat.step(6)
    lat.sync()
    try:
        assert hip.hipSetDevice(4096) != 0   # an ordinary host-side error
        lat.sync()
    finally:
        hip.hipGetLastError()                # torch would report it next
    assert lat.t == 6
    assert torch.isfinite(lat.moments()["rho"]).all()
    assert lbm.lbm_sync(lat.handle) == lbm.LBM_OK
