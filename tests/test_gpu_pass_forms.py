"""Every form of the passes of more than two steps, chosen with lbm_set_pass and
lbm_batch_set_pass: the deep pass with workgroups of 64, 128 and 256 columns,
of four and of three steps, and the block pass with regions of 16 to 32 rows.
Populations are bitwise those of single steps in every storage mode, with either
collision, alone and batched; the first domain error is the oracle's step and
cell whichever step of a deep pass and whichever walk direction it falls in.

Sizes: lattices that wrap inside one tile; one strip of each workgroup width
filled to the last column (50, 114 and 242) and one column more; several
strips with a remainder; segments of one row, of a few and of the whole
lattice, so that bands walk up and down."""
import numpy as np
import pytest
import torch

from paper_2003_07968_amd import lbm
from paper_2003_07968_amd import workloads as W

from .gpu_common import gpu_lattice, log, require_gpu
from .helpers import oracle_params

pytestmark = pytest.mark.gpu

FORMS = [(lbm.LBM_PASS_DEEP, bx, rows) for bx in (64, 128, 256) for rows in (1, 7, 400)] + \
        [(lbm.LBM_PASS_BLOCK, rows, 0) for rows in (16, 20, 24, 32)]
SIZES = [(3, 3), (5, 19), (50, 12), (51, 33), (114, 16), (115, 9), (242, 7), (243, 31), (301, 40)]


def _id(form):
    return f"{'deep' if form[0] == lbm.LBM_PASS_DEEP else 'block'}{form[1]}x{form[2]}"


def _case(nx, ny, storage, collision, seed):
    p = W.params(nx, ny, tr=0.8, storage=storage, collision=collision,
                 m2_trace_alt=seed % 4 == 0, mrt=(1.0, 0.9, 1.1, 1.0, 1.2))
    rg, rl = W.unit_cs_coexistence(0.8)
    rho0 = W.smooth_random(nx, ny, seed, mean=0.5 * (rg + rl), amplitude=0.5 * (rl - rg))
    p["rho_ref"] = W.shift_reference(rho0, storage)
    return p, rho0


@pytest.mark.parametrize("collision", ["bgk", "mrt"])
@pytest.mark.parametrize("storage", ["f64", "f32", "f16", "f16l"])
def test_every_form_bitwise_equal_single_steps(storage, collision):
    require_gpu()
    for k, (nx, ny) in enumerate(SIZES):
        p, rho0 = _case(nx, ny, storage, collision, 300 + k)
        ref = gpu_lattice(p, rho0, launch=(256, 8))
        states = []
        for n in (8, 3, 7, 5):   # passes of four and of three steps, remainders
            ref.step(n)
            states.append((n, ref.populations()))
        for form in FORMS:
            lat = gpu_lattice(p, rho0)
            lat.set_pass(*form)
            assert lat.get_pass() == (4,) + form
            for n, f in states:
                lat.step(n)
                assert torch.equal(lat.populations(), f), (nx, ny, _id(form), n)
            lat.sync()


@pytest.mark.parametrize("collision", ["bgk", "mrt"])
@pytest.mark.parametrize("storage", ["f64", "f32", "f16", "f16l"])
def test_every_form_of_a_batch_bitwise_equal_single_steps(storage, collision):
    require_gpu()
    with torch.cuda.stream(torch.cuda.Stream()):
        cases = [_case(nx, ny, storage, collision, 400 + k) for k, (nx, ny) in enumerate(SIZES)]
        refs = [gpu_lattice(p, r, launch=(256, 8)) for p, r in cases]
        states = []
        for n in (8, 3, 7, 5):
            for s in refs:
                s.step(n)
            states.append((n, [s.populations() for s in refs]))
        for form in FORMS:
            lats = [gpu_lattice(p, r) for p, r in cases]
            batch = lbm.Batch(len(lats))
            for lat in lats:
                batch.add(lat)
            batch.set_pass(*form)
            assert batch.get_pass() == (4,) + form
            for n, fs in states:
                batch.step(n)
                for lat, f, size in zip(lats, fs, SIZES):
                    assert torch.equal(lat.populations(), f), (size, _id(form), n)
            for lat in lats:
                lat.sync()


def _disk(nx, ny, cx, cy, radius, rho_disk, speed):
    """A disk whose rim moves inward leaves the EOS domain at a known later step."""
    yy, xx = np.mgrid[0:ny, 0:nx]
    dx, dy = xx - cx, yy - cy
    r = np.hypot(dx, dy)
    rho0 = np.where(r <= radius, rho_disk, 0.2)
    ring = (r <= radius) & (r > radius - 2.2)
    ux = np.where(ring, -speed * dx / np.maximum(r, 1), 0.0)
    uy = np.where(ring, -speed * dy / np.maximum(r, 1), 0.0)
    return rho0, ux, uy


# the failing cell in an upward and in a downward band, in the first strip's
# interior and at a strip boundary (strips of 48 columns at 64-column workgroups)
@pytest.mark.parametrize("cx,cy", [(20, 9), (48, 30)])
@pytest.mark.parametrize("disk,step", [((4, 0.35, 0.2), 2), ((5, 0.35, 0.2), 3),
                                       ((6, 0.35, 0.2), 4), ((7, 0.35, 0.2), 5)])
def test_deep_pass_domain_error_same_step_and_cell(oracle, disk, step, cx, cy):
    require_gpu()
    nx, ny = 101, 40
    p = W.params(nx, ny, tr=0.8)
    fields = _disk(nx, ny, cx, cy, *disk)
    P = oracle_params(oracle, p)
    with pytest.raises(oracle.OracleError) as ref:
        oracle.step(P, oracle.init(P, *fields), 12)
    assert ref.value.fault.step == step
    msgs = set()
    with torch.cuda.stream(torch.cuda.Stream()):
        for batched in (False, True):
            for form in ((lbm.LBM_PASS_DEEP, 64, 20), (lbm.LBM_PASS_DEEP, 64, 3),
                         (lbm.LBM_PASS_DEEP, 128, 40), (lbm.LBM_PASS_DEEP, 256, 11)):
                for calls in ((16,), (1, 16), (2, 16), (3, 3, 3), (1, 3, 3)):
                    lat = gpu_lattice(p, *fields)
                    target = lat
                    if batched:
                        target = lbm.Batch(1)
                        target.add(lat)
                    target.set_pass(*form)
                    for n in calls:
                        target.step(n)
                    with pytest.raises(lbm.LbmError) as e:
                        lat.sync()
                    assert e.value.status == lbm.LBM_ERR_DOMAIN
                    msgs.add(lbm.lbm_last_error(lat.handle))
    log(f"  {msgs}")
    assert len(msgs) == 1
    msg = msgs.pop()
    assert f"step {step}," in msg and f"cell {ref.value.fault.cell} " in msg
