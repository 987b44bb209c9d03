"""Which pass takes the steps: lbm_get_pass and lbm_batch_get_pass report it,
lbm_set_pass and lbm_batch_set_pass choose it."""
import pytest
import torch

from paper_2003_07968_amd import lbm
from paper_2003_07968_amd import workloads as W

from .gpu_common import gpu_lattice, log, require_gpu

pytestmark = pytest.mark.gpu


def _lattice(nx, ny, storage="f64", force=True, **kw):
    p = W.params(nx, ny, tr=0.8, storage=storage)
    p["force_on"] = force
    rg, rl = W.unit_cs_coexistence(0.8)
    rho0 = W.smooth_random(nx, ny, 9, mean=0.5 * (rg + rl), amplitude=0.4 * (rl - rg))
    p["rho_ref"] = W.shift_reference(rho0, storage)
    return gpu_lattice(p, rho0, **kw)


def _batch(*lats):
    batch = lbm.Batch(len(lats))
    for lat in lats:
        batch.add(lat)
    return batch


def test_reported_pass_follows_every_way_to_set_one():
    require_gpu()
    lat = _lattice(64, 64)
    assert lat.get_pass() == (4, lbm.LBM_PASS_BLOCK, 16, 0)
    lat.set_pass(lbm.LBM_PASS_DEEP, 64, 5)
    assert lat.get_pass() == (4, lbm.LBM_PASS_DEEP, 64, 5) and lat.fusion() == 2
    lat.set_pass(lbm.LBM_PASS_SHORT)
    assert lat.get_pass() == (2, lbm.LBM_PASS_SHORT, 0, 0)
    lat.set_pass(lbm.LBM_PASS_DEFAULT)
    assert lat.get_pass() == (4, lbm.LBM_PASS_BLOCK, 16, 0)
    lat.set_fusion(2, 128, 9)
    assert lat.get_pass() == (2, lbm.LBM_PASS_SHORT, 0, 0)
    lat.set_fusion(1)
    assert lat.get_pass() == (1, lbm.LBM_PASS_SHORT, 0, 0)
    lat.set_fusion(2)
    assert lat.get_pass()[:2] == (4, lbm.LBM_PASS_BLOCK)
    big = _lattice(1200, 900)
    steps, form, width, rows = big.get_pass()
    assert (steps, form) == (4, lbm.LBM_PASS_DEEP) and width in (64, 128, 256) and rows > 1
    assert _lattice(64, 64, force=False).get_pass() == (2, lbm.LBM_PASS_SHORT, 0, 0)


def test_bad_passes_are_refused_and_change_nothing():
    require_gpu()
    lat = _lattice(96, 64)
    batch = _batch(_lattice(96, 64))
    for target in (lat, batch):
        before = target.get_pass()
        for bad in ((3,), (-2,), (lbm.LBM_PASS_DEEP, 192, 8), (lbm.LBM_PASS_DEEP, 256, 0),
                    (lbm.LBM_PASS_BLOCK, 28), (lbm.LBM_PASS_BLOCK, 16, 4),
                    (lbm.LBM_PASS_SHORT, 256), (lbm.LBM_PASS_DEFAULT, 0, 8)):
            with pytest.raises(lbm.LbmError) as e:
                target.set_pass(*bad)
            assert e.value.status == lbm.LBM_ERR_INVALID_ARG and target.get_pass() == before, bad
        target.set_fusion(1)
        with pytest.raises(lbm.LbmError):
            target.set_pass(lbm.LBM_PASS_DEEP, 256, 8)
    no_force = _lattice(64, 64, force=False)
    with pytest.raises(lbm.LbmError):
        no_force.set_pass(lbm.LBM_PASS_BLOCK, 16)


def test_a_batch_returns_to_the_library_choice_and_to_a_tuned_pass():
    require_gpu()
    with torch.cuda.stream(torch.cuda.Stream()):
        ref = _lattice(200, 150, "f32", launch=(256, 8))
        lat = _lattice(200, 150, "f32")
        batch = _batch(lat)
        default = batch.get_pass()
        assert default[:2] == (4, lbm.LBM_PASS_BLOCK)
        batch.set_launch(2, 256, 0)      # pins the two-step pass
        assert batch.get_pass()[:2] == (2, lbm.LBM_PASS_SHORT) and batch.launch()[0] == 2
        batch.step(10)
        batch.set_pass(lbm.LBM_PASS_DEFAULT)
        assert batch.get_pass() == default
        batch.step(10)
        batch.autotune()
        tuned = batch.get_pass()
        log(f"  tuned: {tuned}")
        batch.set_launch(1, 128, 3)
        batch.step(3)
        assert batch.get_pass() == (1, lbm.LBM_PASS_SHORT, 0, 0)
        batch.set_fusion(2)
        if tuned[0] == 4:
            batch.set_pass(*tuned[1:])
            assert batch.get_pass() == tuned
        batch.step(9)
        ref.step(32)
        assert lat.t == 32 and torch.equal(lat.populations(), ref.populations())


def test_a_large_batch_whose_shape_is_chosen_by_a_sample():
    # more members than the choice looks at, the largest at a place that it
    # skips: bitwise the single steps' results
    require_gpu()
    with torch.cuda.stream(torch.cuda.Stream()):
        sizes = [(16 + k % 23, 16 + k % 19) for k in range(600)]
        sizes[301] = (700, 500)
        lats = [_lattice(nx, ny, "f32") for nx, ny in sizes]
        batch = _batch(*lats)
        assert batch.get_pass()[0] == 4
        batch.step(11)
        for k in (0, 1, 2, 300, 301, 302, 450, 599):
            ref = _lattice(*sizes[k], "f32", launch=(256, 8))
            ref.step(11)
            lats[k].sync()
            assert torch.equal(lats[k].populations(), ref.populations()), sizes[k]
