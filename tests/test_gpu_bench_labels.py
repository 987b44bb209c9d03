"""bench.py's kernel label, steps per launch, launch shape and launch count are
those of the launches that ran, for every way to choose them."""
import pytest

from paper_2003_07968_amd import lbm

from .gpu_common import require_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fusion,shape,autotune,kernels", [
    (None, None, False, ("block", "deep")), (2, None, False, ("pass2",)),
    (2, None, True, ("pass2", "step")), (1, None, False, ("step",)),
    (None, (256, 16), False, ("pass2",)), (None, None, True, ("block", "deep", "pass2", "step"))])
def test_benchmark_labels_what_ran(monkeypatch, fusion, shape, autotune, kernels):
    require_gpu()
    import bench
    monkeypatch.setattr(bench, "N", 192)
    seen = []
    for name in ("step", "autotune", "set_launch"):
        real = getattr(lbm.Batch, name)

        def wrapped(self, *a, _real=real):
            out = _real(self, *a)
            seen.append(self.get_pass())
            return out
        monkeypatch.setattr(lbm.Batch, name, wrapped)
    res = bench.run_slab("f32", "bgk", fusion, 24, 0, shape=shape, autotune=autotune)
    steps, form = seen[-1][:2]
    assert res["kernel"] in kernels and res["kernel"] == bench.kernel_of(seen[-1])
    assert res["fusion"] == steps == bench.STEPS_PER_LAUNCH[res["kernel"]]
    assert bench.KERNEL_NAMES[res["kernel"]][1] in res["kernel_name"]
    assert res["timed_launches"] == 24 // steps and len(res["launch"]) == 2
    if form != lbm.LBM_PASS_SHORT:
        assert tuple(res["launch"]) == tuple(seen[-1][2:])
