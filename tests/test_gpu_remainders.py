"""What is left of a call after its groups of four steps, in the launch forms
the library picks for it: bitwise the single steps' results, and no slower than
the forms of one and two steps per launch.

Times: the best of seven samples of 40 calls between two events.  A call of one
to three steps may take 1.25 times as long as in those forms (the choice rests
on predictions that are off by up to 10%, twice, and the two sides are timed
apart); computing a four-step halo for every step took 1.3 to 2 times as long."""

import pytest
import torch

from paper_2003_07968_amd import lbm
from paper_2003_07968_amd import workloads as W

from .gpu_common import gpu_lattice, log, require_gpu

pytestmark = pytest.mark.gpu

# lattices in the block pass, small to as large as it takes; alone and batched
CASES = [("f32", [(512, 512)]), ("f32", [(600, 520)]), ("f16", [(300, 300)]),
         ("f64", [(200, 200)]), ("f64", [(480, 252)]), ("f16l", [(24, 6000)]),
         ("f32", [(223, 33)] * 34), ("f16", [(160 - 4 * k,) * 2 for k in range(10)]),
         ("f64", [(503, 65)] * 3), ("f16l", [(144, 43)] * 14), ("f64", [(64, 64)] * 4)]


def _lattices(storage, sizes, **kw):
    out = []
    for k, (nx, ny) in enumerate(sizes):
        p = W.params(nx, ny, tr=0.8, storage=storage)
        rg, rl = W.unit_cs_coexistence(0.8)
        rho0 = W.smooth_random(nx, ny, 50 + k, mean=0.5 * (rg + rl), amplitude=0.4 * (rl - rg))
        p["rho_ref"] = W.shift_reference(rho0, storage)
        out.append(gpu_lattice(p, rho0, **kw))
    return out


def _target(lats):
    if len(lats) == 1:
        return lats[0]
    batch = lbm.Batch(len(lats))
    for lat in lats:
        batch.add(lat)
    return batch


def _us(call, stream):
    samples = []
    for _ in range(7):
        e0 = torch.cuda.Event(enable_timing=True)
        e1 = torch.cuda.Event(enable_timing=True)
        call()
        e0.record(stream)
        for _ in range(40):
            call()
        e1.record(stream)
        e1.synchronize()
        samples.append(e0.elapsed_time(e1) * 1e3 / 40)
    return min(samples)


@pytest.mark.parametrize("storage,sizes", CASES,
                         ids=[f"{s}-{len(z)}x{z[0][0]}x{z[0][1]}" for s, z in CASES])
def test_remainders_bitwise_and_no_slower(storage, sizes):
    require_gpu()
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        ref = _lattices(storage, sizes, launch=(256, 8))
        lats = _lattices(storage, sizes)
        target = _target(lats)
        for n in (1, 2, 3, 5, 6, 7):
            target.step(n)
            for a, b in zip(ref, lats):
                a.step(n)
                assert torch.equal(a.populations(), b.populations()), n
        short = _lattices(storage, sizes)
        other = _target(short)
        for n in (1, 2, 3):
            if len(sizes) == 1:
                other.set_fusion(2, 256, 0)   # the two-step shape, and no longer pass
            else:
                other.set_launch(2, 256, 0)
            t_other = _us(lambda: other.step(n), stream)
            t = _us(lambda: target.step(n), stream)
            log(f"  {storage} {len(sizes)} x {sizes[0]}: {n} step(s) {t:.1f} us, {t_other:.1f}")
            assert t <= 1.25 * t_other, n
        for lat in lats + short:
            lat.sync()
