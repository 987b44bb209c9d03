"""The FP64 forms of the force, the velocity and the collisions that take fewer
operations are as accurate as the forms of the other storage modes evaluated
in FP64: rms error of the populations against the equations in 80 bits, on
the CPU, after 60 steps of noisy droplets.

Tolerance.  Two evaluations that round equally well differ at random in what
they round to.  The ratio of their rms errors over the 147,456 populations of
four 64 x 64 droplets would scatter by 1/sqrt(2 x 147456) = 0.2% were the
errors independent; streaming and collision tie neighbouring ones together,
ten times that is allowed.  A rounding that always goes the same way (a
constant stored a little too small, say) grows with every step and shows as
several percent.  The kernels' reciprocals and roots are not part of this:
here both sides divide and take roots exactly rounded."""
import os
import re
import shutil
import subprocess

import numpy as np
import pytest

from paper_2003_07968_amd import workloads as W

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
KERNELS = os.path.join(ROOT, "paper_2003_07968_amd", "csrc", "lbm_kernels.hpp")
SRC = os.path.join(ROOT, "tests", "fp64_forms_check.cpp")


def _cut(text, start, end):
    i = text.index(start)
    return text[i:text.index(end, i) + len(end)]


@pytest.fixture(scope="module")
def check(tmp_path_factory):
    if shutil.which("g++") is None or np.finfo(np.longdouble).nmant < 63:
        pytest.skip("needs g++ and 80-bit long double")
    tmp = tmp_path_factory.mktemp("forms")
    with open(KERNELS) as fh:
        text = fh.read()
    head = r"template <class R>\n__device__ __forceinline__ void "
    parts = [_cut(text, "struct Coeffs {", "\n};\n"),
             _cut(text, "template <class R>\nstruct Phys {", "\n};\n")]
    for name in ("force", "velocity", "collide", "collide_mrt"):
        start = re.search(head + name + r"\(", text).group(0)
        parts.append(_cut(text, start, "\n}\n"))
    (tmp / "forms.hpp").write_text("\n".join(parts))
    exe = str(tmp / "fp64_forms_check")
    subprocess.run(["g++", "-std=c++17", "-O2", "-ffp-contract=off", "-mfma", "-I", str(tmp), SRC,
                    "-o", exe], check=True)
    return exe


@pytest.mark.parametrize("tau,sigma,mrt", [
    (0.6, 1.0, None), (0.7, 1.0, None), (0.8, 0.5, None), (1.2, 1.0, None),
    (0.65, 1.0, (1.0, 1.0, 1.0)), (0.8, 1.0, (1.0, 1.0, 1.0)), (0.8, 1.7, (0.9, 1.1, 1.2))])
def test_as_accurate_as_the_other_forms(check, tau, sigma, mrt):
    p = W.params(64, 64, tr=0.8)
    assert (p["eos_a"], p["eos_b"], p["eos_c"], p["eos_k"], p["G"]) == (1.0, 1.0, 1.0, 1.0, -1.0)
    assert p["epsilon"] == 1.73
    gas, liquid = sorted(W.unit_cs_coexistence(0.8))
    args = [64, 64, tau, sigma, repr(p["T"]), int(mrt is not None), *(mrt or (1.0, 1.0, 1.0)),
            repr(gas), repr(liquid), 60, 4]
    out = subprocess.run([check, *map(str, args)], check=True, capture_output=True, text=True,
                         timeout=300).stdout
    fewer, plain, far_fewer, far_plain = map(float, out.split())
    print(f"  tau {tau} sigma {sigma} mrt {mrt}: error {fewer:.3e} against {plain:.3e}, "
          f"from 64 bits {far_fewer:.3e} against {far_plain:.3e}")
    assert 1e-17 < plain < 1e-13
    assert fewer / plain <= 1.02
    assert far_fewer / far_plain <= 1.1
