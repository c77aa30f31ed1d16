"""The FP64 flux body past |S| = kErfNear64 evaluates erfc with half_erfc of
qlskum_erfc.h and no form of its own: the accuracy tests of that header are then
those of the kernel.  Its scaled part erfc(a) exp(a^2) = t R(u) is within 5e-16
relative on [kErfNear64, 10) against 40-digit mpmath: the reciprocal, t = c inv, R's
last fma and the product round by 2^-53 each (4.4e-16), and u = (c - a) inv, whose
error is relative to u, moves R by less than the rest."""
import os
import subprocess

import mpmath as mp
import numpy as np

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_kernel_uses_the_header():
    src = open(os.path.join(ROOT, "paper_2108_07031_amd", "csrc", "qlskum_kernels.hip")).read()
    assert "half_erfc(" in src and "half_erfc_near(" in src
    assert "kErfcPoly64" not in src and "kErfPoly64" not in src and "kErfcN64" not in src


def test_scaled_erfc_past_the_line(tmp_path):
    exe = str(tmp_path / "far")
    subprocess.run(["/opt/rocm/bin/hipcc", "-O2", "-x", "hip",
                    os.path.join(ROOT, "tests", "erfc_far_check.cpp"), "-o", exe],
                   check=True, capture_output=True)
    ys = np.concatenate([[np.nextafter(1.25, 2.0)], np.linspace(1.25, 10.0, 6001)])
    out = subprocess.run([exe], input="\n".join(repr(float(v)) for v in ys),
                         capture_output=True, text=True, check=True).stdout.split()
    assert float(out[0]) == 1.25
    mp.mp.dps = 40
    err = 0
    for v, y in zip(out[1:], ys):
        a = mp.mpf(float(y))
        ref = mp.erfc(a) * mp.exp(a * a)
        err = max(err, abs(mp.mpf(v) - ref) / ref)
    assert err <= 5e-16, float(err)
