"""half_erfc_near (qlskum_erfc.h), the flux body's erfc(-y)/2 for |y| up to
kErfNear64, against 40-digit mpmath: absolute error at most 2^-52 (half an ulp
of the sum, below 1, and one ulp each of y^2 and of y P(y^2), below 1/2)."""
import os
import subprocess

import mpmath as mp
import numpy as np

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_half_erfc_near(tmp_path):
    exe = str(tmp_path / "near")
    subprocess.run(["/opt/rocm/bin/hipcc", "-O2", "-x", "hip",
                    os.path.join(ROOT, "tests", "erfc_near_check.cpp"), "-o", exe],
                   check=True, capture_output=True)
    ys = np.concatenate([np.linspace(-1.25, 1.25, 5001), [0.0, 1e-300, -1e-300, 1e-9]])
    out = subprocess.run([exe], input="\n".join(repr(float(v)) for v in ys),
                         capture_output=True, text=True, check=True).stdout.split()
    assert float(out[0]) == 1.25
    mp.mp.dps = 40
    err = max(abs(mp.mpf(v) - mp.erfc(-mp.mpf(float(y))) / 2) for v, y in zip(out[1:], ys))
    assert err <= mp.mpf(2) ** -52, err
