"""Rounding error of the FP64 first-order residual, measured against the oracle's
source compiled in 80-bit arithmetic: its root mean square over a cloud stays
within three times that of the FP64 oracle for each component.  The oracle rounds
every operation and libm call once (half an ulp); the kernel's reciprocals, roots
and exponential are within one to two ulp.  First order, because there a split
flux is nothing but the conversion of a stored q; with the reconstruction its
rounding is hidden behind that of the q-derivatives."""
import ctypes as C
import os
import re
import subprocess

import numpy as np
import pytest

import oracle
from tests._common import cloud, smooth_state

pytestmark = pytest.mark.gpu


class _Params80(C.Structure):
    _fields_ = [(n, C.c_longdouble if t is C.c_double else t) for n, t in oracle._Params._fields_]


def _evaluate80(tmp, c, U, prm):
    """R of the oracle's source with long double for double."""
    src = open(os.path.join(os.path.dirname(oracle.__file__), "qlskum_oracle.c")).read()
    src = re.sub(r"\bdouble\b", "long double", src).replace("<math.h>", "<tgmath.h>")
    (tmp / "o80.c").write_text(src)
    so = str(tmp / "o80.so")
    subprocess.run(["gcc", "-std=c99", "-O2", "-ffp-contract=off", "-fPIC", "-shared", "-o", so,
                    str(tmp / "o80.c"), "-lm"], check=True)
    lib = C.CDLL(so)
    ld = np.longdouble
    geo = [np.ascontiguousarray(a, ld) for a in (c.x, c.y, c.nx, c.ny)]
    top = [np.ascontiguousarray(c.kind, np.uint8), np.ascontiguousarray(c.nbr_ptr, np.int32),
           np.ascontiguousarray(c.nbr_idx, np.int32)]
    flag = np.zeros(top[2].size, np.uint8)
    ptrs = [a.ctypes.data for a in geo + top] + [flag.ctypes.data]
    bad = C.c_int64(-1)
    assert lib.ora_classify(C.c_int64(c.n), *map(C.c_void_p, ptrs), C.byref(bad)) == 0
    cl, p = oracle._Cloud(c.n, *ptrs), _Params80(**prm)
    U = np.ascontiguousarray(U, ld)
    out = [np.empty((k, c.n), ld) for k in (4, 8, 4, 4, 4, 1)]
    assert lib.ora_evaluate(C.byref(cl), C.byref(p), C.c_void_p(U.ctypes.data),
                            *[C.c_void_p(a.ctypes.data) for a in out], C.byref(bad)) == 0
    return out[4]


@pytest.mark.parametrize("mach", [0.85, 1.3])
def test_first_order_rounding(tmp_path, mach):
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    from paper_2108_07031_amd import qlskum as ql
    print(f"first-order rounding mach={mach}", flush=True)
    c = cloud("jitter")
    U = smooth_state(c, mach=mach, alpha_deg=2.0, amp=0.05)
    prm = dict(mach=mach, alpha_deg=2.0, order=1, outer_bc=1)
    ref = _evaluate80(tmp_path, c, U, oracle.params(**prm))
    s = ql.Solver(c, **prm)
    s.set_state(U)
    R = s.evaluate()["R"]
    s.close()
    def rms(a):
        return np.sqrt((np.abs(a - ref) ** 2).mean(axis=1)).astype(float)
    err, base = rms(R), rms(oracle.Oracle(c, oracle.params(**prm)).evaluate(U)["R"])
    print("  rms error", err, "oracle's", base, flush=True)
    assert np.all(err <= 3.0 * base)
