"""The rate kernel's exponential, compiled for the host from its own source
(fused multiply-adds, ldexp and rounding are the same there), against 40 digits.

Bound.  Of the result's ulp: 0.5 for the last rounding; the argument reduced to
|r| <= 0.347 is off by half an ulp of it, 2.8e-17, an eighth to a quarter of an
ulp of e^r; the polynomial ahead of the last step is off by 2^-53 and enters
with |r|, at most 0.35: 1.1 together.  Below the normal range the last scaling
rounds once more: half of the smallest number.
"""
import ctypes
import decimal
import math
import os
import random
import subprocess

import pytest

from paper_2306_16493_amd import build

SOURCE = """
#include "dev_util.h"
extern "C" void exp_neg_all(long n, const double *x, double *y) {
  for (long i = 0; i < n; i++) y[i] = eph::exp_neg(x[i]);
}
"""


@pytest.fixture(scope="module")
def exp_neg(tmp_path_factory):
    d = tmp_path_factory.mktemp("exp_neg")
    src, out = d / "exp_neg.hip", d / "exp_neg.so"
    src.write_text(SOURCE)
    subprocess.check_call([build.HIPCC, "-std=c++17", "-O2", "-fPIC", "-shared", "--offload-host-only", "-ffp-contract=off",
                           "-I", os.path.join(build.HERE, "csrc"), "-o", str(out), str(src)])
    lib = ctypes.CDLL(str(out))

    def call(x):
        a = (ctypes.c_double * len(x))(*x)
        y = (ctypes.c_double * len(x))()
        lib.exp_neg_all(ctypes.c_long(len(x)), a, y)
        return list(y)

    return call


def test_against_forty_digits(exp_neg):
    decimal.getcontext().prec = 40
    rng = random.Random(3)
    xs = [-rng.uniform(0.0, 745.0) for _ in range(3000)] + [-rng.uniform(0.0, 40.0) for _ in range(6000)]
    xs += [-10.0 ** rng.uniform(-18, 0) for _ in range(1000)]
    xs += [-math.nextafter((n + 0.5) * math.log(2.0), to) for n in range(0, 1070, 5) for to in (0.0, 1e3)]
    worst = 0.0
    for x, y in zip(xs, exp_neg(xs)):
        want = decimal.Decimal(x).exp()
        ulp = decimal.Decimal(math.ulp(float(want)))
        bound = 1.1 if float(want) >= 2.3e-308 else 1.6
        err = float(abs(decimal.Decimal(y) - want) / ulp)
        worst = max(worst, err / bound * 1.1)
        assert err <= bound, (x, y)
    print(f"exp_neg: within {worst:.2f} ulp at {len(xs)} points")


def test_ends(exp_neg):
    assert exp_neg([0.0, -0.0]) == [1.0, 1.0]
    assert exp_neg([-746.0, -800.0, -1e300, -math.inf]) == [0.0] * 4  # what masked terms pass
