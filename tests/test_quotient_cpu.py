"""The quotients by float products that place work on the device (csrc/pa_quotient.h), on the host: for reciprocals within an ulp
either way, at and around multiples of the divisor and over the stated ranges."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

from paper_2503_13773_amd.build import CSRC

SHIM = r'''
#include <math.h>
#include "pa_quotient.h"
extern "C" int bad(const int *x, const int *d, int n, int ulps, int wide) {
    int count = 0;
    for (int i = 0; i < n; ++i) {
        float recip = float(1.0 / d[i]);
        if (ulps) recip = nextafterf(recip, ulps > 0 ? 2.f : 0.f);
        const int got = wide ? kvc::quotient_wide(x[i], d[i], recip) : kvc::quotient(x[i], d[i], recip);
        count += got != x[i] / d[i];
    }
    return count;
}
'''


@pytest.fixture(scope="module")
def bad(tmp_path_factory):
    folder = str(tmp_path_factory.mktemp("quotient"))
    src, out = os.path.join(folder, "q.cpp"), os.path.join(folder, "q.so")
    with open(src, "w") as f:
        f.write(SHIM)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-ffp-contract=off", "-fPIC", "-shared", "-I", CSRC, src, "-o", out])
    fn = ctypes.CDLL(out).bad

    def count(x, d, ulps, wide):
        x, d = np.ascontiguousarray(x, np.int32), np.ascontiguousarray(d, np.int32)
        p = ctypes.POINTER(ctypes.c_int)
        return fn(x.ctypes.data_as(p), d.ctypes.data_as(p), len(x), ulps, wide)
    return count


def pairs(quotients, divisors, limit):
    """(x, d) around q * d for each quotient and divisor, below the limit."""
    q, d = (a.ravel().astype(np.int64) for a in np.meshgrid(quotients, divisors))
    x = np.concatenate([q * d + off for off in (-1, 0, 1)] + [q * d + d - 1])
    d = np.concatenate([d] * 4)
    keep = (x >= 0) & (x < limit)
    return x[keep], d[keep]


@pytest.mark.parametrize("ulps", [-1, 0, 1])
def test_quotients_up_to_2_to_the_20(bad, ulps):
    rng = np.random.default_rng(5)
    divisors = np.unique(np.concatenate([np.arange(1, 300), 2 ** np.arange(0, 30), 2 ** np.arange(1, 30) - 1, 2 ** np.arange(1, 30) + 1, rng.integers(1, 1 << 30, 500)]))
    quotients = np.unique(np.concatenate([np.arange(0, 70), 2 ** np.arange(0, 20), 2 ** np.arange(1, 20) - 1, rng.integers(0, 1 << 20, 800)]))
    x, d = pairs(quotients, divisors, 1 << 30)
    keep = x // d < 1 << 20
    x, d = x[keep], d[keep]
    assert len(x) > 500000 and (x // d).max() > 1000000
    assert bad(x, d, ulps, 0) == 0


@pytest.mark.parametrize("ulps", [-1, 0, 1])
def test_any_quotient(bad, ulps):
    rng = np.random.default_rng(6)
    divisors = np.unique(np.concatenate([np.arange(1, 200), 2 ** np.arange(0, 30), 2 ** np.arange(1, 30) + 1, rng.integers(1, 1 << 30, 300)]))
    quotients = np.unique(np.concatenate([np.arange(0, 70), 2 ** np.arange(0, 30), 2 ** np.arange(1, 31) - 1, rng.integers(0, 1 << 30, 3000), rng.integers(0, 1 << 25, 5000)]))
    x, d = pairs(quotients, divisors, 1 << 30)
    assert len(x) > 300000 and (x // d).max() > 1 << 29
    assert bad(x, d, ulps, 1) == 0
