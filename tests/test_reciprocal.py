"""rcp_any (host build) at the ends of the doubles: infinity for zero and for
what has no finite reciprocal, zero for infinity, otherwise the reciprocal
within an ulp; a result below the normal range within its last bit too."""
import ctypes

import numpy as np

import host_math

DRIVER = r"""
extern "C" void rcp_(const double* x, long n, double* o) { for (long i = 0; i < n; ++i) o[i] = rcp_any(x[i]); }
"""


def test_every_magnitude(tmp_path):
    lib = host_math.build(str(tmp_path), ["rcp_nr", "rcp_any"], DRIVER)
    rng = np.random.default_rng(2)
    x = np.concatenate([[0.0, 5e-324, 1e-320, 2.0 ** -1024, np.nextafter(2.0 ** -1024, 1), 2.0 ** -1022, 1.0, 3.0,
                         2.0 ** 1022, np.finfo(float).max, np.inf],
                        np.ldexp(rng.uniform(1, 2, 4000), rng.integers(-1060, 1023, 4000))])
    x = np.concatenate([x, -x])
    o = np.empty_like(x)
    lib.rcp_(host_math.ptr(x), ctypes.c_long(len(x)), host_math.ptr(o))
    with np.errstate(divide="ignore", over="ignore"):
        want = 1.0 / x
    fin = np.isfinite(want)
    assert np.array_equal(o[~fin], want[~fin])
    assert (np.abs(o - want)[fin] <= np.maximum(np.spacing(np.abs(want[fin])), 5e-324)).all()
