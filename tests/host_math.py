"""Pointwise functions of the stage kernel compiled for the host: the named
definitions are cut out of csrc/stage_kernel.hpp and built with g++ next to
stand-ins for the instructions they use (the hardware's approximations at
their documented accuracy, the single-instruction minima and maxima), so that
they can be compared with the mathematics over many arguments without a GPU."""
import ctypes
import os
import re
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "paper_2004_08503_amd", "csrc", "stage_kernel.hpp")

STAND_INS = r"""
#include <cmath>
#define __device__
#define __forceinline__ inline
static inline float __builtin_amdgcn_exp2f(float x) { return exp2f(x); }
static inline float __builtin_amdgcn_logf(float x) { return log2f(x); }
static inline double __builtin_amdgcn_rcp(double x) { return 1.0 / x * (1.0 + 0x1p-25); }
static inline double __builtin_amdgcn_rsq(double x) { return 1.0 / std::sqrt(x) * (1.0 + 0x1p-25); }
static inline bool __builtin_amdgcn_class(double x, int m) {   // v_cmp_class_f64
  const int n = std::signbit(x) ? 0 : 1;
  switch (std::fpclassify(x)) {
    case FP_NAN: return m & 3;
    case FP_INFINITE: return m & (n ? 0x200 : 0x4);
    case FP_ZERO: return m & (n ? 0x40 : 0x20);
    case FP_SUBNORMAL: return m & (n ? 0x80 : 0x10);
  }
  return m & (n ? 0x100 : 0x8);
}
// v_min_f64 and v_max_f64: a NaN operand gives the other one
static inline double vmin(double a, double b) { return std::fmin(a, b); }
static inline double vmax(double a, double b) { return std::fmax(a, b); }
static inline double vmaxabs(double a, double b) { return std::fmax(std::fabs(a), std::fabs(b)); }
static inline double vpos(double a) { return std::fmax(a, 0.0); }
static inline double vneg(double a) { return std::fmin(a, 0.0); }
struct Phys { double gamma, g1, igm1, fac, f1, gsure, ex, inv_ex; };
static Phys phys(double g) {   // as the host sets them
  return {g, 0.5 * (g - 1), 1 / (g - 1), (g + 1) / (2 * g), 1 - (g + 1) / (2 * g), (g - 1) * (1 - 3e-13),
          (g - 1) / (2 * g), 1 / ((g - 1) / (2 * g))};
}
"""


def definition(src, name):
    """The definition of a function (its template line included) or struct
    at file scope."""
    m = re.search(r"^struct %s \{.*?^\};\n" % name, src, re.M | re.S)
    if m:
        return m.group(0)
    for m in re.finditer(r"^(?:template <[^\n]*>\n)?(?![ /])[^\n]*\b%s\(" % name, src, re.M):
        text = src[m.start():src.index("\n}\n", m.start()) + 3]
        if ";" not in text[:text.index("{")]:
            return text
    raise AssertionError("no definition of %s" % name)


def build(directory, names, driver):
    """The named definitions, in order, followed by driver (extern "C"
    functions), as a loaded library."""
    with open(HEADER) as f:
        src = f.read()
    cpp, so = os.path.join(directory, "host_math.cpp"), os.path.join(directory, "host_math.so")
    with open(cpp, "w") as f:
        f.write(STAND_INS + "\n".join(definition(src, n) for n in names) + driver)
    subprocess.run(["g++", "-O2", "-std=c++17", "-mfma", "-ffp-contract=off", "-shared", "-fPIC", "-o", so, cpp],
                   check=True)
    return ctypes.CDLL(so)


def ptr(a):
    return a.ctypes.data_as(ctypes.c_void_p)
