"""The device's own tanh, sigmoid and Adam quotient, taken from their source and compiled for the host with the hardware's
estimates (v_rsq_f32, v_rcp_f32, v_exp_f32: one unit in the last place each) in place, once rounded to nearest and once off by that
unit either way, against float64: the bounds that their comments state, and what they make of zeros, infinities and NaN."""
import ctypes as ct
import os
import re
import subprocess

import numpy as np
import pytest

from paper_1705_09786_amd import build

HOST = r"""
#include <math.h>
#include <cmath>
#include <cstdint>
#include <cstring>
static int g_off;   // how many units in the last place every estimate is off by
static float est(double v) {
  float f = (float)v;
  if (!std::isfinite(f) || f == 0.f || std::fabs(f) < 1.2e-38f) return f;
  int32_t u;
  memcpy(&u, &f, 4);
  u += g_off;
  memcpy(&f, &u, 4);
  return f;
}
#define __device__
#define __forceinline__ static inline
#define __builtin_amdgcn_rsqf(x) est(1.0 / std::sqrt((double)(x)))
#define __builtin_amdgcn_rcpf(x) est(1.0 / (double)(x))
#define __builtin_amdgcn_exp2f(x) est(std::exp2((double)(x)))
static float __builtin_amdgcn_div_fixupf(float q, float d, float n) {
  if (std::isnan(d) || std::isnan(n) || (d == 0.f && n == 0.f) || (std::isinf(d) && std::isinf(n))) return NAN;
  const float sign = (std::signbit(d) != std::signbit(n)) ? -1.f : 1.f;
  if (d == 0.f || std::isinf(n)) return sign * INFINITY;
  if (n == 0.f || std::isinf(d)) return sign * 0.f;
  return std::copysign(std::fabs(q), sign);
}
%s
extern "C" void run(int which, int off, const float* a, const float* b, float lr, float c2, float eps, float* o, int n) {
  g_off = off;
  for (int i = 0; i < n; ++i) o[i] = which == 0 ? tanh_(a[i]) : which == 1 ? sigmoidf_(a[i]) : adam_quotient<false>(a[i], b[i], lr, 1.f, c2, eps);
}
"""


@pytest.fixture(scope="module")
def device_math(tmp_path_factory):
    text = open(os.path.join(build.HERE, "csrc", "amp_common.hip.h")).read()
    parts = []
    for head in (r"template <bool DIV>\n__device__ __forceinline__ float adam_quotient\(", r"__device__ __forceinline__ float tanh_\(",
                 r"__device__ __forceinline__ float sigmoidf_\("):
        parts.append(re.search(head + r".*?\n}\n", text, re.S).group(0))
    tmp = tmp_path_factory.mktemp("math")
    src, so = tmp / "m.cpp", tmp / "m.so"
    src.write_text(HOST % "\n".join(parts))
    p = subprocess.run(["g++", "-O1", "-ffp-contract=off", "-shared", "-fPIC", "-std=c++17", str(src), "-o", str(so)],
                       stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert p.returncode == 0, p.stdout
    lib = ct.CDLL(str(so))

    def run(which, off, a, b=None, eps=0.0, lr=1.0, c2=1.0):
        a = np.ascontiguousarray(a, np.float32)
        b = np.ascontiguousarray(a if b is None else b, np.float32)
        o = np.empty_like(a)
        p = lambda v: v.ctypes.data_as(ct.POINTER(ct.c_float))
        lib.run(which, off, p(a), p(b), ct.c_float(lr), ct.c_float(c2), ct.c_float(eps), p(o), a.size)
        return o
    return run


def ulps(got, ref):
    """|got - ref| in units of the last place of ref's binary32 neighbours."""
    unit = np.spacing(np.maximum(np.abs(ref), 1.2e-38).astype(np.float32)).astype(np.float64)
    return np.abs(got.astype(np.float64) - ref) / unit


def spread(lo, hi, n, seed, sign=True):
    r = np.random.default_rng(seed)
    v = np.exp(r.uniform(np.log(lo), np.log(hi), n))
    return (v * (r.choice([-1.0, 1.0], n) if sign else 1.0)).astype(np.float32)


# An estimate off by a unit adds what it is worth in the result: the correction squares the reciprocal's error away, so tanh's
# and the sigmoid's bounds grow by the exponential's unit alone (tanh: times e^2x / (e^2x + 1)^2 * 2 / tanh, 0.6 at 1; the sigmoid's
# exponential is the library's here).  The bounds are those of the comments, which give one decimal.
@pytest.mark.parametrize("lo,hi,worst", [(1e-6, 1e-2, 0.9), (1e-2, 0.3, 0.9), (0.3, 1.0, 0.95), (1.0, 3.0, 1.15), (3.0, 10.5, 1.15), (9.9, 80.0, 1.0)])
@pytest.mark.parametrize("off", [0, 1, -1])
def test_tanh(device_math, lo, hi, worst, off):
    x = np.concatenate([spread(lo, hi, 200000, 1), np.float32([lo, -lo, hi, -hi, 1.0, -1.0, np.nextafter(np.float32(1), np.float32(0)), 10.0])])
    assert ulps(device_math(0, off, x), np.tanh(x.astype(np.float64))).max() <= worst + (0.6 if off and hi > 1.0 else 0.0)


@pytest.mark.parametrize("off", [0, 1, -1])
def test_sigmoid(device_math, off):
    x = np.concatenate([spread(1e-4, 80.0, 300000, 2), np.float32([0.0, 80.0, -80.0])])
    assert ulps(device_math(1, off, x), 1.0 / (1.0 + np.exp(-x.astype(np.float64)))).max() <= 2.6
    # beyond: e^-x near and above the largest binary32; below the smallest normal number the result may be zero
    x = np.linspace(-104.0, -80.0, 20001).astype(np.float32)
    assert (np.abs(device_math(1, off, x) - 1.0 / (1.0 + np.exp(-x.astype(np.float64)))) <= 1.2e-38 + 3e-7 * np.exp(x.astype(np.float64))).all()


# A root's estimate off by a unit is squared away as the reciprocal's is; sum and quotient round once each.
@pytest.mark.parametrize("off", [0, 1, -1])
@pytest.mark.parametrize("eps", [1e-8, 1e-3, 1e-20, 0.0])
@pytest.mark.parametrize("lo,hi", [(1e-45, 1e-37), (0.9e-37, 1.1e-37), (1e-37, 1e-28), (1.2e-29, 1.3e-29), (1e-28, 1e-12), (1e-12, 1.0), (1.0, 1e6), (1e6, 3.4e38),
                                   (3.2e38, 3.402e38)])
def test_adam_quotient(device_math, lo, hi, eps, off):
    x = spread(lo, hi, 100000, 3, sign=False)
    x = x[(x > 0) & np.isfinite(x)]
    eps = np.float32(eps)
    d = np.sqrt(x.astype(np.float64)) + float(eps)
    n = (spread(1e-3, 1e3, x.size, 4).astype(np.float64) * d * 1e-3).astype(np.float32)   # what a step's numerator is to its denominator
    keep = np.abs(n) > 1e-30   # (a residual below the smallest normal number is not corrected)
    ref = n.astype(np.float64) / d
    assert ulps(device_math(2, off, n, x, eps), ref)[keep].max() <= 2.4
    assert np.allclose(device_math(2, off, n, x, eps), ref, rtol=1e-6, atol=1e-30)
    # the bias correction of an early update on top of the moment
    if hi < 1e30:
        d = np.sqrt(x.astype(np.float64) * 1000.0) + float(eps)
        got, ref = device_math(2, off, n, x, eps, lr=0.5, c2=1000.0), 0.5 * n.astype(np.float64) / d
        normal = keep & (x > 1.2e-38)   # (the product is rounded to binary32's last denormal bit)
        assert ulps(got, ref)[normal].max() <= 2.9


def test_special_values(device_math):
    inf, nan = np.inf, np.nan
    same = lambda got, want: np.testing.assert_array_equal(got, np.float32(want))
    for off in (0, 1, -1):
        same(device_math(0, off, [0.0, inf, -inf, nan, 1e30, -1e30]), [0.0, 1.0, -1.0, nan, 1.0, -1.0])
        same(device_math(1, off, [inf, -inf, nan, 1e30, -1e30]), [1.0, 0.0, nan, 1.0, 0.0])
        # n / (sqrt(x) + eps) as a division has it: with and without eps
        same(device_math(2, off, [0.0, 3.0, -3.0, 0.0, 3.0, nan, 3.0, inf, inf], [0.0, 0.0, 0.0, inf, inf, 1.0, nan, 1.0, inf], 0.0),
             [nan, inf, -inf, 0.0, 0.0, nan, nan, inf, nan])
        same(device_math(2, off, [0.0, 2.0, 3.0], [0.0, 0.0, inf], 0.5), [0.0, 4.0, 0.0])
        same(device_math(2, off, [3.0, 0.0], [1.0, 1.0], inf), [0.0, 0.0])
