"""The maps of device.h that the strips, the Gram kernels, the cell launches and
the batched sweep run (g_lambda_uniform, g_lambda_small, div_uniform), compiled
for the CPU and compared with the exact quotient and row.  The two approximate
instructions they start from are given every error up to 2 units in the last
place (the hardware's is 1)."""
import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1308_1419_amd", "csrc")

RUNTIME = r"""
#pragma once
#include <math.h>
#include <string.h>
#define __device__
#define __forceinline__ inline
#define __restrict__
struct { unsigned x, y; } threadIdx;
static int error;
static float off(double v) {
  float f = (float)v;
  int b;
  memcpy(&b, &f, 4);
  b += error;
  memcpy(&f, &b, 4);
  return f;
}
#define __builtin_amdgcn_rsqf(v) off(1.0 / sqrt((double)(v)))
#define __builtin_amdgcn_rcpf(v) off(1.0 / (double)(v))
#define __builtin_amdgcn_sqrtf(v) sqrtf(v)
#define __builtin_amdgcn_readfirstlane(v) (v)
static int __syncthreads_count(int v) { return v; }
static void atomicAdd(unsigned long long *, unsigned long long) {}
"""

MAIN = r"""
#include <stdint.h>
#include "device.h"
extern "C" void set_error(int e) { error = e; }
extern "C" void maps(const uint32_t *lam, int64_t n, int which, uint32_t *i, uint32_t *j) {
  for (int64_t k = 0; k < n; ++k) {
    if (which == 0) tdmap::g_lambda(lam[k], i[k], j[k]);
    if (which == 1) tdmap::g_lambda_uniform(lam[k], i[k], j[k]);
    if (which == 2) tdmap::g_lambda_small(lam[k], i[k], j[k]);
  }
}
extern "C" void quotients(const uint32_t *u, const uint32_t *d, int64_t n, uint32_t *q, uint32_t *r) {
  for (int64_t k = 0; k < n; ++k) q[k] = tdmap::div_uniform(u[k], d[k], r[k]);
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("no g++")
    d = tmp_path_factory.mktemp("maps")
    (d / "hip").mkdir()
    (d / "hip" / "hip_runtime.h").write_text(RUNTIME)
    (d / "maps.cpp").write_text(MAIN)
    out = str(d / "maps.so")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-ffp-contract=off", "-fPIC", "-shared", "-I", str(d),
                           "-I", CSRC, str(d / "maps.cpp"), "-o", out, "-lm"])
    return ctypes.CDLL(out)


def _ptr(a):
    return a.ctypes.data_as(ctypes.c_void_p)


@pytest.mark.parametrize("error", [-2, -1, 0, 1, 2])
@pytest.mark.parametrize("which,top", [(0, 1 << 32), (1, 1 << 32), (2, 1 << 28)])
def test_rows_and_columns(lib, which, top, error):
    row = np.arange(92682, dtype=np.uint64)
    start = row * (row + 1) // 2
    rng = np.random.default_rng(5)
    lam = np.concatenate([start, start + 1, start + row // 2, start + row - (row > 0), start + row,
                          rng.integers(0, top, 200000, dtype=np.uint64),
                          np.array([top - 1], dtype=np.uint64)])
    lam = lam[lam < top]
    i = np.searchsorted(start, lam, side="right") - 1
    j = lam - start[i]
    assert np.all(j <= i)
    lam = lam.astype(np.uint32)
    gi, gj = np.empty_like(lam), np.empty_like(lam)
    lib.set_error(error)
    lib.maps(_ptr(lam), ctypes.c_int64(len(lam)), which, _ptr(gi), _ptr(gj))
    assert np.array_equal(gi, i) and np.array_equal(gj, j)


@pytest.mark.parametrize("error", [-2, -1, 0, 1, 2])
def test_quotients(lib, error):
    # u < 2^24 and u / n + 1 < 2^22, at and beside multiples of n
    rng = np.random.default_rng(6)
    n = np.concatenate([np.arange(1, 5000), 2 ** rng.uniform(0, 22, 200000)]).astype(np.int64)
    n = np.concatenate([n, n, n, n])
    most = np.minimum((1 << 24) // n, (1 << 22) - 2)
    q = (rng.random(len(n)) * (most + 1)).astype(np.int64)
    u = q * n + rng.integers(-1, 2, len(n))
    ok = (u >= 0) & (u < 1 << 24) & (u // n + 1 < 1 << 22)
    u, n = u[ok].astype(np.uint32), n[ok].astype(np.uint32)
    gq, gr = np.empty_like(u), np.empty_like(u)
    lib.set_error(error)
    lib.quotients(_ptr(u), _ptr(n), ctypes.c_int64(len(u)), _ptr(gq), _ptr(gr))
    assert np.array_equal(gq, u // n) and np.array_equal(gr, u % n)
