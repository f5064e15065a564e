"""csrc/normal_math.hpp on the CPU: its tables equal the ones made again, and its
functions, compiled for the host, are no further from 64-bit-mantissa references than the
device library's log, sqrt and sincospi (largest errors of those over the same kinds of
words: 0.641, 0.884 and, for a normal, 2.497 units in the last place)."""
import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest

import normal_tables as nt

SHIM = r"""
#include <cmath>
#include <cstdint>
#include <cstring>
#define __device__
#define __forceinline__ inline
struct double2 { double x, y; };
using std::fma;
inline int __double2hiint(double v) { uint64_t b; memcpy(&b, &v, 8); return (int)(b >> 32); }
inline int __double2loint(double v) { uint64_t b; memcpy(&b, &v, 8); return (int)b; }
inline double __hiloint2double(int h, int l)
{ uint64_t b = ((uint64_t)(uint32_t)h << 32) | (uint32_t)l; double v; memcpy(&v, &b, 8); return v; }
static struct { unsigned x; } threadIdx = {0}, blockDim = {1};
inline double __builtin_amdgcn_rsq(double x) { return 1.0 / std::sqrt(x); }
"""
HOST = r"""
#include "normal_math.hpp"
extern "C" void words(long n, const uint32_t* wa, const uint32_t* wb, double* o)
{
    using namespace oasmc;
    NormalTables t;
    stage_tables(t);
    for (long i = 0; i < n; ++i, o += 5) {
        o[0] = minus2_log_word(t, wa[i]);
        circle_word(t, wb[i], o[1], o[2]);
        box_muller(t, wa[i], wb[i], o[3], o[4]);
    }
}
"""


def test_tables_made_again():
    log, circle = nt.header_tables()
    assert circle == nt.circle()
    for i in (0, 12, 20, 46, 63, 64, 80, 107, 112, 115, 126, 127):  # worst ones among them
        assert log[i] == nt.log_entry(i), i
    for i, (c, h) in enumerate(log[:127]):
        num, den = c.as_integer_ratio()
        assert den <= 1 << 29 and (c * 2 ** 29).is_integer()
        assert abs(c * (1 + i / 128) - 1) < 2 ** -7.9 and abs(c * (1 + (i + 1) / 128) - 1) < 2 ** -7.9
        err = abs(2 * (nt.ln(num, den) + (nt.LN2 if i >= 64 else 0)) - nt.fixed(h))
        assert err < nt.ONE >> (60 if i >= 64 else 57), i


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no host compiler")
    d = tmp_path_factory.mktemp("normal_math")
    (d / "device_common.hpp").write_text(SHIM)
    shutil.copy(nt.HEADER, d / "normal_math.hpp")
    (d / "host.cpp").write_text(HOST)
    so = str(d / "host.so")
    subprocess.run([gxx, "-O2", "-std=c++17", "-shared", "-fPIC", "-o", so, str(d / "host.cpp")], check=True)
    lib = ctypes.CDLL(so)

    def words(wa, wb):
        out = np.empty((len(wa), 5))
        lib.words(ctypes.c_long(len(wa)), wa.ctypes.data_as(ctypes.c_void_p), wb.ctypes.data_as(ctypes.c_void_p),
                  out.ctypes.data_as(ctypes.c_void_p))
        return out
    return words


def _references(wa, wb):
    """-2 log, sine, cosine and the normals with 64-bit mantissas (angles reduced to an
    eighth of a turn in integers)."""
    ld = np.longdouble
    lg = -2 * np.log((wa.astype(ld) + ld(0.5)) / ld(2 ** 32))
    a = 2 * wb.astype(np.uint64) + 1  # in 2^-33 turns
    octant, r = (a >> np.uint64(30)).astype(int), (a & np.uint64(2 ** 30 - 1)).astype(ld)
    r = np.where(octant % 2 == 1, ld(2 ** 30) - r, r)
    pi = ld("3.14159265358979323846264338327950288")
    s, c = np.sin(2 * pi * (r / ld(2 ** 33))), np.cos(2 * pi * (r / ld(2 ** 33)))
    swap = np.isin(octant, (1, 2, 5, 6))
    s, c = np.where(swap, c, s), np.where(swap, s, c)
    s, c = np.where(octant >= 4, -s, s), np.where(np.isin(octant, (2, 3, 4, 5)), -c, c)
    root = np.sqrt(lg)
    return [lg, s, c, root * c, root * s]


@pytest.mark.skipif(np.finfo(np.longdouble).nmant < 63, reason="no 64-bit mantissas here")
def test_errors_within_the_librarys(host):
    rng = np.random.default_rng(3)
    n = 1 << 20
    wa, wb = (rng.integers(0, 2 ** 32, n, dtype=np.uint32) for _ in range(2))
    near = (rng.integers(0, 8, n) * (1 << 29) + rng.integers(-(5 << 24), 5 << 24, n)).astype(np.int64) % 2 ** 32
    edge = np.concatenate([np.arange(2000), 2 ** 32 - 1 - np.arange(2000),
                           (2 ** np.arange(32)[:, None] + np.arange(-2, 3)).ravel() % 2 ** 32])
    wa = np.concatenate([wa, rng.integers(0, 2 ** 32, n, dtype=np.uint32), edge.astype(np.uint32)])
    wb = np.concatenate([wb, near.astype(np.uint32), np.roll(edge, 7).astype(np.uint32)])
    got = host(wa, wb)
    for j, (ref, bound) in enumerate(zip(_references(wa, wb), (0.641, 0.884, 0.884, 2.497, 2.497))):
        ulp = np.ldexp(1.0, np.frexp(np.abs(ref).astype(np.float64))[1] - 53)
        err = np.abs(got[:, j].astype(np.longdouble) - ref) / ulp
        assert float(err.max()) < bound, (j, float(err.max()), hex(wa[err.argmax()]), hex(wb[err.argmax()]))
