"""The tables of csrc/normal_math.hpp made again, in integer arithmetic of 120 fraction
bits (`python tests/normal_tables.py` prints them).

Both are accurate tables in the sense of S. Gal ("Computing elementary functions: a new
approach for achieving high accuracy and good performance", 1986): the points are moved
from their even spacing to where the tabulated values lie close to representable ones."""
import math
import os
import re

P = 120
ONE = 1 << P
HEADER = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2408_12057_amd",
                      "csrc", "normal_math.hpp")


def _atanh_inv(n):
    """atanh(1 / n)."""
    x = ONE // n
    s, k = x, 1
    while x:
        x //= n * n
        k += 2
        s += x // k
    return s


def _atan_inv(n):
    x = ONE // n
    s, k, sign = x, 1, 1
    while x:
        x //= n * n
        k += 2
        sign = -sign
        s += sign * (x // k)
    return s


LN2 = 2 * _atanh_inv(3)
PI = 4 * (4 * _atan_inv(5) - _atan_inv(239))
TURN32 = 2 * PI >> 32  # 2 pi 2^-32


def ln(num, den):
    """log(num / den) for a ratio in (1/2, 2)."""
    y = ((num - den) << P) // (num + den)
    y2, t, s, k = y * y >> P, y, y, 1
    while t not in (0, -1):
        t = t * y2 >> P
        k += 2
        s += t // k
    return 2 * s


def sincos(x):
    """sin and cos of a fixed-point angle."""
    s, t, k = x, x, 1
    while t not in (0, -1):
        t = -(t * x >> P) * x // ((k + 1) * (k + 2)) >> P
        k += 2
        s += t
    c, t, k = ONE, ONE, 0
    while t not in (0, -1):
        t = -(t * x >> P) * x // ((k + 1) * (k + 2)) >> P
        k += 2
        c += t
    return s, c


def to_double(v):
    """The binary64 number nearest to a fixed-point value (integer division rounds right)."""
    return v / ONE


def fixed(f):
    num, den = f.as_integer_ratio()
    return (num << P) // den


def log_entry(i):
    """{c, h} of the mantissas [1 + i / 128, 1 + (i + 1) / 128): c near the reciprocal of
    their middle, with 26 bits (29 in the upper half, which counts to the next octave),
    and h = 2 log c (plus 2 log 2) at a multiple of 2^-44: the first c of the range whose
    h lies within the limit of such a multiple, or the one that comes closest.  The last
    entry is exact."""
    if i == 127:
        return 0.5, -0.0
    up = i >= 64
    bits = 29 if up else 26
    base = (256 << bits) // (257 + 2 * i)
    reach = 12000 if not up else 60000 if i < 112 else 150000
    cell = 1 << (P - 44)
    l0 = ln(base, 1 << bits) + (LN2 if up else 0)
    best = None
    for j in range(-reach, reach + 1):
        e = (j << P) // base
        e2 = e * e >> P
        e3 = e2 * e >> P
        v = l0 + e - e2 // 2 + e3 // 3 - (e2 * e2 >> P) // 4 + (e3 * e2 >> P) // 5
        q = (2 * v + cell // 2) // cell
        err = abs(2 * v - q * cell)
        if best is None or err < best[0]:
            best = (err, j, q)
        limit = (ONE >> 58) if not up else (ONE >> 62) if i < 112 else abs(2 * v) >> 57
        if best[0] < limit:
            break
    return (base + best[1]) / (1 << bits), math.ldexp(best[2], -44)


def circle_offset(i):
    """Displacement of point i (1 .. 16) from i / 128 of a turn in 2^-32 turns: the
    smallest beyond 64 (or any before) that brings the best sine and cosine so far within
    0.006 units in the last place of binary64 numbers."""
    s0, c0 = sincos(2 * PI * i // 128)

    def distance(v):
        f = to_double(v)
        return abs(fixed(f) - v) / (ONE * math.ulp(f))

    best = None
    for o in range(1 << 17):
        # (about point 16 either sign gives the other's mirror image)
        for sign in (1,) if o == 0 else (-1,) if i == 16 else (1, -1):
            e = sign * o * TURN32
            e2 = e * e >> P
            e4 = e2 * e2 >> P
            e6 = e4 * e2 >> P
            ce = ONE - e2 // 2 + e4 // 24 - e6 // 720
            se = e - ((e2 * e >> P) // 6) + ((e4 * e >> P) // 120) - ((e6 * e >> P) // 5040)
            d = max(distance((s0 * ce + c0 * se) >> P), distance((c0 * ce - s0 * se) >> P))
            if best is None or d < best[0]:
                best = (d, sign * o)
        if best[0] < 0.006 and o > 64:
            break
    return best[1]


def circle():
    """[(offset, sin, cos)] of the 128 points: the first sixteenth searched, the rest by
    symmetry, and the points next to the axes replaced by the axes themselves."""
    def point(i, o):
        s, c = sincos(2 * PI * i // 128 + o * TURN32)
        return o, to_double(s), to_double(c)

    pts = {0: (0, 0.0, 1.0)}
    for i in range(1, 17):
        pts[i] = point(i, circle_offset(i))
    for i in range(17, 33):
        o, s, c = pts[32 - i]
        pts[i] = (-o, c, s)
    for i in range(33, 65):
        o, s, c = pts[64 - i]
        pts[i] = (-o, s, -c)
    for i in range(65, 128):
        o, s, c = pts[128 - i]
        pts[i] = (-o, -s, c)
    for axis, s, c in ((0, 0.0, 1.0), (32, 1.0, 0.0), (64, 0.0, -1.0), (96, -1.0, 0.0)):
        for d in (-1, 0, 1):
            pts[(axis + d) % 128] = (-d << 25, s, c)
    return [pts[i] for i in range(128)]


def header_tables():
    """(log entries, circle points) as the header holds them."""
    src = open(HEADER).read()

    def body(name):
        return re.search(name + r"\[\w+\] = \{\n(.*?)\n\};", src, re.S).group(1)

    def pairs(name):
        return [(float.fromhex(a), float.fromhex(b)) for a, b in re.findall(r"\{([^{},]+), ([^{},]+)\}", body(name))]

    offsets = [int(v) for v in re.findall(r"-?\d+", body("kCircleOffset"))]
    return pairs("kLogTable"), [(o, s, c) for o, (s, c) in zip(offsets, pairs("kCircleTable"))]


if __name__ == "__main__":
    for i in range(128):
        print("{%s, %s}," % tuple(v.hex() for v in log_entry(i)))
    for o, s, c in circle():
        print(o, "{%s, %s}," % (s.hex(), c.hex()))
