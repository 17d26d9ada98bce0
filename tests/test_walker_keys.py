"""The 32-bit keys of cubic sites: distinct for every two sites that can meet in
one walk, and never 0, up to the limit the library uses them for."""
import os
import re

import numpy as np

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _constants():
    src = open(os.path.join(ROOT, "paper_2002_03000_amd", "csrc", "pperm_internal.h")).read()
    c = {k: int(v, 16) for k, v in re.findall(r"(SITE3_\w+) = 0x([0-9A-Fa-f]+)u", src)}
    c["max_n"] = int(re.search(r"COMPACT3_MAX_N = (\d+);", src).group(1))
    return c


def _shortest(offset, y_mul, z_mul, radius, nonzero):
    """Smallest |x| + |y| + |z| <= radius with x + y_mul y + z_mul z + offset = 0
    modulo 2^32 (radius + 1 if there is none; nonzero: other than no step)."""
    best = radius + 1
    y = np.arange(-radius, radius + 1, dtype=np.int64)
    for z in range(-radius, radius + 1):
        t = (offset + y_mul * (y & 0xFFFFFFFF) + z_mul * (z & 0xFFFFFFFF)) & 0xFFFFFFFF
        x = (-t) & 0xFFFFFFFF
        x = np.where(x >= 1 << 31, x - (1 << 32), x)
        d = np.abs(x) + np.abs(y) + abs(z)
        if nonzero:
            d = d[d > 0]
        best = min(best, int(d.min()))
    return best


def test_cubic_keys_are_distinct_and_never_zero():
    c = _constants()
    y, z = c["SITE3_Y"], c["SITE3_Z"]
    assert (z * c["SITE3_Z_INV"]) & 0xFFFFFFFF == 1
    # two sites of a walk, or a site and a neighbour of its end: at most n_max + 1 apart
    assert _shortest(0, y, z, 2400, True) == 2293 > c["max_n"] + 1
    # every site, and every neighbour of one, is at most n_max + 1 from the origin
    assert _shortest(c["SITE3_0"], y, z, 2400, False) == 2065 > c["max_n"] + 1
