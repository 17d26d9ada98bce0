"""A host model of the wave walker's occupancy table: that the cubic walks of the
small-table GPU tests (this seed, these sizes) do meet sites whose seven places are
all taken, so that those tests take the path around them.  The square lattice's
fifteen places run out in none: its smallest tables do not reach that path."""
import os
import re

import numpy as np
import pytest

import oracle

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2002_03000_amd", "csrc")
LOW = 0xFFFFFFFF


def _source_constants():
    keys = open(os.path.join(CSRC, "pperm_internal.h")).read()
    c = {k: int(v, 16) for k, v in re.findall(r"(SITE3_\w+) = 0x([0-9A-Fa-f]+)u", keys)}
    walker = open(os.path.join(CSRC, "pperm_kernels.hip")).read()
    # the hash of a key in subtable o, and the slot it gives
    m = re.search(r"lane_mul = \(\(0x(\w+)u \* \(uint32_t\)\(poff \+ 1\)\) \^ "
                  r"\(0x(\w+)u \* \(uint32_t\)\(poff \+ 3\)\)\) \| 1u;", walker)
    assert "__umulhi(S_::word(k) * lane_mul, lane_sub)" in walker
    assert "static Key origin() { return 0x80008000u; }" in walker
    c["mul"] = [((int(m[1], 16) * (o + 1) & LOW) ^ (int(m[2], 16) * (o + 3) & LOW)) | 1 for o in range(15)]
    return c


def _key(dim, site, c):
    if dim == 2:
        return (0x80008000 + site[0] + (site[1] << 16)) & LOW
    return (c["SITE3_0"] + site[0] + c["SITE3_Y"] * site[1] + c["SITE3_Z"] * site[2]) & LOW


def _philox(counter, key):
    x0, x1, x2, x3 = counter
    k0, k1 = key
    for _ in range(10):
        p0, p1 = np.uint64(0xD2511F53) * x0, np.uint64(0xCD9E8D57) * x2
        s, low = np.uint64(32), np.uint64(LOW)
        x0, x1, x2, x3 = (p1 >> s) ^ x1 ^ np.uint64(k0), p1 & low, (p0 >> s) ^ x3 ^ np.uint64(k1), p0 & low
        k0, k1 = (k0 + 0x9E3779B9) & LOW, (k1 + 0xBB67AE85) & LOW
    return x0


def _rosenbluth_sequence(dim, n_max, slots, seed, s, tours, c):
    """A sequence's Rosenbluth walks with their table: the trajectory digest, the
    sites that found all their places taken, and the scans that had such a site
    beside the walk's end."""
    steps = [tuple(sign * (a == axis) for a in range(dim)) for axis in range(dim) for sign in (1, -1)]
    subtables = 15 if dim == 2 else 7
    sub = slots // subtables
    digest, taken, beside = 2166136261, 0, 0
    events = np.arange(n_max, dtype=np.uint64)
    zero = np.zeros_like(events)
    for t in range(tours):
        draw = _philox((events, zero, zero + np.uint64(t), zero + np.uint64(s)), (seed, 0)).tolist()
        table, walk, outside = {}, set(), set()

        def put(site):
            word = _key(dim, site, c)
            places = [o * sub + ((word * c["mul"][o] & LOW) * sub >> 32) for o in range(subtables)]
            free = [p for p in places if p not in table]
            slot = free[0] if free else next(i for i in range(slots) if i not in table)
            assert slot < sub * subtables
            table[slot] = site
            walk.add(site)
            if not free:
                outside.add(site)

        end = (0,) * dim
        put(end)
        for b0 in draw:
            beside_end = [tuple(x + y for x, y in zip(end, d)) for d in steps]
            free = [i for i, q in enumerate(beside_end) if q not in walk]
            beside += any(q in outside for q in beside_end)
            if not free:
                break
            i = free[b0 * len(free) >> 32]
            digest = ((digest ^ (i | len(free) << 3)) * 16777619) & LOW
            end = beside_end[i]
            put(end)
        taken += len(outside)
    return digest, taken, beside


@pytest.mark.parametrize("dim,n_max,slots,N,tours", [(3, 63, 96, 60, 7), (3, 126, 192, 60, 7), (2, 41, 64, 60, 7)])
def test_small_cubic_tables_leave_sites_without_a_place(dim, n_max, slots, N, tours):
    c = _source_constants()
    o = oracle.Oracle(dim, n_max, N, 91, mode=oracle.MODE_ROSENBLUTH)
    o.run_tours(tours)
    taken = beside = 0
    for s in range(N):
        digest, t, b = _rosenbluth_sequence(dim, n_max, slots, 91, s, tours, c)
        assert digest == o.stats["digest"][s]              # (the walks are the library's)
        taken += t
        beside += b
    assert (taken > 0 and beside > 0) == (dim == 3), (taken, beside)
