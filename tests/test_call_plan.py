"""The routes of bf_add and bf_contains and the memory they take, as the host
rules give them (bfb_call_plan of include/bf_bench.h; no GPU needed)."""
from __future__ import annotations

import ctypes
import math
import random

import pytest

from test_abi import LIB, _ensure_built

KIB, MIB, GIB = 1 << 10, 1 << 20, 1 << 30
SECTORIZED, CLASSIC = 0, 1
ADD, CONTAINS = 0, 1
AUTO, PARTITIONED_STRATEGY = 0, 2
DIRECT, PARTITIONED, LDS, GROUPED = range(4)
ARRAY = 256 * MIB  # BF_NOALLOC_SCRATCH_BYTES
STEP = 8192        # records of a first-pass step


class Call(ctypes.Structure):
    _fields_ = [("route", ctypes.c_uint32), ("reserved", ctypes.c_uint32), ("workspace_bytes", ctypes.c_uint64),
                ("noalloc_pass_keys", ctypes.c_uint64), ("noalloc_pass_bytes", ctypes.c_uint64)]


def call_plan(nbytes, op, n, s=8, bits=32, k=8, layout=SECTORIZED, strategy=AUTO):
    _ensure_built()
    lib = ctypes.CDLL(LIB)
    u32, u64 = ctypes.c_uint32, ctypes.c_uint64
    lib.bfb_call_plan.argtypes = [u32, u64, u32, u32, u32, u32, u32, ctypes.c_int, u64, ctypes.POINTER(Call)]
    out = Call()
    size = nbytes * 8 // 64 * 64 if layout == CLASSIC else nbytes // (s * bits // 8)
    assert lib.bfb_call_plan(layout, size, s, bits, 0, k, strategy, op, n, ctypes.byref(out)) == 0
    return out


def test_arguments_are_checked():
    _ensure_built()
    lib = ctypes.CDLL(LIB)
    out = Call()
    u32, u64 = ctypes.c_uint32, ctypes.c_uint64
    lib.bfb_call_plan.argtypes = [u32, u64, u32, u32, u32, u32, u32, ctypes.c_int, u64, ctypes.c_void_p]
    good = (0, 4096, 8, 32, 0, 8, 0, 0, 1000)
    assert lib.bfb_call_plan(*good, ctypes.addressof(out)) == 0
    assert lib.bfb_call_plan(*good, None) == -1
    for at, value in [(0, 3), (0, 9), (1, 0), (1, 2**32 + 1), (2, 3), (2, 32), (3, 16), (5, 7), (5, 33), (6, 3), (7, 2),
                      (8, 0)]:
        bad = list(good)
        bad[at] = value
        assert lib.bfb_call_plan(*bad, ctypes.addressof(out)) == -1, (at, value)


@pytest.mark.parametrize("nbytes,op,n,route", [
    (4 * KIB, ADD, 8 * 4 * KIB - 1, DIRECT), (4 * KIB, ADD, 8 * 4 * KIB, LDS),
    (160 * KIB, ADD, 8 * 160 * KIB, LDS), (160 * KIB + 32, ADD, 1 << 24, PARTITIONED),
    (GIB, ADD, 1 << 20, DIRECT), (GIB, ADD, 1 << 28, PARTITIONED),
    (64 * KIB, CONTAINS, (1 << 21) - 1, DIRECT), (64 * KIB, CONTAINS, 1 << 21, LDS),
    (16 * KIB, CONTAINS, 1 << 21, DIRECT), (16 * KIB, CONTAINS, 1 << 22, LDS),
    (8 * MIB, CONTAINS, 1 << 24, GROUPED), (16 * MIB, CONTAINS, 1 << 23, GROUPED), (32 * MIB, CONTAINS, 3 << 21, GROUPED),
    (128 * MIB, CONTAINS, 12_400_000, GROUPED), (GIB, CONTAINS, 40_000_000, GROUPED),
    (4 * MIB, CONTAINS, 1 << 26, DIRECT), (2 * GIB + 32, CONTAINS, 1 << 28, DIRECT),
    (32 * MIB, CONTAINS, 1 << 26, GROUPED), (GIB, CONTAINS, 1 << 28, GROUPED), (GIB, CONTAINS, 1 << 24, DIRECT),
])
def test_routes(nbytes, op, n, route):
    c = call_plan(nbytes, op, n)
    assert c.route == route
    assert (c.workspace_bytes > 0) == (route in (PARTITIONED, GROUPED))


def _two_pass_bytes(chunks, n, k):
    """The two-digit workspace from its parts; k records per key (1: one)."""
    def up(v, m):
        return -(-v // m) * m

    steps = -(-n // (STEP if k == 1 else 512 * (STEP // 512 // k)))  # classic: whole keys of 512 threads
    records = n * k
    digits2 = 1 << math.isqrt(chunks - 1).bit_length()
    digits1 = -(-chunks // digits2)
    share = -(-records // digits1)
    per_digit = max(-(-share // 65536), min(-(-512 // digits1), share // STEP), 1)
    items = digits1 * per_digit
    batches = items * -(-(-(-steps // per_digit)) // 1024)
    # a run of c records takes ceil(c / unit) units; every batch ends with a partial step
    unit = 8 if digits1 >= 256 else 16
    steps2 = (records // unit + min(steps * digits1, records)) // (STEP // unit) + batches
    parts = [8 * steps * STEP, 4 * digits1 * up(steps, 16), 4 * steps2 * STEP, 2 * steps2 * STEP,
             4 * digits2 * up(steps2, 16), 4 * items, 4 * (items + 1)]
    return sum(up(p, 256) for p in parts)


@pytest.mark.parametrize("nbytes", [65 * MIB, GIB, 4 * GIB, 16 * GIB, 32 * GIB])
@pytest.mark.parametrize("layout,k", [(SECTORIZED, 8), (CLASSIC, 12)])
def test_partitioned_workspace_is_what_the_add_takes(nbytes, layout, k):
    """A server admits an add at the bytes that the add takes from the pool:
    its buffers, not an estimate; of several passes the largest."""
    if layout == CLASSIC and nbytes > 16 * GIB:
        pytest.skip("classic filters are partitioned up to 2^37 bits")
    per_key = k if layout == CLASSIC else 1
    most = (1 << 28) // per_key
    for n in (most, most // 7, 12_345_678 // per_key):
        c = call_plan(nbytes, ADD, n, k=k, layout=layout, strategy=PARTITIONED_STRATEGY)
        assert c.route == PARTITIONED
        assert c.workspace_bytes == _two_pass_bytes(nbytes // (64 * KIB), n, per_key)
    c = call_plan(nbytes, ADD, 3 * most, k=k, layout=layout, strategy=PARTITIONED_STRATEGY)
    assert c.workspace_bytes == _two_pass_bytes(nbytes // (64 * KIB), most, per_key)


def test_noalloc_limits_and_passes():
    """The adds that bf_add_noalloc takes, and that none of their passes
    exceeds the array."""
    def noalloc(nbytes, n, **kw):
        c = call_plan(nbytes, ADD, n, strategy=PARTITIONED_STRATEGY, **kw)
        if c.noalloc_pass_keys:
            assert 0 < c.noalloc_pass_keys <= n and c.noalloc_pass_bytes <= ARRAY, (nbytes, n, kw)
        return c.noalloc_pass_keys

    assert noalloc(64 * MIB, 40_000_000) == 40_000_000
    assert 0 < noalloc(64 * MIB, 42_500_003) < 42_500_003  # two passes
    assert noalloc(64 * MIB, 46_000_000) == 0
    assert noalloc(GIB, 12_000_000) == 12_000_000
    assert noalloc(GIB, 16_000_000) == 0
    rng = random.Random(1)
    for _ in range(3000):
        nbytes = int(2 ** rng.uniform(20, 35)) // 4096 * 4096
        if rng.random() < 0.3:
            noalloc(nbytes, rng.randrange(1, 6_000_000), layout=CLASSIC, k=rng.choice([4, 6, 8, 12, 16]))
        else:
            s, bits = rng.choice([(1, 64), (2, 32), (8, 32), (4, 64), (16, 64)])
            noalloc(nbytes, rng.randrange(1, 45_000_000), s=s, bits=bits, k=16)


@pytest.mark.parametrize("s,bits,k,nbytes,n,route", [
    # where the grouped form was measured slower than the direct one, and faster
    (16, 64, 16, 1030 * MIB, 39_000_000, DIRECT), (16, 64, 16, GIB, 1 << 27, GROUPED),
    (16, 64, 16, 66 * MIB, 11_000_000, DIRECT), (16, 64, 16, 128 * MIB, 1 << 25, GROUPED),
    (8, 32, 9, 66 * MIB, 11_000_000, DIRECT), (8, 32, 9, 128 * MIB, 1 << 25, GROUPED),
    (8, 32, 9, 2000 * MIB, 68_000_000, DIRECT), (8, 32, 9, 2000 * MIB, 1 << 27, GROUPED),
    (8, 32, 9, 20 * MIB, 9_000_000, DIRECT), (8, 32, 9, 20 * MIB, 1 << 26, GROUPED),
    (4, 64, 16, 260 * MIB, 15_900_000, DIRECT), (4, 64, 16, GIB, 1 << 26, GROUPED),
    # a k that is not compiled in, blocks of 64 bytes and more: two digits have no kernel
    (16, 32, 20, GIB, 1 << 28, DIRECT),
    (8, 32, 9, 160 * KIB, 1 << 21, DIRECT), (8, 32, 9, 160 * KIB, 1 << 22, LDS), (8, 32, 9, 64 * KIB, 1 << 21, LDS),
])
def test_lookup_routes_of_other_layouts(s, bits, k, nbytes, n, route):
    assert call_plan(nbytes, CONTAINS, n, s=s, bits=bits, k=k).route == route
