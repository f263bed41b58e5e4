"""The partitioned insert's host arithmetic (csrc/cf_bulk_plan.hpp), compiled
here as plain C++ and evaluated over every geometry, the bucket counts around
the powers of two and the batch sizes around the rule's lines: an entry holds
its tag, index and bucket, every region of the workspace lies inside it and
holds what the kernels put there, and launches stay inside their limits."""
import ctypes
import os
import shutil
import subprocess

import pytest

from paper_2603_15486_amd import build as B

HERE = os.path.dirname(os.path.abspath(__file__))
PASS = 1 << 27          # keys of one pass
SEGS, TILE, BINS = 8, 4096, 1024
LDS = 160 << 10         # bytes of a compute unit
FIELDS = ("shift", "parts", "bins", "fine", "cap1", "cap2", "list_cap", "cursors", "o_cur",
          "o_listn", "o_a", "o_a32", "o_b", "o_b32", "o_list", "o_list32", "o_ovl", "bytes")


class Plan:
    def __init__(self, lib, m, b, f, n):
        out = (ctypes.c_uint64 * len(FIELDS))()
        lib.plan(m, b, f, n, out)
        self.__dict__.update(zip(FIELDS, out))


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    cxx = shutil.which("g++") or shutil.which("c++") or B.hipcc()
    out = str(tmp_path_factory.mktemp("plan") / "libplan.so")
    subprocess.check_call([cxx, "-std=c++17", "-O1", "-shared", "-fPIC", "-I", B.CSRC,
                           os.path.join(HERE, "native", "bulk_plan.cpp"), "-o", out])
    so = ctypes.CDLL(out)
    u32, u64 = ctypes.c_uint32, ctypes.c_uint64
    so.wanted.argtypes = so.most.argtypes = so.least.argtypes = so.fits.argtypes = \
        [u64, u32, u32, ctypes.c_int, u64]
    so.most.restype = so.least.restype = u64
    so.plan.argtypes = [u64, u32, u32, u64, ctypes.POINTER(u64)]
    so.plan.restype = None
    so.entry_survives.argtypes = [u32, u32, u32, u32]
    so.lds_bytes.argtypes = [u32, u32]
    so.lds_bytes.restype = u64
    return so


def bucket_counts():
    out = set()
    for k in range(0, 33):
        for base in (1 << k, 3 << k >> 1):
            out.update(base + d for d in (-3, -2, -1, 0, 1, 2, 3, 7))
    return sorted(m for m in out if 1 <= m <= 1 << 32)


def line(b, f, walk, n, table):
    """Bytes of table per key up to which a batch of n keys goes partitioned."""
    if n >= 1 << 22:
        if table >= 2 << 30:
            return 32 if f == 16 else 16
        return 12 if f == 8 else {16: (24, 12), 32: (16, 8)}[f][walk]
    if n >= 1 << 21:
        return 8 if f == 8 else {16: (16, 12), 32: (16, 8)}[f][walk]
    if f == 32:
        return 0 if b == 32 or n < 1 << 20 else 6 if n < 3 << 19 else 8
    if n >= 1 << 20:
        return 12 if f == 16 and not walk and n >= 3 << 19 else 8
    return 6 if f == 16 and n >= 3 << 18 else 4


def batch_sizes(m, b, f):
    out, slots, table = set(), m * b, m * b * f // 8
    for base in (1 << 19, 3 << 18, 1 << 20, 3 << 19, 1 << 21, 1 << 22, PASS, 2 * PASS, slots, 2 * slots,
                 *(table // k for k in (4, 6, 8, 12, 16, 24, 32))):
        out.update(base + d for d in (-1, 0, 1, 2))
    return sorted(n for n in out if n >= 1)


def passes(n):
    k = (n + PASS - 1) // PASS
    return sorted({n * (i + 1) // k - n * i // k for i in range(k)})


@pytest.mark.parametrize("walk", [0, 1])
@pytest.mark.parametrize("f", [8, 16, 32])
@pytest.mark.parametrize("b", [4, 8, 16, 32])
def test_every_plan_that_is_run_addresses_what_is_there(lib, b, f, walk):
    bucket = b * f // 8
    seen = 0
    for m in bucket_counts():
        slots = m * b
        for n in batch_sizes(m, b, f):
            if not lib.wanted(m, b, f, walk, n):
                continue
            share = 4 if n < 1 << 20 else 8 if n < 1 << 22 else 12 if m * bucket < 2 << 30 else 16
            assert n >= 1 << 19 and n <= 2 * slots + 1 and min(n, PASS) * share >= slots
            for size in passes(n):
                seen += 1
                at = (m, b, f, size)
                assert size <= PASS, at
                p = Plan(lib, m, b, f, size)
                # parts: whole buckets, 16-byte moves, a part in LDS
                assert p.parts == (m + (1 << p.shift) - 1) >> p.shift, at
                assert bucket << p.shift <= 64 << 10 and (bucket << p.shift) % 16 == 0, at
                # bins: every part has one, counters fit LDS, numbers fit 16 bits
                assert p.bins << p.fine >= p.parts > (p.bins - 1) << p.fine, at
                assert p.bins <= BINS and 1 << p.fine <= BINS, at
                assert lib.lds_bytes(f, max(p.bins, 1 << p.fine)) + 256 <= LDS, at
                assert p.bins * SEGS * -(-p.cap1 // TILE) < 1 << 31, at
                # the entry with every field at its largest
                top = min(1 << (p.shift + p.fine), m) - 1
                assert lib.entry_survives(f, (1 << f) - 1, size - 1, top), at
                assert lib.entry_survives(f, 1, size - 1, top), at
                # regions, in order and without overlap
                n1, n2, wide = p.bins * SEGS * p.cap1, p.parts * p.cap2, 4 if f == 32 else 0
                lists = p.parts * p.list_cap
                assert p.cursors == 2 * (p.bins * SEGS + (p.parts if p.fine else 0)) + 1
                need = [(p.o_cur, 4 * p.cursors), (p.o_listn, 4 * (p.parts + 1)), (p.o_a, 8 * n1),
                        (p.o_a32, wide * n1), (p.o_b, 8 * n2), (p.o_b32, wide * n2),
                        (p.o_list, 8 * lists), (p.o_list32, wide * lists), (p.o_ovl, 4 * size)]
                for (o, s), (nxt, _) in zip(need, need[1:] + [(p.bytes, 0)]):
                    assert o % 256 == 0 and o + s <= nxt, at
                # the bytes per key that cf.h states
                assert (31 if f == 32 else 21) * size <= p.bytes <= (46 if f == 32 else 35) * size, at
                # the overflow list's eviction queue lies over the first level's
                # entries, and a part's list holds every entry the part can get
                assert 8 * n1 >= 4 * size, at
                assert p.list_cap == (p.cap2 if p.fine else SEGS * p.cap1), at
                # room for the mean of a uniform hash
                tiles = -(-size // TILE)
                per_run = min(size, -(-tiles // SEGS) * TILE)
                assert p.cap1 >= min(1.0, (1 << (p.shift + p.fine)) / m) * per_run, at
                if p.fine:
                    assert p.cap2 >= size * (1 << p.shift) / m, at
    assert seen > 100


def test_a_bucket_too_many_for_an_entry(lib):
    """2^29 buckets of 4 x 16 bits need all of an entry's 21 bucket bits; a
    few buckets more need 22, and the batch goes direct."""
    assert lib.fits(1 << 29, 4, 16, 0, PASS)
    assert Plan(lib, 1 << 29, 4, 16, PASS).shift + Plan(lib, 1 << 29, 4, 16, PASS).fine == 21
    assert lib.wanted(1 << 29, 4, 16, 0, PASS)
    for m in ((1 << 29) + 1, (1 << 29) + 2, (1 << 29) + 3):
        p = Plan(lib, m, 4, 16, PASS)
        assert p.shift + p.fine == 22
        assert not lib.entry_survives(16, 1, 0, 1 << 21)
        assert not lib.fits(m, 4, 16, 0, PASS)
        assert not lib.wanted(m, 4, 16, 0, PASS) and not lib.wanted(m, 4, 16, 0, 2 * PASS)


@pytest.mark.parametrize("walk", [0, 1])
@pytest.mark.parametrize("f", [8, 16, 32])
@pytest.mark.parametrize("b", [4, 8, 16, 32])
def test_a_workspace_serves_every_smaller_batch(lib, b, f, walk):
    """The size grows with the batch, and the cursors, which a new workspace
    has cleared once, are as many for every batch."""
    for m in bucket_counts():
        held, cursors = 0, None
        for n in batch_sizes(m, b, f):
            if not lib.wanted(m, b, f, walk, n):
                continue
            p = Plan(lib, m, b, f, min(n, PASS))
            assert p.bytes >= held and cursors in (None, p.cursors), (m, b, f, n)
            held, cursors = p.bytes, p.cursors


@pytest.mark.parametrize("walk", [0, 1])
@pytest.mark.parametrize("f", [8, 16, 32])
@pytest.mark.parametrize("b", [4, 8, 16, 32])
def test_the_largest_partitioned_batch_below_any_other(lib, b, f, walk):
    """What is reserved for batches of up to n keys serves all of them, also
    where n itself is too large for the table to go partitioned."""
    for m in bucket_counts():
        held = 0
        for n in batch_sizes(m, b, f) + [8 * m * b]:
            if lib.wanted(m, b, f, walk, n):
                held = max(held, n)
            most = lib.most(m, b, f, walk, n)
            assert held <= most <= n and (most == 0) == (held == 0), (m, b, f, n)
            if most:
                assert lib.wanted(m, b, f, walk, most), (m, b, f, n)
                # smaller batches than the least that does go direct, all of them
                least = lib.least(m, b, f, walk, most)
                assert lib.wanted(m, b, f, walk, least), (m, b, f, n)
                assert not lib.wanted(m, b, f, walk, least - 1), (m, b, f, n)
                assert all(lib.wanted(m, b, f, walk, k) == (k >= least)
                           for k in batch_sizes(m, b, f) if k <= most), (m, b, f, n)
