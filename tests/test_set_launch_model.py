"""Host model of the filter set's newer launches (csrc/cf_set.hip,
cf_set_persist.hpp, cf_set_requests.hpp), beside tests/test_set_index_model.py,
which models the partition and the class kernels:

  * chunk_for: the chunk a batch is cut into, and what it needs of the scratch;
  * sorted entries: filter id and place in the chunk in one word;
  * phase_front_kernel and the phase kernels of groups of classes: every
    operation of a batch gets its result from exactly one of them, for eager
    batches and for a graph's grid over a smaller batch, and every scratch and
    LDS index is inside its array;
  * requests_lane and the request kernels: the table's order and positions,
    each block's stretch, the key and flag each position reaches, and the
    eviction queue's slices.
"""
import numpy as np
import pytest

from test_set_index_model import K_BLOCK, K_MAX_BINS, K_MAX_CHUNK, K_MAX_CLASSES, layout

K_SMALL_CHUNK, K_FRONT_BLOCK, K_REQ_OPS = 256, 512, 1024
CUS = 256
LDS = 64 << 10


def chunk_for(chunk, n, cus=CUS):
    c = chunk
    while c > K_SMALL_CHUNK and (n + c - 1) // c < cus:
        c //= 2
    return chunk if c % 64 else c


def test_every_chunk_fits_the_scratch():
    for chunk in range(64, K_MAX_CHUNK + 1, 64):
        for n in (1, 63, 64, 65, 4095, 4096, 20000, 1 << 15, (1 << 18) + 1, (1 << 20) - 1, 1 << 22):
            c = chunk_for(chunk, n)
            assert 64 <= c <= chunk and c % 64 == 0
            grid = (n + c - 1) // c
            L = layout(n)  # the smallest set that takes the batch
            assert grid * c >= n and grid * c <= L["sorted"] and grid * c <= L["queue"]
            assert grid * (K_MAX_BINS + 1) <= L["binoff"]
            assert c <= (K_MAX_CHUNK // K_FRONT_BLOCK) * K_FRONT_BLOCK
            assert c * 13 + (2 * K_MAX_BINS + 3) * 4 + 2 * K_MAX_CLASSES <= LDS


def test_an_entry_holds_every_filter_and_place():
    fid = np.array([0, 1, 255, 4095, 4096, 65535], dtype=np.uint64)[:, None]
    place = np.array([0, 1, 63, 2047, 4095], dtype=np.uint64)[None, :]
    e = (fid * K_MAX_CHUNK + place).astype(np.uint32)
    assert np.array_equal(e // K_MAX_CHUNK, np.broadcast_to(fid, e.shape))
    assert np.array_equal(e & (K_MAX_CHUNK - 1), np.broadcast_to(place, e.shape))


def run_phases(ops, fids, cls, groups, chunk, n, max_batch, grid):
    """How often each operation's result is written, by the front kernel and
    the phase kernels of every group; checks every index."""
    ncls = int(cls[cls != 0xFF].max()) + 1
    nb = 3 * ncls
    L = layout(max_batch)
    writes = np.zeros(max_batch, dtype=np.int64)
    binoff = np.zeros((grid, nb + 1), dtype=np.int64)
    entries = np.zeros(grid * chunk, dtype=np.uint32)
    assert grid * (nb + 1) <= L["binoff"]
    first = np.zeros(K_MAX_CLASSES, dtype=bool)
    first[groups[0]] = True
    for blk in range(grid):
        lo = blk * chunk
        have = 0 if lo >= n else min(chunk, n - lo)
        i = np.arange(lo, lo + have)
        op, fid = ops[i].astype(np.int64), fids[i].astype(np.int64)
        c = np.where(fid < cls.size, cls[np.minimum(fid, cls.size - 1)], 0xFF)
        x = np.where((op <= 2) & (c < ncls), op * ncls + c, nb)
        hist = np.bincount(x, minlength=nb + 1)
        base = np.concatenate([[0], np.cumsum(hist)])
        binoff[blk] = base[:-1]
        order = np.argsort(x, kind="stable")
        e = ((fid[order] * K_MAX_CHUNK + order) & 0xFFFFFFFF).astype(np.uint32)
        assert lo + have <= L["sorted"]
        entries[lo:lo + have] = e
        nq = base[ncls]
        # the queries: positions [0, nq) by class, flags at their places
        place = (e[:nq] & (K_MAX_CHUNK - 1)).astype(np.int64)
        assert np.array_equal(place, order[:nq]) and np.all(place < chunk)
        at = np.searchsorted(base[1:ncls + 1], np.arange(nq), side="right")
        assert np.array_equal(at, x[order[:nq]])
        assert np.array_equal(e[:nq] // K_MAX_CHUNK, fid[order[:nq]])
        answered = place[first[at]]
        np.add.at(writes, lo + answered, 1)
        np.add.at(writes, lo + np.flatnonzero(x == nb), 1)
    for phase in range(3):
        for g, classes in enumerate(groups):
            if phase == 0 and g == 0:
                continue
            for blk in range(grid * len(classes)):
                cid, c = blk // len(classes), classes[blk % len(classes)]
                b = phase * ncls + c
                b0, b1 = binoff[cid, b], binoff[cid, b + 1]
                assert 0 <= b0 <= b1 <= chunk
                if b0 == b1:
                    continue
                v = entries[cid * chunk + b0:cid * chunk + b1]
                i = cid * chunk + (v & (K_MAX_CHUNK - 1)).astype(np.int64)
                assert np.all(i < n) and np.all(ops[i] == phase)
                assert np.array_equal(v // K_MAX_CHUNK, fids[i])
                assert np.all(cls[fids[i]] == c)
                if phase == 2:  # the queue's slice of the bin
                    assert cid * chunk + b1 <= L["queue"]
                np.add.at(writes, i, 1)
    return writes


# classes of the set, and its groups (a set whose filters all agree has one)
@pytest.mark.parametrize("ncls,groups", [
    (1, [[0]]), (2, [[0, 1]]), (4, [[0, 2], [1, 3]]), (12, [[k, k + 4, k + 8] for k in range(4)]),
    (16, [[k] for k in range(16)]), (16, [list(range(16))])])
@pytest.mark.parametrize("n,max_batch", [(1, 64), (20_000, 20_000), (9_999, 1 << 16), (0, 4096)])
@pytest.mark.parametrize("chunk", [64, 320, 2048, 4096])
def test_each_operation_has_one_writer(ncls, groups, n, max_batch, chunk):
    rng = np.random.default_rng(n + 7 * ncls + chunk)
    nf = 40
    cls = np.concatenate([np.arange(ncls), rng.integers(0, ncls, nf - ncls)])
    cls[nf - 1] = cls[nf - 2] = 0xFF if ncls < nf - 2 else cls[nf - 1]  # detached
    ops = rng.integers(0, 3, max_batch).astype(np.uint8)
    fids = rng.integers(0, nf, max_batch).astype(np.uint32)
    ops[::37], fids[5::41] = 9, rng.integers(nf, 1 << 32)
    for sized_for in {max(n, 1), max_batch}:  # eager, and a graph's launch
        c = chunk_for(chunk, sized_for)
        grid = (sized_for + c - 1) // c
        w = run_phases(ops, fids, cls, groups, c, n, max_batch, grid)
        assert np.all(w[:n] == 1) and np.all(w[n:] == 0)


def find_entry(off, lo, hi, p):
    while hi - lo > 1:
        mid = (lo + hi) >> 1
        if off[mid] <= p:
            lo = mid
        else:
            hi = mid
    return lo


@pytest.mark.parametrize("ncls,groups", [
    (1, [[0]]), (3, [[0, 2], [1]]), (16, [[k, k + 8] for k in range(8)])])
@pytest.mark.parametrize("count,largest", [(1, 1), (7, 5000), (400, 40), (60, 3000)])
def test_request_batches(ncls, groups, count, largest):
    rng = np.random.default_rng(count + ncls)
    op = rng.integers(0, 3, count)
    cl = rng.integers(0, ncls, count)
    n = np.exp(rng.uniform(0, np.log(largest + 1), count)).astype(np.int64)
    total = int(n.sum())
    ne, nj = np.zeros(3 * ncls, int), np.zeros(3 * ncls, int)
    np.add.at(ne, op * ncls + cl, 1)
    np.add.at(nj, op * ncls + cl, n)
    # the table: phase by phase, a group's classes together, arrival order
    e0, j0, e, j = {}, {}, 0, 0
    for ph in range(3):
        for g in groups:
            for c in g:
                b = ph * ncls + c
                e0[b], j0[b] = e, j
                e, j = e + ne[b], j + nj[b]
    assert e == count and j == total
    tab, off = np.full(count, -1), np.zeros(count, dtype=np.int64)
    ce, cj = dict(e0), dict(j0)
    for k in range(count):
        b = op[k] * ncls + cl[k]
        tab[ce[b]], off[ce[b]] = k, cj[b]
        ce[b], cj[b] = ce[b] + 1, cj[b] + n[k]
    assert np.all(tab >= 0) and np.all(np.diff(off) > 0)
    done = [np.zeros(x, dtype=np.int64) for x in n]
    queue = np.zeros(total, dtype=np.int64)
    for ph in range(3):
        for g in groups:
            spans, blocks = [], 0
            for c in g:
                b = ph * ncls + c
                if nj[b]:
                    spans.append((c, blocks, j0[b], j0[b] + nj[b], e0[b], e0[b] + ne[b]))
                    blocks += -(-nj[b] // K_REQ_OPS)
            for blk in range(blocks):
                s = 0
                while s + 1 < len(spans) and blk >= spans[s + 1][1]:
                    s += 1
                c, b0, lo, hi, ea, eb = spans[s]
                p0 = lo + (blk - b0) * K_REQ_OPS
                p1 = min(hi, p0 + K_REQ_OPS)
                assert lo <= p0 < p1 <= hi
                a, z = find_entry(off, ea, eb, p0), find_entry(off, ea, eb, p1 - 1) + 1
                for p in range(p0, p1):
                    k = find_entry(off, a, z, p)
                    r = tab[k]
                    assert op[r] == ph and cl[r] == c and 0 <= p - off[k] < n[r]
                    done[r][p - off[k]] += 1
                if ph == 2:
                    queue[p0:p1] += 1
    assert all(np.all(d == 1) for d in done)
    assert queue.max(initial=0) <= 1 and total <= layout(total)["queue"]
