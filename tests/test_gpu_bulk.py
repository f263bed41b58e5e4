"""The partitioned insert (batches of 2^19 keys and more that are large
against the table): one and two levels of grouping, a cut last part, bins that overflow,
tables that are already partly full, and capture.  Whatever the path, every
key is stored or logged: flags, counts, kick bound and the stored
(bucket pair, fingerprint) content must be those of the inserted keys."""
import numpy as np
import pytest

import oracle
from oracle import OracleFilter
from gpu_util import (GEOMS, dev_u64, dev_zeros_u8, dev_zeros_u32, expected_groups, host_u64,
                      multiset_equal)
from workloads import keys as K

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def cf():
    import paper_2603_15486_amd as mod
    return mod


def _nonzero_slots(words, f):
    return int((words.view({8: torch.int8, 16: torch.int16, 32: torch.int32}[f]) != 0).sum())


@pytest.mark.parametrize("b,f", GEOMS)
@pytest.mark.parametrize("pl", [oracle.PLACE_XOR, oracle.PLACE_OFFSET])
def test_direct_insert_of_the_same_batch(cf, b, f, pl):
    """A batch of this size through cf_insert_noalloc, which never goes
    partitioned: the direct kernel under the same contention."""
    m = (1 << 20) // b - (5 if pl else 0)
    n = int(0.9 * m * b)
    g = cf.CuckooFilter(m, b, f, seed=12, placement=pl)
    keys = K.keys(12, 0, n)
    ok = dev_zeros_u8(n)
    g.insert_noalloc(dev_u64(keys), ok)
    assert int(ok.sum()) == n - g.failures() == g.count()
    words = g.export_table()
    assert _nonzero_slots(words, f) == g.count()
    r = OracleFilter(m, b, f, seed=12, placement=pl)
    r.load_words(host_u64(words))
    assert multiset_equal(r.stored_groups(), expected_groups(r, keys, lost=g.lost()))
    g.close()
    r.close()


# tables of one level of parts (up to 1024) and, the last four, of two; the
# offset ones end in a cut part, the 4-byte buckets of an odd count in one
# that is no multiple of 16 bytes
@pytest.mark.parametrize("m,b,f,pl,hk,before,after", [
    ((1 << 17) + 3, 16, 16, 1, 1, 0.5, 0.92), (1 << 16, 32, 32, 0, 0, 0.5, 0.92),
    (1 << 18, 8, 8, 0, 0, 0.5, 0.9), ((1 << 22) + 4097, 4, 8, 1, 0, 0.5, 0.85),
    (3 * (1 << 18) + 7, 16, 16, 1, 0, 0.5, 0.92), (1 << 20, 8, 32, 0, 1, 0.5, 0.9),
    (1 << 21, 4, 16, 0, 0, 0.5, 0.85), (1 << 19, 32, 32, 0, 0, 0.1, 0.36),
    ((1 << 23) + 4097, 4, 16, 1, 0, 0.05, 0.31), ((1 << 21) + 5, 16, 16, 1, 1, 0.5, 0.9),
    ((1 << 24) + 4097, 4, 8, 1, 0, 0.02, 0.15), ((1 << 19) + 3, 32, 32, 1, 1, 0.6, 0.92)])
def test_partitioned_fill_on_a_part_full_table(cf, m, b, f, pl, hk, before, after):
    slots = m * b
    g = cf.CuckooFilter(m, b, f, hash=hk, seed=5, placement=pl)
    first = int(before * slots) + 3
    n = int(after * slots) - first
    assert n >= slots // (4 if n < 1 << 20 else 8 if n < 1 << 22 else 12) and n >= 1 << 19
    keys = K.keys(5, 0, first + n)
    g.insert(dev_u64(keys[:first]))
    ok, kicks = dev_zeros_u8(n), dev_zeros_u32(n)
    g.insert(dev_u64(keys[first:]), ok, kicks)
    assert g.failures() == 0 and bool(ok.all())
    assert int(kicks.max()) <= 128 and int(kicks.min()) >= 0
    words = g.export_table()
    assert g.count() == _nonzero_slots(words, f) == keys.size
    assert bool(g.query(dev_u64(keys)).all())
    r = OracleFilter(m, b, f, hash_kind=hk, seed=5, placement=pl)
    r.load_words(host_u64(words))
    assert r.digest_table() == r.digest_keys(keys)
    g.close()
    r.close()


def test_overflowing_bin(cf):
    """Keys crowded into one part overflow its bin and take the other list;
    nothing is lost."""
    m, b, f = 1 << 16, 16, 16
    r = OracleFilter(m, b, f, seed=6)
    pool = K.keys(6, 0, 3 << 20)
    i1 = np.asarray(r.derive_batch(pool)[1])
    crowd = pool[i1 < 256][:9000]  # 2048 expected, and twice the part's slots
    keys = np.concatenate([crowd, K.keys(6, 1 << 30, 1 << 19)])
    assert crowd.size == 9000
    g = cf.CuckooFilter(m, b, f, seed=6)
    ok, kicks = dev_zeros_u8(keys.size), dev_zeros_u32(keys.size)
    g.insert(dev_u64(keys), ok, kicks)
    assert g.failures() == 0 and bool(ok.all()) and g.count() == keys.size
    r.load_words(host_u64(g.export_table()))
    assert multiset_equal(r.stored_groups(), r.key_groups(keys))
    g.close()
    r.close()


@pytest.mark.parametrize("b,f", [(4, 8), (16, 16), (8, 32)])
def test_copies_of_few_keys_fail_and_are_logged(cf, b, f):
    """Copies beyond a pair's 2b slots cannot be stored: each is reported,
    counted and logged."""
    m = (1 << 20) // b
    base = K.keys(7, 0, 64)
    keys = np.concatenate([np.repeat(base, 4 * b), K.keys(7, 1000, 1 << 19)])
    g = cf.CuckooFilter(m, b, f, max_evict=8, seed=7)
    ok = dev_zeros_u8(keys.size)
    g.insert(dev_u64(keys), ok)
    fails = g.failures()
    assert fails >= 64 * 2 * b and int(ok.sum()) == keys.size - fails == g.count()
    r = OracleFilter(m, b, f, max_evict=8, seed=7)
    r.load_words(host_u64(g.export_table()))
    assert r.count == g.count()
    assert multiset_equal(r.stored_groups(), expected_groups(r, keys, lost=g.lost()))
    g.close()
    r.close()


@pytest.mark.parametrize("m,b,f", [(64, 16, 16), (1 << 14, 16, 8)])
def test_batch_that_cannot_fit(cf, m, b, f):
    """Batches of 512 and of two times the slots: what does not fit is
    reported, counted and logged (the log keeps its first entries)."""
    n = 1 << 19
    g = cf.CuckooFilter(m, b, f, max_evict=4, seed=13, lost_capacity=n)
    keys = K.keys(13, 0, n)
    ok = dev_zeros_u8(n)
    g.insert(dev_u64(keys), ok)
    fails = g.failures()
    assert int(ok.sum()) == n - fails == g.count() <= m * b
    r = OracleFilter(m, b, f, max_evict=4, seed=13)
    r.load_words(host_u64(g.export_table()))
    lost = g.lost(n)
    assert len(lost[0]) == fails and r.count == g.count()
    want = (r.digest_keys(keys) - r.digest_pairs(*lost)) % 2**64
    assert r.digest_table() % 2**64 == want
    g.close()
    r.close()


def test_captured_and_replayed(cf):
    """Reset and partitioned insert in one graph, replayed between eager
    work: each replay leaves the same content."""
    m, b, f = 1 << 17, 8, 16
    n = int(0.9 * m * b)
    g = cf.CuckooFilter(m, b, f, seed=8)
    keys = dev_u64(K.keys(8, 0, n))
    ok = dev_zeros_u8(n)
    g.reserve(n)
    g.insert(keys, ok)
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        g.reset()
        g.insert(keys, ok)
    for k in range(3):
        ok.zero_()
        g.reset()
        g.insert(keys[: n // 2 + k], ok[: n // 2 + k])
        torch.cuda.synchronize()
        ok.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert bool(ok.all()) and g.count() == n and g.failures() == 0
        assert bool(g.query(keys).all())
        assert _nonzero_slots(g.export_table(), f) == n
    g.close()


@pytest.mark.parametrize("extra", [0, 1, 3])
def test_most_bucket_bits_of_an_entry(cf, extra):
    """2^29 buckets of 4 x 16 bits (4 GiB) take every bucket bit of an entry; with a
    few buckets more there is none left for the topmost, and the batch goes
    direct.  Either way every key is found where queries look."""
    m, n = (1 << 29) + extra, 1 << 27
    g = cf.CuckooFilter(m, 4, 16, seed=14, placement=oracle.PLACE_OFFSET)
    keys = torch.empty(n, dtype=torch.int64, device="cuda")
    cf.cf_keygen(keys, 14, 0)
    ok = dev_zeros_u8(n)
    g.insert(keys, ok)
    assert g.failures() == 0 and bool(ok.all()) and g.count() == n
    assert bool(g.query(keys).all())
    g.close()
