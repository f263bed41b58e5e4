"""The partitioned insert at its limits: batches of several passes, and bins
that overflow in each of its grouping steps (the first split, the split into
parts, the move to the second bucket), for 8-byte and 12-byte entries, on
tables of one and of two grouping levels.  Nothing may be lost: flags, counts
and the stored (bucket pair, fingerprint) content are those of the keys."""
import os

import numpy as np
import pytest

from oracle import OracleFilter
from gpu_util import dev_u64, dev_zeros_u8, dev_zeros_u32, host_u64
from workloads import keys as K

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def cf():
    import paper_2603_15486_amd as mod
    return mod


def _filter(cf, pass_keys, *args, **kw):
    """A filter whose partitioned passes have at most pass_keys keys."""
    os.environ["CF_INSERT_PASS_KEYS"] = str(pass_keys)
    try:
        return cf.CuckooFilter(*args, **kw)
    finally:
        os.environ.pop("CF_INSERT_PASS_KEYS")


def _copies(i, c):
    """Keys `i` of stream 32, c of each, spread over a batch by the caller."""
    return np.repeat(K.keys(32, 0, i), c)


# tables of one and of two levels, 8-byte and 12-byte entries; passes that
# divide the batch unevenly
@pytest.mark.parametrize("m,b,f,pl,n,pass_keys", [
    ((1 << 17) + 3, 16, 16, 1, (1 << 20) + 77, 300_001), (1 << 18, 8, 8, 0, 1 << 20, 1 << 18),
    (1 << 19, 8, 32, 0, (1 << 21) + 1, 700_000), ((1 << 23) + 4097, 4, 16, 1, 6_000_007, 1_500_000),
    ((1 << 21) + 5, 8, 32, 1, 8_500_007, 2_200_007), (1 << 18, 32, 16, 0, 3 << 20, 1 << 16)])
@pytest.mark.parametrize("evict", [0, 1])
def test_several_passes(cf, m, b, f, pl, n, pass_keys, evict):
    """Every flag, kick count, log entry and index of a pass belongs to its own
    keys: only copies of a few keys fail, and keys that share a bucket with
    them (their search displaces a copy, which then has no place)."""
    hot, c = 16, 4 * b
    keys = np.concatenate([K.keys(31, 0, n - hot * c), _copies(hot, c)])
    # even bucket counts, so that copies spread over the passes
    perm = np.random.default_rng(31).permutation(n)
    keys = keys[perm]
    is_hot = perm >= n - hot * c
    D = 64
    r = OracleFilter(m, b, f, seed=31, placement=pl)
    _, i1, i2 = (np.asarray(x) for x in r.derive_batch(keys))
    full = np.concatenate([i1[is_hot], i2[is_hot]])
    may_fail = np.isin(i1, full) | np.isin(i2, full)
    g = _filter(cf, pass_keys, m, b, f, seed=31, placement=pl, evict=evict, max_evict=D)
    d = dev_u64(keys)
    for _ in range(2):  # the second on the workspace as the first left it
        g.reset()
        ok, kicks = dev_zeros_u8(n), dev_zeros_u32(n)
        g.insert(d, ok, kicks)
        okv, kv = ok.cpu().numpy().astype(bool), kicks.cpu().numpy()
        fails = g.failures()
        assert fails >= hot * 2 * b and int(okv.sum()) == n - fails == g.count()
        # the random walk may also get there by a few steps; with flags at
        # other keys' places nearly all of them would be elsewhere
        assert (~okv & ~may_fail).sum() <= (fails // 4 if evict else 0)
        assert kv.min() >= 0 and kv.max() <= D and (kv[~okv] == D).all()
        r.load_words(host_u64(g.export_table()))
        lost = g.lost()
        assert len(lost[0]) == fails
        want = (r.digest_keys(keys) - r.digest_pairs(*lost)) % 2**64
        assert r.digest_table() % 2**64 == want
    r.close()
    g.close()


def test_two_passes_of_the_longest(cf):
    """A batch of more than 2^27 keys."""
    m, b, f, n = 1 << 24, 16, 16, (1 << 27) + 12345
    g = cf.CuckooFilter(m, b, f, seed=33)
    keys = torch.empty(n, dtype=torch.int64, device="cuda")
    cf.cf_keygen(keys, 33, 0)
    ok = dev_zeros_u8(n)
    g.insert(keys, ok)
    assert g.failures() == 0 and bool(ok.all()) and g.count() == n
    assert bool(g.query(keys).all())
    g.close()


def _check(g, r, keys, ok, more=0):
    assert g.failures() == 0 and bool(ok.all())
    r.load_words(host_u64(g.export_table()))
    assert r.digest_table() % 2**64 == (r.digest_keys(keys) + more) % 2**64
    assert bool(g.query(dev_u64(keys)).all())


# (table, batch, buckets of the crowded part, its entries' capacity, crowd):
# the crowd with the part's share of the other keys exceeds the capacity, and
# fits the part's slots
@pytest.mark.parametrize("m,b,f,pl,n,part,cap,crowd", [
    # one level: the first split, eight runs
    (1 << 19, 8, 32, 0, 1 << 21, 2048, 8 * 1328, 9000),
    # two levels: the split into parts
    ((1 << 21) + 5, 16, 16, 1, 4_400_000, 2048, 4848, 6000),
    ((1 << 21) + 5, 8, 32, 1, 4_300_000, 2048, 4752, 9000)])
def test_crowded_part(cf, m, b, f, pl, n, part, cap, crowd):
    r = OracleFilter(m, b, f, seed=34, placement=pl)
    first = []
    for lo in range(0, 40 << 20, 1 << 21):
        pool = K.keys(34, (1 << 40) + lo, 1 << 21)
        first.append(pool[np.asarray(r.derive_batch(pool)[1]) < part])
        if sum(map(len, first)) >= crowd:
            break
    first = np.concatenate(first)[:crowd]
    assert first.size == crowd and crowd + n * part // m > cap
    keys = np.concatenate([first, K.keys(34, 0, n)])
    keys = keys[np.random.default_rng(34).permutation(keys.size)]
    g = cf.CuckooFilter(m, b, f, seed=34, placement=pl)
    ok = dev_zeros_u8(keys.size)
    g.insert(dev_u64(keys), ok)
    _check(g, r, keys, ok)
    g.close()
    r.close()


# every even bucket is full from the start, so keys with an even i1 move to
# their i2; those of the crowd all move to one part
@pytest.mark.parametrize("m,b,f,n,part,cap,crowd", [
    (1 << 18, 16, 16, 1 << 20, 1024, 8 * 736, 9000),       # one level
    (1 << 20, 8, 32, 1 << 21, 2048, 8 * 720, 9000),        # one level, 12 bytes
    (1 << 22, 16, 16, 6_000_000, 2048, 3392, 5200)])       # two levels
def test_crowded_second_buckets(cf, m, b, f, n, part, cap, crowd):
    r = OracleFilter(m, b, f, seed=35)
    tags = np.random.default_rng(35).integers(1, 1 << f, (m, b)).astype(f"u{f // 8}")
    tags[1::2] = 0
    words = tags.reshape(-1).view(np.uint64)
    first = []
    for lo in range(0, 60 << 20, 1 << 21):
        pool = K.keys(35, (1 << 40) + lo, 1 << 21)
        _, i1, i2 = (np.asarray(x) for x in r.derive_batch(pool))
        first.append(pool[(i1 % 2 == 0) & (i2 < part)])
        if sum(map(len, first)) >= crowd:
            break
    first = np.concatenate(first)[:crowd]
    assert first.size == crowd and crowd + n * part // m // 2 > cap
    keys = np.concatenate([first, K.keys(35, 0, n)])
    keys = keys[np.random.default_rng(36).permutation(keys.size)]
    g = cf.CuckooFilter(m, b, f, seed=35)
    g.import_table(torch.from_numpy(words.view(np.int64)).cuda())
    ok = dev_zeros_u8(keys.size)
    g.insert(dev_u64(keys), ok)
    at = np.nonzero(tags)
    _check(g, r, keys, ok, r.digest_pairs(at[0], tags[at].astype(np.uint32)))
    g.close()
    r.close()


def test_captured_without_a_workspace(cf):
    """A batch that would go partitioned, captured on a filter that has only an
    eviction queue, goes direct."""
    m, b, f = 1 << 16, 16, 16
    n = int(0.9 * m * b)
    g = cf.CuckooFilter(m, b, f, max_evict=32, seed=37)
    keys = dev_u64(K.keys(37, 0, 3 * m * b))
    g.insert(keys)  # more than twice the slots: direct
    ok = dev_zeros_u8(n)
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        g.reset()
        g.insert(keys[:n], ok)
    for k in range(3):
        g.reset()
        g.insert(keys[n:2 * n - k])
        ok.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert bool(ok.all()) and g.count() == n and bool(g.query(keys[:n]).all())
    g.close()
