"""A set of many classes, one batch through the class kernels against the same
operations in small batches, which run one launch per phase and group of
classes: same answers, counts and stored content."""
import numpy as np
import pytest

from oracle import OracleFilter
from gpu_util import dev_u64, host_u64
from workloads import keys as K

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def cf():
    import paper_2603_15486_amd as mod
    return mod


# (f, hash, placement) of the classes, and bucket sizes each: groups that mix
# fingerprint widths, and groups of one class
@pytest.mark.parametrize("combos,bs,small", [
    ([(8, 0, 0), (16, 0, 0), (32, 0, 0)], (4, 32), 30_011),
    ([(f, h, p) for f in (8, 16, 32) for h in (0, 1) for p in (0, 1)], (8,), 4_099),
    ([(16, 1, 1)], (4, 8, 16, 32), 65_537)])
@pytest.mark.parametrize("streams", [0, 1])
def test_class_kernels_equal_small_batches(cf, combos, bs, small, streams):
    n = (1 << 20) + 4097
    specs = [(f, h, p, b) for f, h, p in combos for b in bs]
    nf = len(specs)
    slots = 4 * n // nf
    params = [cf.make_params((1 << (slots // b).bit_length()) - (3 if p else 0), b, f, hash=h,
                             placement=p, seed=31 + i) for i, (f, h, p, b) in enumerate(specs)]
    rng = np.random.default_rng(5)
    pre = K.keys(9, 0, n)
    pre_fid = rng.integers(0, nf, n).astype(np.uint32)
    # a third each: queries of stored and other keys, deletes of stored keys
    # (each once), inserts of new ones; then some invalid operations
    kind = rng.integers(0, 3, n).astype(np.uint8)
    keys, fids = pre.copy(), pre_fid.copy()
    other = (kind == 0) & (rng.random(n) < 0.5)
    keys[other] = K.negatives(9, 0, int(other.sum()))
    new = kind == 2
    keys[new] = K.keys(9, 1 << 40, int(new.sum()))
    fids[new] = rng.integers(0, nf, int(new.sum()))
    bad = rng.random(n) < 0.01
    kind[bad] = 7
    perm = rng.permutation(n)
    kind, fids, keys = kind[perm], fids[perm], keys[perm]

    def run(s, sel, step):
        out = np.zeros(sel.size, dtype=np.uint8)
        for lo in range(0, sel.size, step):
            i = sel[lo:lo + step]
            out[lo:lo + step] = s.execute(torch.from_numpy(kind[i]).cuda(),
                                          torch.from_numpy(fids[i].view(np.int32)).cuda(),
                                          dev_u64(keys[i])).cpu().numpy()
        return out

    sets = []
    for _ in range(2):
        s = cf.CuckooFilterSet(params, n)
        s.streams = streams
        ops = torch.full((n,), cf.CF_OP_INSERT, dtype=torch.uint8, device="cuda")
        ok = s.execute(ops, torch.from_numpy(pre_fid.view(np.int32)).cuda(), dev_u64(pre))
        assert bool(ok.all())
        sets.append(s)
    whole = run(sets[0], np.arange(n), n)
    for sel in (np.flatnonzero(kind == 0), np.flatnonzero(kind == 1), np.flatnonzero(kind == 2),
                np.flatnonzero(kind == 7)):
        assert np.array_equal(run(sets[1], sel, small), whole[sel])
    assert np.all(whole[kind == 7] == 0xFF) and np.all(whole[kind == 2] == 1)
    assert np.all(whole[kind == 1] == 1)
    assert np.array_equal(sets[0].counts(), sets[1].counts())
    assert not sets[0].failures().any() and not sets[1].failures().any()
    for i, (f, h, p, b) in enumerate(specs):
        r = OracleFilter(params[i].num_buckets, b, f, hash_kind=h, seed=31 + i, placement=p)
        digests = []
        for s in sets:
            r.load_words(host_u64(s.export_table(i)))
            digests.append(r.digest_table())
        assert digests[0] == digests[1]
        r.close()
    for s in sets:
        s.close()
