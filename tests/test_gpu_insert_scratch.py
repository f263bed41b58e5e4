"""What a filter's inserts allocate and keep: cf_reserve and a larger batch
before cover every smaller one, whichever way the batches go."""
import pytest

from gpu_util import dev_u64, dev_zeros_u8
from workloads import keys as K

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def cf():
    import paper_2603_15486_amd as mod
    return mod


def _free():
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0]


def _inserts_allocate_nothing(cf, g, keys, sizes):
    """Inserts of these sizes into an emptied filter leave free memory alone."""
    warm = cf.CuckooFilter(g.num_buckets, g.slots_per_bucket, g.params.fp_bits)
    for n in sizes:  # what the runtime itself takes for these launches
        warm.reset()
        warm.insert(keys[:n])
        warm.query(keys[:n])
    for n in sizes:
        ok = dev_zeros_u8(n)
        g.reset()
        g.query(keys[:n])
        free = _free()
        g.insert(keys[:n], ok)
        assert _free() == free, n
        assert bool(ok.all()) and g.count() == n and bool(g.query(keys[:n]).all())


def test_reserve_beyond_twice_the_slots(cf):
    """A reserve for batches that go direct covers the smaller ones that go
    partitioned."""
    m, b, f = 1 << 16, 16, 16
    g = cf.CuckooFilter(m, b, f, seed=21)
    keys = dev_u64(K.keys(21, 0, int(0.95 * m * b)))
    g.reserve(1 << 24)
    _inserts_allocate_nothing(cf, g, keys, (keys.numel(), 1 << 19, 5000))
    g.close()


def test_smaller_batches_after_a_partitioned_one(cf):
    """A batch that goes partitioned leaves scratch for the smaller ones that
    go direct, eager or captured."""
    m, b, f = 1 << 18, 16, 16
    g = cf.CuckooFilter(m, b, f, seed=22)
    keys = dev_u64(K.keys(22, 0, int(0.95 * m * b)))
    n = (1 << 20) - 1  # one key short of the rule's line
    g.insert(keys)
    _inserts_allocate_nothing(cf, g, keys, (n, 1 << 19, 5000))
    ok = dev_zeros_u8(n)
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        g.reset()
        g.insert(keys[:n], ok)
    for _ in range(3):
        g.reset()
        g.insert(keys[n:2 * n])
        ok.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert bool(ok.all()) and g.count() == n and bool(g.query(keys[:n]).all())
    g.close()


def test_smaller_batches_after_one_that_cannot_fit(cf):
    """A batch of more than twice the slots goes direct; the smaller ones that
    would go partitioned have no workspace then, and allocate none."""
    m, b, f = 1 << 16, 16, 16
    g = cf.CuckooFilter(m, b, f, max_evict=32, seed=23)
    keys = dev_u64(K.keys(23, 0, 3 * m * b))
    g.insert(keys)
    _inserts_allocate_nothing(cf, g, keys, (int(0.9 * m * b), 1 << 19, 1 << 17))
    g.close()


def test_captured_insert_outlives_its_workspace(cf):
    """A larger batch replaces the workspace; graphs captured before keep
    theirs and leave the new one alone."""
    m, b, f = 1 << 17, 16, 16
    sizes = [int(share * m * b) for share in (0.3, 0.5, 0.9)]
    g = cf.CuckooFilter(m, b, f, seed=24)
    keys = dev_u64(K.keys(24, 0, sizes[-1]))
    ok = dev_zeros_u8(sizes[-1])
    graphs = []
    for n in sizes:
        g.reset()
        g.insert(keys[:n])  # outgrows the one before
        graph = torch.cuda.CUDAGraph()
        torch.cuda.synchronize()
        with torch.cuda.graph(graph):
            g.reset()
            g.insert(keys[:n], ok[:n])
        graphs.append(graph)
    for k in (0, 1, 2, 0, 2, 1, 1, 0):
        n = sizes[k]
        ok.zero_()
        torch.cuda.synchronize()
        graphs[k].replay()
        torch.cuda.synchronize()
        assert int(ok.sum()) == n == g.count() and bool(g.query(keys[:n]).all())
        g.reset()
        g.insert(keys, ok)
        assert bool(ok.all()) and g.count() == sizes[-1]
    del graphs
    g.close()
