"""Batches of the serving loop with requests on a filter that was detached
through the server's set: those get 0xFF, as in a mixed batch, and the others
are served."""
import numpy as np
import pytest

from gpu_util import dev_u64
from workloads import keys as K

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def cf():
    import paper_2603_15486_amd as mod
    return mod


def test_requests_on_a_detached_filter_in_a_batch(cf):
    nf, per, rounds = 3, 5000, 20
    params = [cf.make_params(1 << 10, 16, 16, seed=f) for f in range(nf)]
    srv = cf.CuckooServer(params, max_batch=1 << 20, direct_below=1)
    keys = [dev_u64(K.keys(40 + f, 0, per)) for f in range(nf)]
    for f in range(nf):
        srv.set.apply(f, cf.CF_OP_INSERT, keys[f])
    torch.cuda.synchronize()
    srv.set.detach(1)
    out = [torch.zeros(per, dtype=torch.uint8, device="cuda") for _ in range(rounds * nf)]
    torch.cuda.synchronize()
    ids = [srv.submit(k % nf, cf.CF_OP_QUERY, keys[k % nf], out[k]) for k in range(rounds * nf)]
    for k, rid in enumerate(ids):
        assert srv.wait(rid).status == cf.CF_OK, k
    for k, o in enumerate(out):
        assert np.all(o.cpu().numpy() == (0xFF if k % nf == 1 else 1)), k
    srv.close()
