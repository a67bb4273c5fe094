"""SISe_sp with neighbour lists of every length around what a node's lanes read
at once (4 each, of 1 to 64 lanes): none, one, a chunk less one, a chunk, more
than one chunk, in lists that are not symmetric, for every number of lanes a
node can have, against the oracle (states equal, continuous state 1e-12)."""
import os

import numpy as np
import pytest

from paper_1605_01421_amd import workloads as W

pytestmark = pytest.mark.gpu

NTHREADS = min(16, os.cpu_count() or 1)


@pytest.mark.parametrize("opts", [dict(), dict(pack=4), dict(pack=8), dict(pack=16), dict(pack=32), dict(pack=64),
                                  dict(lanes=64, wide=40), dict(lanes=1, group=-1),
                                  dict(lanes=64, wide=5, group=20, pack=8)])
def test_neighbour_lists(opts):
    import oracle
    from paper_1605_01421_amd import siminf
    rng = np.random.default_rng(3)
    Nn, days = 300, 25
    sizes = [0, 1, 2, 3, 4, 5, 7, 8, 9, 15, 16, 17, 31, 32, 33, 63, 64, 65, 127, 255, 256, 257, 299]
    ptr, idx, dist = [0], [], []
    for i in range(Nn):
        k = sizes[i % len(sizes)]
        others = np.delete(np.arange(Nn), i)
        j = np.sort(rng.choice(others, size=min(k, Nn - 1), replace=False))
        idx.append(j)
        dist.append(rng.uniform(20.0, 900.0, len(j)))
        ptr.append(ptr[-1] + len(j))
    nb = dict(ptr=np.array(ptr, np.int32), idx=np.concatenate(idx).astype(np.int32), dist=np.concatenate(dist))
    u0 = np.stack([rng.integers(0, 60, Nn), rng.integers(0, 4, Nn)], 1)
    u0[::29] = 0  # empty nodes: their sum is 0, but they post and wait
    spec = W.sise_sp_spec(u0, np.arange(days + 1), 0.02, 0.1, 1.0, (0.1, 0.12, 0.12, 0.1), 0.01, nb, phi0=0.2)
    print("[gpu] coupling", opts, flush=True)
    ref = oracle.run(spec, 5, 1, nthreads=NTHREADS)
    m = siminf.Model(spec, **opts)
    m.run(5, 1)
    assert m.wait() == 0 and ref["status"] == 0
    U, V = m.trajectory()
    assert np.array_equal(U, ref["U"])
    np.testing.assert_allclose(V, ref["V"], rtol=1e-12, atol=0)
