"""Ring appends at the edges of the append's tiles: words of 64 edges, tiles of
2048 edges, and tiles that span more than 2048 rows (long runs of vertices
without edges between the few that have some).

The incremental append's arrays equal those of a full rebuild
(evq_tuning.append_rebuild) exactly, and the ring masks equal the oracle's
replay of the history.  Integers: tolerance zero.
"""
import numpy as np
import pytest

import oracle
import synth
from gpu_util import union_triples_from_export

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def evq():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2502_10579_amd as m
    return m


def sparse_instance(V, n_base, K, n_upd, seed):
    """n_base distinct base triples whose sources are 5000 ids apart at least now and then: most vertices have
    no edge."""
    rng = np.random.default_rng(seed)
    base = np.stack([np.sort(rng.integers(0, V, n_base)), rng.integers(0, V, n_base),
                     rng.integers(1, 50, n_base)], 1).astype(np.uint32)
    base = np.unique(base, axis=0)
    while len(base) < n_base:
        more = np.array([[rng.integers(0, V), rng.integers(0, V), 50]], dtype=np.uint32)
        base = np.unique(np.concatenate([base, more]), axis=0)
    dels = [base[rng.choice(len(base), n_upd, replace=False)] for _ in range(K)]
    adds = [np.stack([rng.integers(0, V, n_upd), rng.integers(0, V, n_upd), rng.integers(1, 50, n_upd)],
                     1).astype(np.uint32) for _ in range(K)]
    return synth.Instance(V, base, dels, adds)


@pytest.mark.parametrize("order", [0, 1])
@pytest.mark.parametrize("V,n_base,K,n_upd", [
    (9, 64, 1, 3), (40, 63, 3, 0), (40, 128, 8, 5), (200000, 2048, 64, 7), (200000, 2049, 65, 9),
    (300000, 6143, 128, 20), (1000, 8192, 100, 40)])
def test_append_equals_rebuild(evq, V, n_base, K, n_upd, order):
    inst = sparse_instance(V, n_base, K + 3, n_upd, 7 * n_base + K)
    got = []
    with evq.tuning(vertex_order=order):
        for rebuild in (0, 1):
            with evq.tuning(append_rebuild=rebuild):
                with evq.Graph(V, inst.base, inst.dels[:K], inst.adds[:K]) as g:
                    for a in range(3):
                        g.append(inst.dels[K + a], inst.adds[K + a])
                    got.append(g.export())
    for k in got[0]:
        assert np.array_equal(got[0][k], got[1][k]), k
    if K + 3 > 128:
        return  # past the oracle's snapshots: the rebuild stands in for it
    trip, bits = oracle.replay(inst)
    want = {}
    for r, b in zip(trip, bits):
        m = int(b[0]) | (int(b[1]) << 64)
        ring = sum(1 << (t % K) for t in range(3, K + 3) if (m >> t) & 1)
        if ring:
            want[tuple(int(x) for x in r)] = ring
    assert union_triples_from_export(got[0], K) == want
