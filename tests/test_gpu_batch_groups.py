"""Batched bound solves over every lane-group size and task size: how a task's
edges reach the lanes of a group depends on the group's lanes (1 to 64) and on
the edges per task (4, 8, 16).  Each query of a batch equals the oracle on every
snapshot of its window; windows of one and two mask words, whole and partial.
Values are uint32: tolerance zero.
"""
import numpy as np
import pytest

import oracle
import synth
from gpu_util import assert_equal_values

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def evq():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2502_10579_amd as m
    before = m.batch_config()
    yield m
    m.set_batch_config(**before)


@pytest.mark.parametrize("chunk", [4, 8, 16])
@pytest.mark.parametrize("V,E,K,upd", [(70, 700, 8, 6), (300, 5000, 64, 40), (91, 900, 100, 6)])
def test_group_sizes(evq, V, E, K, upd, chunk):
    inst = synth.random_instance(V, E, K, upd, upd, 9, V + K)
    rep = oracle.replay(inst)
    rng = np.random.default_rng(V + chunk)
    evq.set_batch_config(lanes=1, chunk=chunk, group=64)
    with evq.Graph.from_instance(inst) as g:
        for n in (1, 2, 3, 5, 9, 20, 40):  # groups of 1, 2, 4, 8, 16, 32 and 64 lanes
            a = int(rng.integers(0, 5))
            qs = []
            for _ in range(n):
                b = int(rng.integers(0, K))
                qs.append((a, int(rng.integers(0, V)), b, int(rng.integers(1, K - b + 1))))
            for q, r in zip(qs, g.query_batch(qs)):
                want = oracle.window_values(inst, *q, replayed=rep)
                assert_equal_values(evq.to_u32(r.expand()).reshape(V, q[3]), want, f"n={n} chunk={chunk} {q}")
                r.free()
