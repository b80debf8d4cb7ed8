"""The reduction leaves out edges that the bounds show to be useless, unless the
intersection solve reached less than a thousandth of the unstable vertices: then
next to nothing could be left out, and the bounds are not read.

A source whose edge into a large subgraph changes in every snapshot, and a
stable path beside it of few vertices or many.  The edges from the subgraph into
the path's first vertex cannot improve it.  Values equal the oracle's: tolerance
zero.
"""
import numpy as np
import pytest

import oracle
import synth
from gpu_util import assert_equal_values, gpu_values

pytestmark = pytest.mark.gpu

K, N, USELESS = 8, 3000, 500  # snapshots, vertices of the subgraph, its edges into the path


@pytest.fixture(scope="module")
def evq():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2502_10579_amd as m
    return m


def instance(path):
    """0 -> 1 changes; 1 -> 2 .. N + 1 in a ring with chords; 0 -> P stable, P -> P + 1 -> ... (path vertices)."""
    rng = np.random.default_rng(path)
    P = N + 2
    ring = np.arange(1, N + 1)
    rows = [np.stack([ring, ring + 1, np.full(N, 3)], 1),
            np.stack([rng.integers(1, N + 2, 2 * N), rng.integers(2, N + 2, 2 * N), rng.integers(1, 9, 2 * N)], 1),
            np.array([[0, P, 50], [1, P, 3]])]
    rows.append(np.stack([np.arange(2, 2 + USELESS), np.full(USELESS, P), np.full(USELESS, 60)], 1))
    rows += [np.array([[P + i, P + i + 1, 2]]) for i in range(path - 1)]
    first = lambda k: np.array([[0, 1, 10 + k]], np.uint32)
    base = np.unique(np.concatenate([first(0)] + rows).astype(np.uint32), axis=0)
    return synth.Instance(P + path, base, [first(k) for k in range(K)], [first(k + 1) for k in range(K)])


@pytest.mark.parametrize("path,left_out", [(1, False), (2, True), (40, True)])
def test_bounds_are_read_where_they_leave_edges_out(evq, path, left_out):
    inst = instance(path)
    rep = oracle.replay(inst)
    between = len(inst.base) - 2  # every edge but the two from the source has unstable ends
    with evq.Graph.from_instance(inst) as g:
        got, st = gpu_values(g, oracle.SSSP, 0, 0, K, stats=True)
        assert_equal_values(got, oracle.window_values(inst, oracle.SSSP, 0, 0, K, replayed=rep), f"path={path}")
        assert st["n_unstable"] == N + 1 + path
        if left_out:
            assert st["n_relax_edges"] <= between - USELESS, st
        else:
            assert st["n_relax_edges"] == between, st
        for a in range(1, 5):
            for b, L in ((0, K), (2, 5)):
                want = oracle.window_values(inst, a, 0, b, L, replayed=rep)
                for kind in ({}, {"sequential": True}):
                    assert_equal_values(gpu_values(g, a, 0, b, L, **kind), want, f"path={path} algo={a} {(b, L)} {kind}")
