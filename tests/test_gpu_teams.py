"""Small iterations run by a team of blocks inside one launch: frontiers whose
edge counts lie on either side of a wave, a block, the team's limit and the
appending limit, long chains that one launch carries over many iterations, and
the relaxation's team rounds.

Every window's values equal the oracle's with the team and the appended lists
off (append_edges 0) and on.  Values are uint32: tolerance zero.
"""
import numpy as np
import pytest

import oracle
import synth
from gpu_util import assert_equal_values, gpu_values

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def evq():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2502_10579_amd as m
    return m


def layered_instance(widths, deg, K, churn, seed):
    """Layers of the given widths; every vertex has `deg` edges into the next layer, drawn so that the whole next
    layer is reached.  Each batch replaces `churn` edges, so that windows have partial edges in every layer."""
    rng = np.random.default_rng(seed)
    at = np.concatenate([[0], np.cumsum(widths)])
    rows = []
    for i in range(len(widths) - 1):
        n, m = widths[i], widths[i + 1]
        d = max(deg, -(-m // n))
        src = np.repeat(np.arange(n), d)
        dst = np.concatenate([np.arange(m), rng.integers(0, m, n * d - m)]) if n * d >= m else rng.integers(0, m, n * d)
        rows.append(np.stack([at[i] + src, at[i + 1] + dst, rng.integers(1, 40, n * d)], 1))
    base = np.unique(np.concatenate(rows).astype(np.uint32), axis=0)
    dels, adds, cur = [], [], base
    for _ in range(K):
        out = cur[rng.choice(len(cur), min(churn, len(cur)), replace=False)]
        new = out.copy()
        new[:, 2] = rng.integers(1, 40, len(out))
        dels.append(out)
        adds.append(new)
    return synth.Instance(int(at[-1]), base, dels, adds)


SHAPES = {
    "chain": ([1] * 3000, 1),  # more iterations than one launch carries
    "tiles": ([1, 1, 63, 64, 65, 511, 512, 513, 7, 1, 1, 4095, 4096, 4097, 3, 1], 2),
    # about 32760, 32768 and 32776 edges (less a few equal draws) from the fourth layer: the team's limit
    "limit_below": ([1, 64, 512, 4095, 900, 30, 1, 1], 8),
    "limit": ([1, 64, 512, 4096, 900, 30, 1, 1], 8),
    "limit_above": ([1, 64, 512, 4097, 900, 30, 1, 1], 8),
    # about 131064 and 131080 edges: the appending limit
    "append": ([1, 64, 2048, 16383, 500, 16385, 40, 1, 1, 1], 8),
}


@pytest.mark.parametrize("K", [5, 70])
@pytest.mark.parametrize("shape", list(SHAPES))
def test_frontier_sizes(evq, shape, K):
    widths, deg = SHAPES[shape]
    inst = layered_instance(widths, deg, K, 3 if shape == "chain" else 60, len(widths) + K)
    rep = oracle.replay(inst)
    V = inst.num_vertices
    with evq.Graph.from_instance(inst) as g:
        for a in (0, 1, 2, 4):
            for b, L in ((0, K), (K - 3, 3)):
                want = oracle.window_values(inst, a, 0, b, L, replayed=rep)
                for limit in (0, 1 << 17):
                    with evq.tuning(append_edges=limit):
                        got = gpu_values(g, a, 0, b, L)
                    assert_equal_values(got, want, f"{shape} V={V} K={K} algo={a} window=({b},{L}) append={limit}")


@pytest.mark.parametrize("a", range(5))
@pytest.mark.parametrize("wmax", [1, 3, 4294967295])
def test_reduction_at_ties(evq, a, wmax):
    """The reduced subgraph leaves out the edges that the bounds show to be useless: equal weights make the
    bounds of an edge's ends tie, the largest weights saturate, and a third of the vertices is unreached."""
    V, K = 90, 9
    inst = synth.random_instance(60, 150, K, 12, 12, 5, 31 + a)
    top = np.uint64(wmax)
    scale = lambda e: np.stack([e[:, 0], e[:, 1], (np.uint64(1) + (e[:, 2].astype(np.uint64) - 1) * (top - 1) // 4)],
                               1).astype(np.uint32)
    inst = synth.Instance(V, scale(inst.base), [scale(d) for d in inst.dels], [scale(x) for x in inst.adds])
    rep = oracle.replay(inst)
    with evq.Graph.from_instance(inst) as g:
        for src in (0, 17, 75):
            for b, L in ((0, K), (0, 1), (3, 4), (K - 1, 1)):
                want = oracle.window_values(inst, a, src, b, L, replayed=rep)
                for kind in ({}, {"plain": True}, {"sequential": True}):
                    assert_equal_values(gpu_values(g, a, src, b, L, **kind), want, f"wmax={wmax} {src} {b} {L} {kind}")
