"""launch_depth holds where no small iterations run many to a launch: the
near/far and bucketed schedules, and bound solves that append nothing.  Such a
loop issues its non-empty iterations and launch_depth more before it knows that
it is done.
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


@pytest.mark.parametrize("depth", [1, 3, 6])
@pytest.mark.parametrize("schedule,cup", [(dict(delta=8), True), (dict(delta=8, heavy=4), True),
                                          (dict(append_edges=0), True), (dict(bucket_width=10), False)])
def test_launches_in_flight(evq, schedule, cup, depth):
    inst = synth.rmat_instance(10, 8000, 8, 60, 60, seed=4)
    src = int(synth.pick_sources(inst, 1, seed=4)[0])
    want = {w: oracle.window_values(inst, oracle.SSSP, src, *w) for w in ((0, 8), (1, 6))}
    with evq.Graph.from_instance(inst) as g, evq.tuning(launch_depth=depth, **schedule):
        for (b, L), values in want.items():
            evq.timing_enable(True)
            evq.timing_reset()
            try:
                got, st = gpu_values(g, oracle.SSSP, src, b, L, stats=True)
                launches = {k: n for k, (n, ms) in evq.timing_report().items()}
            finally:
                evq.timing_enable(False)
            assert_equal_values(got, values, f"{schedule} depth={depth} window=({b},{L})")
            cap = launches["solve_expand_cap_all" if L == inst.K else "solve_expand_cap"]
            assert cap == st["iters_cap"] + depth, (cap, st["iters_cap"])
            if cup:
                assert launches["solve_expand_cup"] == st["iters_cup"] + depth, (launches, st["iters_cup"])


@pytest.mark.parametrize("depth", [1, 3, 6])
@pytest.mark.parametrize("layers,steady", [(12, False), (24, True)])
def test_launches_in_flight_above_the_teams_limit(evq, layers, steady, depth):
    """Layers of 8200 vertices and 32800 edges: every list but the source's goes to the launches."""
    n, d, K = 8200, 4, 2
    src, j = np.repeat(np.arange(n), d), np.tile(np.arange(d), n)
    rows = [np.stack([np.zeros(n, np.int64), 1 + np.arange(n), np.full(n, 2)], 1)]
    rows += [np.stack([1 + i * n + src, 1 + (i + 1) * n + (src + 977 * j) % n, 1 + j], 1) for i in range(layers)]
    base = np.concatenate(rows).astype(np.uint32)
    extra = [np.array([[5, 6, 9 + k]], np.uint32) for k in range(K)]
    inst = synth.Instance(1 + (layers + 1) * n, base, [extra[0][:0]] * K, extra)
    want = oracle.window_values(inst, oracle.BFS, 0, 0, K)
    with evq.Graph.from_instance(inst) as g, evq.tuning(launch_depth=depth):
        evq.timing_enable(True)
        evq.timing_reset()
        try:
            got, st = gpu_values(g, oracle.BFS, 0, 0, K, stats=True)
            launches = {k: n for k, (n, ms) in evq.timing_report().items()}
        finally:
            evq.timing_enable(False)
        assert_equal_values(got, want, f"layers={layers} depth={depth}")
        assert st["iters_cap"] == layers + 1  # the last layer has no edges
        assert launches["solve_expand_cap_all"] == st["iters_cap"] + (depth if steady else 1), (launches, st)
        out = evq.to_u32(g.query_noalloc(oracle.BFS, 0, 0, K)).reshape(want.shape)
        assert_equal_values(out, want, f"layers={layers} depth={depth} without allocation")
