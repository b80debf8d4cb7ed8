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
