"""The plain evaluation runs its iterations in teams only where all of its tasks
are one round of a team; a larger graph's go to the launches, launch_depth of
them in flight.  Values equal the oracle's: tolerance zero.
"""
import pytest

import oracle
import synth
from gpu_util import assert_equal_values, gpu_values

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V,E,teams", [(256, 1500, True), (3000, 6000, True), (9000, 40000, False)])
def test_plain_evaluation(V, E, teams):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2502_10579_amd as evq
    K = 8  # 8 lanes: a round of 64 members is 4096 tasks of up to 8 edges, about one per vertex and one more per 8 edges
    inst = synth.random_instance(V, E, K, 20, 20, 9, V)
    with evq.Graph.from_instance(inst) as g:
        for a in (oracle.SSSP, oracle.SSWP):
            want = oracle.window_values(inst, a, 1, 0, K)
            evq.timing_enable(True)
            evq.timing_reset()
            try:
                got, st = gpu_values(g, a, 1, 0, K, plain=True, stats=True)
                launches = {k: n for k, (n, ms) in evq.timing_report().items()}
            finally:
                evq.timing_enable(False)
            assert_equal_values(got, want, f"V={V} algo={a}")
            assert st["iters_relax"] > 3
            if teams:
                assert launches["relax_team"] == launches["relax"] < st["iters_relax"], launches
            else:
                assert "relax_team" not in launches and launches["relax"] == st["iters_relax"] + 3, launches
