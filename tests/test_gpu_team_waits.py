"""A wait among the blocks that run small iterations together is bounded, and a
call in which one runs out fails instead of answering from half-written lists.

The bound is read once per process, so a child process with a bound of no polls
at all runs the queries: every member but the first leaves at once, the first
gives up at its first barrier, and each kernel ends normally.  The same calls
with the small iterations left to the launches, in the same process and on the
same workspaces, equal the oracle.  Values are uint32: tolerance zero.
"""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

HERE = os.path.dirname(os.path.abspath(__file__))

CHILD = """
import sys
sys.path[:0] = [{root!r}, {here!r}]
import numpy as np
import torch
import oracle
import paper_2502_10579_amd as evq
from gpu_util import gpu_values
from test_gpu_teams import layered_instance

NO_TEAMS = dict(append_edges=0, relax_staged=0)
inst = layered_instance([1, 3, 64, 70, 513, 40, 1, 1, 900, 5, 1], 3, 6, 40, 7)
rep = oracle.replay(inst)
with evq.Graph.from_instance(inst) as g:
    def noalloc(a, b, L):
        return evq.to_u32(g.query_noalloc(a, 0, b, L)).reshape(g.num_vertices, L)
    calls = dict(query=lambda a, b, L: gpu_values(g, a, 0, b, L), noalloc=noalloc,
                 bounds=lambda a, b, L: g.query_bounds(a, 0, b, L))
    for a in (0, 2, 4):
        for b, L in ((0, 6), (1, 4)):
            want = oracle.window_values(inst, a, 0, b, L, replayed=rep)
            # append_edges 0: the bound solves have no team, so the relaxation's is the first
            for tn in ({{}}, dict(append_edges=0)):
                for name, call in calls.items():
                    if tn and name == "bounds":
                        continue
                    with evq.tuning(**tn):
                        try:
                            call(a, b, L)
                            print("ANSWERED", name, a, b, L, tn, flush=True)
                        except evq.EvqError as e:
                            ok = e.status == evq.EVQ_EDEVICE and "gave up" in str(e)
                            ok = ok and ("snapshot relaxation" if tn else "bound solve") in str(e)
                            print("FAILED" if ok else "OTHER %s" % e, flush=True)
            with evq.tuning(**NO_TEAMS):
                for name in ("query", "noalloc"):
                    got = calls[name](a, b, L)
                    print("EQUAL" if np.array_equal(got, want) else "WRONG %s %d %d %d" % (name, a, b, L), flush=True)
"""


def test_a_team_that_gives_up_fails_the_call():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    r = subprocess.run([sys.executable, "-c", CHILD.format(root=os.path.dirname(HERE), here=HERE)],
                       capture_output=True, text=True, timeout=100, env=dict(os.environ, EVQ_TEAM_SPINS="0"))
    assert r.returncode == 0, r.stderr[-3000:]
    lines = [l for l in r.stdout.splitlines() if l.split(" ")[0] in ("ANSWERED", "FAILED", "OTHER", "EQUAL", "WRONG")]
    assert lines == (["FAILED"] * 5 + ["EQUAL"] * 2) * 6, r.stdout[-3000:]
