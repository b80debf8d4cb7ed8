"""A team takes a list only if its members do it in four rounds: of 512 edges
each in the bound solves, of 64 tasks each in a relaxation of 8 lanes.  A longer
list goes to the launches, as where other streams keep the device busy and few
members register.

The most members of a team are read once per process, so a child process with
two of them runs the queries.  What it traces says how many iterations each
launch ran; the values equal the oracle's.  Values are uint32: tolerance zero.
"""
import os
import re
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

HERE = os.path.dirname(os.path.abspath(__file__))
WIDE, THIN = 20, 20  # layers
EDGES, TASKS = 2 * 4 * 512, 2 * 4 * 64  # what a team of two takes

CHILD = """
import sys
sys.path[:0] = [{root!r}, {here!r}]
import numpy as np
import torch
import oracle
import synth
import paper_2502_10579_amd as evq
from gpu_util import gpu_values

def instance(width, K):
    # source -> 1 -> {wide} layers of `width` vertices, an edge each into the next -> a chain of {thin}; the first
    # edge has another weight in every snapshot, so every vertex behind it is unstable
    widths = [1, 1] + [width] * {wide} + [1] * {thin}
    at = np.concatenate([[0], np.cumsum(widths)])
    rows = []
    for i in range(1, len(widths) - 1):
        n, m = widths[i], widths[i + 1]
        d = np.arange(max(n, m))
        rows.append(np.stack([at[i] + d % n, at[i + 1] + d % m, np.full(len(d), 3)], 1))
    first = lambda k: np.array([[0, 1, 10 + k]], np.uint32)
    base = np.concatenate([first(0)] + rows).astype(np.uint32)
    return synth.Instance(int(at[-1]), base, [first(k) for k in range(K)], [first(k + 1) for k in range(K)])

for width in {widths}:
    inst = instance(width, 8)
    want = oracle.window_values(inst, oracle.SSSP, 0, 0, 8)
    with evq.Graph.from_instance(inst) as g:
        for tn in (dict(), dict(direct_tasks=0)):
            with evq.tuning(**tn):
                gpu_values(g, oracle.SSSP, 0, 0, 8)  # the kernels are loaded: both blocks register at once
            print("CASE", width, file=sys.stderr, flush=True)
            with evq.tuning(trace_loops=1, **tn):
                got = gpu_values(g, oracle.SSSP, 0, 0, 8)
            assert np.array_equal(got, want), (width, tn)
        got = evq.to_u32(g.query_noalloc(oracle.SSSP, 0, 0, 8)).reshape(g.num_vertices, 8)
        assert np.array_equal(got, want), (width, "noalloc")
"""


def test_lists_beyond_a_small_team_go_to_the_launches():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    widths = (TASKS, TASKS + 1, EDGES, EDGES + 1)
    code = CHILD.format(root=os.path.dirname(HERE), here=HERE, wide=WIDE, thin=THIN, widths=widths)
    r = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=100,
                       env=dict(os.environ, EVQ_TEAM_BLOCKS="2"))
    assert r.returncode == 0, r.stderr[-3000:]
    cases = re.split(r"^CASE (\d+)$", r.stderr, flags=re.M)[1:]
    assert len(cases) == 2 * 2 * len(widths)
    for width, trace in zip(map(int, cases[::2]), cases[1::2]):
        for loop, most in (("bound solve", EDGES), ("snapshot relaxation", TASKS)):
            # per launch: items processed, iterations run
            got = [(int(n), int(k)) for n, k in re.findall(loop + r" iteration \d+: (\d+) \((\d+) iterations\)", trace)]
            wide = [k for n, k in got if n == width]      # a wide layer alone
            runs = [n for n, k in got if k > 1]           # several iterations in one launch
            whole = [n for n in runs if n > WIDE * width]  # ... the wide layers among them
            what = f"{loop}, width {width}: {got}"
            if width <= most:
                assert whole and len(wide) <= 2, what
            else:
                assert not whole and len(wide) >= WIDE - 1, what
            assert any(n >= THIN - 2 for n in runs), what  # the chain behind them by a team in either case
