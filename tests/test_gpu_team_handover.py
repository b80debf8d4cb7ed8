"""Lists passed between a team and the launches, at the team's limits: 32768 edges
in a bound solve, and one round of 64 members in the relaxation (4096 tasks at 8
lanes, 512 at 64 and 128).  Layers of exactly the limit and of one more; what the
loops trace says who ran which.  Also a no-allocation query whose scratch holds
one task list only, and queries from several threads at once.

Values equal the oracle's.  They are uint32: tolerance zero.
"""
import re
import threading

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


def layers(widths, degree, K, extra=None):
    """Layers of the given widths, degree[i] distinct edges of weight 3 from each vertex of layer i into the next, and
    one more from the first vertex of the layers in `extra`.  The source's edge to vertex 1 has another weight in each
    snapshot and a heavy one in all of them: every vertex behind it is reached and unstable."""
    at = np.concatenate([[0], np.cumsum(widths)])
    rows = [np.array([[0, 1, 900]])]
    for i in range(1, len(widths) - 1):
        n, m, d = widths[i], widths[i + 1], degree[i]
        src, j = np.repeat(np.arange(n), d), np.tile(np.arange(d), n)
        rows.append(np.stack([at[i] + src, at[i + 1] + (src * d + j) % m, np.full(n * d, 3)], 1))
        if extra and i in extra:
            rows.append(np.array([[at[i], at[i + 1] + d % m, 4]]))
    first = lambda k: np.array([[0, 1, 10 + k]], np.uint32)
    base = np.concatenate([first(0)] + rows).astype(np.uint32)
    assert len(np.unique(base, axis=0)) == len(base)
    return synth.Instance(int(at[-1]), base, [first(k) for k in range(K)], [first(k + 1) for k in range(K)])


def words(trace, loop):
    """Per launch of each of the loops: (items, iterations)."""
    out = []
    for i, n, k in re.findall(loop + r" iteration (\d+): (\d+) \((\d+) iterations\)", trace):
        if i == "0":
            out.append([])
        out[-1].append((int(n), int(k)))
    return out


def test_bound_solve_limit(evq, capfd):
    # 4096 x 8 edges are the limit, one more goes to the launches
    widths, degree = [1, 1, 64, 4096, 4096, 4096, 4096, 64, 1, 1, 1], [1, 64, 64, 8, 8, 8, 8, 1, 1, 1]
    inst = layers(widths, degree, 8, extra={5})
    for a in (oracle.SSSP, oracle.SSNP):
        want = oracle.window_values(inst, a, 0, 0, 8)
        with evq.Graph.from_instance(inst) as g:
            gpu_values(g, a, 0, 0, 8)  # the kernels are loaded: all of a team's blocks register at once
            capfd.readouterr()
            with evq.tuning(trace_loops=1):
                got = gpu_values(g, a, 0, 0, 8)
            trace = capfd.readouterr().err
        assert_equal_values(got, want, f"algo={a}")
        loops = words(trace, "bound solve")
        assert len(loops) == 2, trace
        for w in loops:
            at = w.index((4096, 1))  # the layer of 32769 edges alone
            before, after = w[:at], w[at + 1:]
            assert before[-1][1] > 1 and before[-1][0] >= 64 + 2 * 4096, w
            assert after[0][1] > 1 and after[0][0] >= 4096 + 64, w


@pytest.mark.parametrize("L,M", [(8, 4096), (64, 512), (100, 512)])
@pytest.mark.parametrize("direct", [0, 1 << 18])
def test_relaxation_limit(evq, capfd, L, M, direct):
    widths = [1, 1] + [M // 2] * 3 + [M + 1] * 2 + [M] * 2 + [M + 1] + [1] * 10
    degree = [1, M // 2, 1, 1, 3, 1, 1, 1, 2] + [1] * 10  # the whole next layer is reached
    inst = layers(widths, degree, L)
    want = oracle.window_values(inst, oracle.SSSP, 0, 0, L)
    with evq.Graph.from_instance(inst) as g:
        for staged in (2, 4):
            with evq.tuning(direct_tasks=direct, relax_staged=staged):
                gpu_values(g, oracle.SSSP, 0, 0, L)  # the kernels are loaded
            capfd.readouterr()
            with evq.tuning(trace_loops=1, direct_tasks=direct, relax_staged=staged):
                got = gpu_values(g, oracle.SSSP, 0, 0, L)
            trace = capfd.readouterr().err
            assert_equal_values(got, want, f"L={L} direct={direct} staged={staged}")
            (w,) = words(trace, "snapshot relaxation")
            assert w.count((M + 1, 1)) == 3, w  # one more task than the limit: the launches
            at = w.index((M + 1, 1))
            assert w[at - 1][1] > 1 and w[at - 1][0] >= 3 * (M // 2), w  # a team before them,
            assert (2 * M, 2) in w[at + 2:], w                            # one for the two layers at the limit,
            assert w[-1][1] > 1 or w[-2][1] > 1, w                        # and one for the chain behind


def test_noalloc_with_room_for_one_task_list(evq, capfd):
    V, K = 100000, 8
    rng = np.random.default_rng(5)
    first = lambda k: np.array([[0, 1, 10 + k]], np.uint32)
    seen = set()
    with_teams = lambda w: any(k > 1 for n, k in w)
    for E in (6400000, 7100000):
        rest = np.stack([rng.integers(1, V, E), rng.integers(1, V, E), rng.integers(1, 100, E)], 1).astype(np.uint32)
        inst = synth.Instance(V, np.concatenate([first(0), np.array([[0, 1, 900]], np.uint32), rest]),
                              [first(k) for k in range(K)], [first(k + 1) for k in range(K)])
        with evq.Graph.from_instance(inst) as g:
            want = oracle.window_values(inst, oracle.SSSP, 0, 0, K)
            for tn in (dict(), dict(append_edges=0)):
                capfd.readouterr()
                with evq.tuning(trace_loops=1, **tn):
                    got = evq.to_u32(g.query_noalloc(oracle.SSSP, 0, 0, K)).reshape(V, K)
                (w,) = words(capfd.readouterr().err, "snapshot relaxation")
                assert_equal_values(got, want, f"E={E} {tn}")
                seen.add((E, with_teams(w)))
    assert seen == {(6400000, True), (7100000, False)}, seen


def test_teams_on_several_streams(evq):
    import torch
    small = layers([1, 1, 64, 700, 3000, 64, 1, 1, 1, 1, 1, 1], [1, 64, 20, 9, 1, 1, 1, 1, 1, 1, 1], 8)
    odd = synth.random_instance(9001, 60000, 8, 300, 300, 9, 11)
    jobs = []
    graphs = [evq.Graph.from_instance(i) for i in (small, odd)]
    for g, inst in zip(graphs, (small, odd)):
        for a in (oracle.SSSP, oracle.SSWP):
            for b, L in ((0, 8), (2, 5)):
                jobs.append((g, a, b, L, oracle.window_values(inst, a, 0, b, L)))
    wrong = []

    def work(i):
        try:
            s = torch.cuda.Stream()
            for k in range(12):
                g, a, b, L, want = jobs[(i + k) % len(jobs)]
                out = torch.empty((g.num_vertices, L), dtype=torch.int32, device="cuda")
                g.query(a, 0, b, L, out=out, stream=s.cuda_stream)
                s.synchronize()
                assert_equal_values(evq.to_u32(out).reshape(want.shape), want, f"thread {i} query {k}")
        except BaseException as e:  # carried to the test's thread
            wrong.append(e)

    torch.cuda.synchronize()
    threads = [threading.Thread(target=work, args=(i,)) for i in range(6)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for g in graphs:
        g.close()
    if wrong:
        raise wrong[0]
