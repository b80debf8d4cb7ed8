"""A workspace that one thread's queries share serves graphs of growing sizes:
the part of a buffer that a smaller graph never used is unset memory.

A larger graph whose buffers still fit (they are allocated with slack) must
not read stray flags or stamps from it, also past its last vertex when the
vertices are no multiple of 8.  Each size is queried on a fresh thread (its
workspace is new) after device memory full of ones went back to the pool,
against the oracle.  Values are uint32: tolerance zero.
"""
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


@pytest.mark.parametrize("sizes", [(70, 90), (9, 1001), (64, 72, 73), (90, 70, 91)])
def test_growing_graphs_on_one_workspace(evq, sizes):
    # graphs built and freed first leave their edges (no zeros) in the pool that workspaces come from
    big = synth.random_instance(3000, 60000, 8, 50, 50, 9, 3)
    for _ in range(3):
        evq.Graph.from_instance(big).close()
    wrong = []

    def work():
        try:
            for i, V in enumerate(sizes):
                inst = synth.random_instance(V, 10 * V, 8, 6, 6, 9, 40 + i)
                with evq.Graph.from_instance(inst) as g:
                    for a in (oracle.SSSP, oracle.SSWP):
                        for b, L in ((0, 8), (2, 5)):
                            want = oracle.window_values(inst, a, 1, b, L)
                            assert_equal_values(gpu_values(g, a, 1, b, L), want, f"V={V} algo={a} window {(b, L)}")
        except BaseException as e:  # carried to the test's thread
            wrong.append(e)

    t = threading.Thread(target=work)
    t.start()
    t.join()
    if wrong:
        raise wrong[0]
