"""The relaxation's second task buffer belongs to the kernels that list tasks
into it: with relax_staged 0, and in the one-lane layout of the sequential
evaluation, a query takes a single one.  A workspace belongs to one thread, so
each query runs on a fresh one, and the pool's bytes in use before and after it
are what its workspace takes.
"""
import ctypes
import gc
import threading

import numpy as np
import pytest

import oracle
import synth
from gpu_util import assert_equal_values, gpu_values

pytestmark = pytest.mark.gpu

USED_NOW = 7  # hipMemPoolAttrUsedMemCurrent


@pytest.fixture(scope="module")
def evq():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2502_10579_amd as m
    return m


def _pool_bytes(evq):
    pool, used = ctypes.c_void_p(), ctypes.c_uint64()
    assert evq.lib.hipDeviceGetDefaultMemPool(ctypes.byref(pool), 0) == 0
    assert evq.lib.hipMemPoolGetAttribute(pool, USED_NOW, ctypes.byref(used)) == 0
    return used.value


def test_one_task_buffer_without_teams(evq):
    import torch
    inst = synth.random_instance(20000, 120000, 8, 4000, 4000, 9, 5)
    want = oracle.window_values(inst, oracle.SSSP, 1, 0, 8)
    took, unstable = {}, {}
    with evq.Graph.from_instance(inst) as g:
        gpu_values(g, oracle.SSSP, 1, 0, 8)  # what a graph builds by its second query
        gpu_values(g, oracle.SSSP, 1, 0, 8)
        for staged in (0, 2):
            for kind in ({}, {"sequential": True}):
                def work():
                    with evq.tuning(relax_staged=staged):
                        gc.collect()  # results of earlier tests that nothing holds any more
                        torch.cuda.synchronize()
                        before = _pool_bytes(evq)
                        got, st = gpu_values(g, oracle.SSSP, 1, 0, 8, stats=True, **kind)
                        torch.cuda.synchronize()
                        took[staged, len(kind)] = _pool_bytes(evq) - before
                    unstable[staged, len(kind)] = st["n_unstable"]
                    assert_equal_values(got, want, f"staged={staged} {kind}")
                t = threading.Thread(target=work)
                t.start()
                t.join()
    assert len(unstable) == 4 and min(unstable.values()) > 1000, unstable
    buffer = 8 * unstable[2, 0]  # bytes it holds at least: 8 per vertex
    assert took[2, 0] - took[0, 0] >= buffer, (took, unstable)
    assert abs(took[2, 1] - took[0, 1]) < buffer, (took, unstable)
