"""A served result freed while the copy out of it is still queued: its memory goes to nobody else
before the copy has read it."""

import time

import numpy as np
import pytest

import oracle
from paper_2607_17571_amd import inputs, wg
from tests.gpu_util import to_gpu

pytestmark = pytest.mark.gpu


def test_copy_queued_behind_other_work():
    import torch

    src, dst = inputs.chain(293)
    ref = oracle.tc(src, dst)
    others = [("sg", *inputs.erdos_renyi(2500, 1900, seed=s)) for s in range(6)] + \
             [("tc", *inputs.erdos_renyi(1500, 1300, seed=s)) for s in range(6)]
    with_inputs = [(q, to_gpu(s), to_gpu(d)) for q, s, d in others]
    server = wg.Server(0, slots=2)
    try:
        job = server.submit("tc", to_gpu(src), to_gpu(dst))
        time.sleep(0.2)  # (solved before the stream of the copy is busy)
        torch.cuda._sleep(50_000_000)  # some tens of milliseconds on the current stream
        s, d, _, _ = job.wait()  # copies behind that, and frees the result without waiting for it
        jobs = [server.submit(q, a, b) for q, a, b in with_inputs]
        for j in jobs:
            j.wait(want_result=False)
        np.testing.assert_array_equal(s.cpu().numpy(), ref.src)
        np.testing.assert_array_equal(d.cpu().numpy(), ref.dst)
    finally:
        server.close()


def _pool_used():
    """Bytes in use of the device's stream-ordered pool."""
    import ctypes

    hip = ctypes.CDLL("libamdhip64.so")
    pool, used = ctypes.c_void_p(), ctypes.c_uint64()
    assert hip.hipDeviceGetDefaultMemPool(ctypes.byref(pool), 0) == 0
    assert hip.hipMemPoolGetAttribute(pool, 7, ctypes.byref(used)) == 0  # hipMemPoolAttrUsedMemCurrent
    return used.value


def _until(condition, seconds=2.0):
    end = time.time() + seconds
    while not condition() and time.time() < end:
        time.sleep(0.005)
    return condition()


def test_memory_comes_back_without_another_call():
    """The last results freed with their copies queued: credited to the server when the memory is back,
    not before, and given back by an idle server and by one that is closed."""
    import torch

    src, dst = inputs.grid_dag(40)  # 672,400 - 1,600 tuples
    s, d = to_gpu(src), to_gpu(dst)
    for close in (False, True):
        server = wg.Server(0, slots=1)
        try:
            server.submit("tc", s, d).wait(want_result=False)  # (its buffers are there)
            torch.cuda.synchronize()
            assert _until(lambda: server.stats()["held_bytes"] == 0)
            before = _pool_used()
            job = server.submit("tc", s, d)
            time.sleep(0.2)
            torch.cuda._sleep(100_000_000)
            job.wait()
            assert server.stats()["held_bytes"] > 4 * 600_000  # (the copy has not run)
            torch.cuda.synchronize()
            if close:
                server.close()
            assert _until(lambda: _pool_used() <= before)
            if not close:
                assert server.stats()["held_bytes"] == 0
        finally:
            server.close()


def test_request_gets_the_memory_of_freed_results():
    """A request that fits only once results freed with their copies queued are back waits for them."""
    import torch

    s, d = map(to_gpu, inputs.rmat(14, 13_000, *inputs.RMAT_ABCD, seed=2))
    server = wg.Server(0, slots=2, mem_budget_bytes=2 << 30)
    try:
        held = []
        for _ in range(200):  # results until one more solve does not fit beside them
            job = server.submit("tc", s, d)
            assert _until(job.done, 20)
            if job.info()["status"] != wg.WG_OK:
                break
            held.append(job)
        assert job.info()["status"] == wg.WG_ERR_CAPACITY
        torch.cuda._sleep(100_000_000)
        sizes = [j.wait()[2]["result_tuples"] for j in held]
        again = [server.submit("tc", s, d) for _ in range(3)]
        assert [j.wait()[2]["result_tuples"] for j in again] == sizes[:3]
    finally:
        server.close()
