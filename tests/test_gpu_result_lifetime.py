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
