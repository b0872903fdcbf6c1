"""A memory budget that the iterations' launches alone fit is enough for the default options too, whatever
the forms on the renumbered graph held before they declined or keep from an earlier solve."""

import numpy as np
import pytest

import oracle
from paper_2607_17571_amd import inputs, wg
from tests.gpu_util import assert_same, run

pytestmark = pytest.mark.gpu


class _PeakAllocator(wg.TorchAllocator):
    """Torch's allocator with the bytes the engine holds, now and at most."""

    held = peak = 0

    def _on_alloc(self, nbytes, stream, user):
        self.held += nbytes
        self.peak = max(self.peak, self.held)
        return super()._on_alloc(nbytes, stream, user)

    def _on_free(self, ptr, nbytes, stream, user):
        self.held -= nbytes
        return super()._on_free(ptr, nbytes, stream, user)


def _iterations_peak(query, src, dst):
    hook = _PeakAllocator(0)
    eng = wg.Engine(0, allocator=hook)
    try:
        run(eng, query, src, dst, wg.make_options(batch_k=2))
    finally:
        eng.close()
    return hook.peak


def _wide_ids(src, dst, top):
    """... with an edge between the largest ids there are."""
    return np.append(src, np.uint32(top - 1)), np.append(dst, np.uint32(top))


def _hub(n, deg):
    """A random graph and a vertex of `deg` out-edges, which SG's pair form does not take."""
    src, dst = inputs.erdos_renyi(n, int(0.8 * n), seed=3)
    return np.concatenate([src, np.zeros(deg, np.uint32)]), np.concatenate([dst, np.arange(n, n + deg, dtype=np.uint32)])


def _deep_star(rows, leaves):
    """A chain of few rows, the last of which has many leaves."""
    chain = np.arange(rows - 1, dtype=np.uint32)
    return (np.concatenate([chain, np.full(leaves, rows - 1, np.uint32)]),
            np.concatenate([chain + np.uint32(1), np.arange(rows, rows + leaves, dtype=np.uint32)]))


# (the iterations' buffers grow in each)
DECLINED = {
    "sg_hub": ("sg", lambda: _hub(40_000, 2_000)),
    "sg_hub_span": ("sg", lambda: _wide_ids(*_hub(40_000, 2_000), (1 << 24) - 1)),
    "sg_hub_by_rank": ("sg", lambda: _wide_ids(*_hub(40_000, 2_000), (1 << 28) - 1)),
    "tc_few_rows_span": ("tc", lambda: _wide_ids(*_deep_star(100, 20_000), (1 << 24) - 1)),
}


@pytest.mark.parametrize("graph", sorted(DECLINED))
def test_forms_that_decline(graph):
    query, make = DECLINED[graph]
    src, dst = make()
    opts = wg.make_options(mem_budget_bytes=_iterations_peak(query, src, dst))
    eng = wg.Engine(0)
    try:
        for _ in range(2):
            s, d, st = run(eng, query, src, dst, opts)
            assert_same(s, d, st, getattr(oracle, query)(src, dst))
    finally:
        eng.close()


@pytest.mark.parametrize("options", [{}, {"batch_k": 2}])
def test_buffers_of_an_earlier_solve(options):
    """What a closure on the renumbered graph left in the engine makes room for the next solve's
    launches: here iterations that need nearly all of the budget."""
    first = inputs.erdos_renyi(8_000, 6_500, seed=5)
    src, dst = inputs.rmat(13, 7_000, *inputs.RMAT_ABCD, seed=2)
    peak = _iterations_peak("tc", src, dst)
    eng = wg.Engine(0)
    try:
        run(eng, "tc", *first)
        opts = wg.make_options(mem_budget_bytes=peak, **options)
        s, d, st = run(eng, "tc", src, dst, opts)
        assert_same(s, d, st, oracle.tc(src, dst))
    finally:
        eng.close()
