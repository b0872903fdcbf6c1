"""The forms on the renumbered graph at the edges of their rules, through the C ABI, against the
oracle: same-generation as matrices and as pairs, triangles beyond 65,536 columns, closures as slabs
and by tiers, ids by rank.  Every form leaves to the iterations' launches what it does not take, with
the same result, so each test says which of them it is for (stage_bytes are the iterations' alone)."""

import time

import numpy as np
import pytest

import oracle
from paper_2607_17571_amd import inputs, wg
from tests.gpu_util import assert_same, run, to_gpu

pytestmark = pytest.mark.gpu

SG = {
    "matrices": lambda: inputs.rmat(12, 3600, *inputs.RMAT_ABCD, seed=12),
    "matrices_by_degree": lambda: [np.concatenate(p) for p in zip(inputs.erdos_renyi(9_000, 5_000, seed=9), inputs.out_star(100))],
    "pairs": lambda: inputs.erdos_renyi(60_000, 48_000, seed=5),
    "pairs_table_grown": lambda: inputs.binary_tree(9),
    "pairs_wide": lambda: inputs.scatter_ids(*inputs.erdos_renyi(5_000, 4_500, seed=6), 23, seed=1),
    "grid": lambda: inputs.grid_dag(30),
}


@pytest.fixture(scope="module")
def engine():
    return wg.Engine(0)


def by_forms(st):
    return sum(st["stage_bytes"].values()) == 0


def sg_form(src, dst):
    """The form of same-generation a graph takes, by the rule of the sizes."""
    edges = np.unique((src.astype(np.uint64) << np.uint64(32)) | dst)
    deg = np.unique(edges >> np.uint64(32), return_counts=True)[1].astype(np.int64)
    cols, base, wide = np.unique(dst).size, int((deg * (deg - 1)).sum()), bool(deg.max() > 64)
    if cols <= 18_431 and deg.size + cols + 2 <= 36_864 and (base * 256 >= cols * cols or wide):
        return "matrices"
    return "" if wide else "pairs"


@pytest.mark.parametrize("irreflexive", [False, True])
@pytest.mark.parametrize("graph", sorted(SG))
def test_same_generation(engine, graph, irreflexive):
    src, dst = SG[graph]()
    form = {"grid": "pairs"}.get(graph, graph.split("_")[0])
    assert sg_form(src, dst) == form
    opts = wg.make_options(flags=wg.WG_SG_IRREFLEXIVE if irreflexive else 0)
    ref = oracle.sg(src, dst, irreflexive=irreflexive)
    s, d, st = run(engine, "sg", src, dst, opts)
    assert_same(s, d, st, ref)
    assert by_forms(st)
    if graph == "pairs_table_grown":  # (more pairs than the first table's list holds)
        base = 2 * np.unique(src).size
        assert ref.src.size / 2 > max(1024, 1 << (8 * base - 1).bit_length()) / 2


WIDE = {  # ids over 32 bits: by rank
    "tc_slabs": ("tc", lambda: inputs.rmat(12, 3_600, *inputs.RMAT_ABCD, seed=12)),
    "tc_tiers": ("tc", lambda: inputs.erdos_renyi(60_000, 50_000, seed=5)),
    "sg_pairs": ("sg", lambda: inputs.erdos_renyi(20_000, 16_000, seed=6)),
    "sg_pairs_wide_keys": ("sg", lambda: inputs.erdos_renyi(90_000, 70_000, seed=7)),
    "sg_matrices": ("sg", lambda: inputs.rmat(11, 1_800, *inputs.RMAT_ABCD, seed=12)),
    "few_rows": ("tc", lambda: inputs.complete_dag(60)),
}


@pytest.mark.parametrize("bits", [25, 32])
@pytest.mark.parametrize("graph", sorted(WIDE))
def test_ids_by_rank(engine, graph, bits):
    query, make = WIDE[graph]
    src, dst = inputs.scatter_ids(*make(), bits, seed=bits)
    if bits == 32:  # the largest id there is
        top = np.uint32(0xFFFFFFFF)
        src, dst = np.where(src == src.max(), top, src), np.where(dst == src.max(), top, dst)
    s, d, st = run(engine, query, src, dst)
    assert_same(s, d, st, getattr(oracle, query)(src, dst))
    assert st["key_bytes"] == 8 and by_forms(st) == (graph != "few_rows")
    if query == "sg":
        assert sg_form(src, dst) == graph.split("_")[1]
    elif graph != "few_rows":
        assert (st["resumes"] > 0) == (graph == "tc_tiers")  # (tiers that rows outgrew)


@pytest.mark.parametrize("digit_bits", [0, 10])
def test_sort_configuration_reported_by_rank(engine, digit_bits):
    """The digits reported are those of the ids' own keys, as the iterations (batch_k) report them."""
    src, dst = inputs.scatter_ids(*inputs.rmat(11, 1_800, *inputs.RMAT_ABCD, seed=12), 28, seed=3)
    st, ref = (run(engine, "tc", src, dst, wg.make_options(radix_digit_bits=digit_bits, batch_k=k))[2] for k in (0, 2))
    for key in ("field_bits", "key_bytes", "digit_bits", "sort_passes"):
        assert st[key] == ref[key], key


@pytest.mark.parametrize("count,length", [(700, 200), (2_700, 100), (40, 3_400)])
def test_thin_rows_of_wide_graphs(engine, count, length):
    """Chains side by side, more than 131,072 columns in all: rows up to 64 levels deep, deeper, and past
    the levels counted in LDS."""
    v = np.arange(count * length, dtype=np.uint32).reshape(count, length)
    order = np.random.default_rng(7).permutation(count * (length - 1))
    src, dst = v[:, :-1].ravel()[order], v[:, 1:].ravel()[order]
    s, d, st = run(engine, "tc", src, dst)
    i, j = np.triu_indices(length, 1)
    np.testing.assert_array_equal(s, v[:, i].ravel())
    np.testing.assert_array_equal(d, v[:, j].ravel())
    sizes = [count * (length - 1 - k) for k in range(length)]
    assert st["iterations"] == length - 1 and st["delta_sizes"] == sizes
    assert st["join_candidates"] == sum(sizes[1:]) and by_forms(st)


@pytest.mark.parametrize("depth", [16, 17, 18])
def test_wide_levels_of_wide_graphs(engine, depth):
    """Binary trees, rows of some hundred thousand tuples among many short ones: three bitmaps in LDS, the
    widest graph of those (262,142 columns), and levels too wide for the tiers of a wider one, which is
    left to the iterations when the others have run."""
    src, dst = inputs.binary_tree(depth)
    s, d, st = run(engine, "tc", src, dst)
    assert_same(s, d, st, oracle.tc(src, dst))
    assert by_forms(st) == (depth < 18)


@pytest.mark.parametrize("rows,leaves", [(200, 4_000), (20_000, 20)])
def test_fans_take_the_tiers(engine, rows, leaves):
    """Rows that outgrow the thread tier and lead nowhere: as slabs, a pass over all edges for every 32
    leaves, they took 32 and 21 ms."""
    src = np.repeat(np.arange(rows, dtype=np.uint32), leaves)
    dst = np.arange(rows, rows * (leaves + 1), dtype=np.uint32)
    s, d = to_gpu(src), to_gpu(dst)
    ms = []
    for _ in range(4):
        t = time.perf_counter()
        out_s, out_d, st = engine.solve("tc", s, d)
        ms.append((time.perf_counter() - t) * 1e3)
    np.testing.assert_array_equal(out_s.cpu().numpy(), src)
    np.testing.assert_array_equal(out_d.cpu().numpy(), dst)
    assert (st["iterations"], st["delta_sizes"], st["join_candidates"]) == (1, [rows * leaves, 0], 0)
    assert min(ms) < 5


def _fan(rows, leaves, first=0):
    ids = np.arange(first, first + rows * (leaves + 1), dtype=np.uint32)
    return np.repeat(ids[:rows], leaves), ids[rows:]


def _offset(graph, by=200):
    return tuple(x + np.uint32(by) for x in graph)


# (a sample of 2,048 edges that holds them all, or a part of them)
FEW_ROWS = {
    "one": ("tc", lambda: _fan(1, 200), False), "fans_111": ("tc", lambda: _fan(111, 10), False),
    "fans_127": ("tc", lambda: _fan(127, 10), False), "fans_128": ("tc", lambda: _fan(128, 10), True),
    "dense": ("tc", lambda: _offset(inputs.erdos_renyi(120, 3_000, seed=2)), False),
    "chain": ("tc", lambda: _offset(inputs.chain(129)), True),
    "fat_127": ("tc", lambda: _fan(127, 400), False), "fat_128": ("tc", lambda: _fan(128, 400), True),
    "fat_one": ("tc", lambda: _fan(1, 60_000), False),
    "fat_few_often": ("tc", lambda: [np.concatenate(p) for p in zip(_fan(20, 20_000), _fan(108, 2, first=500_000))], True),
    "sg_one": ("sg", lambda: _fan(1, 200), True), "sg_fans": ("sg", lambda: _fan(100, 30), True),
    "sg_dense": ("sg", lambda: _offset(inputs.erdos_renyi(120, 3_000, seed=2)), True),
}


@pytest.mark.parametrize("graph", sorted(FEW_ROWS))
def test_few_rows(engine, graph):
    """Closures of fewer than 128 rows are the iterations', however few of them the sample sees; SG's are not."""
    query, make, forms = FEW_ROWS[graph]
    src, dst = make()
    s, d, st = run(engine, query, src, dst)
    assert_same(s, d, st, getattr(oracle, query)(src, dst))
    assert by_forms(st) == forms


@pytest.mark.parametrize("rows,leaves,forms", [(20, 10, False), (20, 50, False), (31, 50, False), (32, 50, True)])
def test_few_rows_of_a_batch(engine, rows, leaves, forms):
    import torch

    src, dst = _fan(rows, leaves)
    n = src.size
    s, d, offs, st = engine.solve_batch("tc", to_gpu(np.tile(src, 4)), to_gpu(np.tile(dst, 4)),
                                        torch.arange(0, 5 * n, n, dtype=torch.int64, device="cuda"))
    np.testing.assert_array_equal(s.cpu().numpy(), np.tile(src, 4))
    np.testing.assert_array_equal(d.cpu().numpy(), np.tile(dst, 4))
    assert offs.tolist() == list(range(0, 5 * n, n)) and st["iterations"] == 1
    assert by_forms(st) == forms


DEEP = {
    "tc_slabs": ("tc", lambda: inputs.chain(30_000)),
    "tc_tiers": ("tc", lambda: inputs.chain(60_000)),
    "sg_pairs": ("sg", lambda: _two_chains(4_000)),
}


def _tree(n, children):
    v = np.arange(1, n, dtype=np.uint32)
    return (v - 1) // np.uint32(children), v


@pytest.mark.parametrize("n,children,forms", [(3_000, 8, True), (3_000, 2, True), (19_000, 8, False), (19_000, 2, False)])
def test_pairs_that_grow(engine, n, children, forms):
    """Pairs that multiply from round to round: matrices where the columns allow, else the iterations."""
    import torch

    s, d = map(to_gpu, _tree(n, children))
    a_s, a_d, a = engine.solve("sg", s, d)
    b_s, b_d, b = engine.solve("sg", s, d, wg.make_options(batch_k=2))
    assert by_forms(a) == forms and sg_form(*_tree(n, children)) == "pairs"
    assert torch.equal(a_s.view(torch.int32), b_s.view(torch.int32)) and torch.equal(a_d.view(torch.int32), b_d.view(torch.int32))
    for key in ("iterations", "delta_sizes", "join_candidates"):
        assert a[key] == b[key], key


@pytest.mark.parametrize("n,hub", [(4_095, 0), (4_096, 0), (9_000, 0), (4_400, 70)])
def test_same_generation_of_many_rounds(n, hub):
    """More rounds than are allotted at first, as pairs and (beside a vertex of 70 out-edges) as
    matrices: grown, and not left to the iterations."""
    src, dst = _two_chains(n)
    pairs = 2 * n
    if hub:
        leaf = np.arange(30_000, 30_000 + hub, dtype=np.uint32)
        src, dst = np.append(src, np.full(hub, 29_999, np.uint32)), np.append(dst, leaf)
        pairs += hub * (hub - 1)
    eng = wg.Engine(0)
    try:
        for _ in range(2):
            s, d, st = run(eng, "sg", src, dst)
            assert (st["iterations"], st["result_tuples"]) == (n, pairs) and by_forms(st)
            assert st["delta_sizes"] == [pairs - 2 * (n - 1)] + [2] * (n - 1) + [0]
            assert st["join_candidates"] == 2 * (n - 1)
            keep = s < 29_000
            np.testing.assert_array_equal(s[keep], np.arange(2 * n))
            np.testing.assert_array_equal(d[keep], np.roll(np.arange(2 * n), n))
    finally:
        eng.close()


def _two_chains(n):
    """One root over two chains of n vertices: n rounds of one pair each."""
    s = np.arange(2 * n, dtype=np.uint32)
    s, d = np.delete(s, [n - 1, 2 * n - 1]), np.delete(s, [0, n])
    return np.append(s, np.uint32([2 * n, 2 * n])), np.append(d, np.uint32([0, n]))


@pytest.mark.parametrize("graph", sorted(DEEP))
def test_iteration_limit_bounds_the_work(engine, graph):
    """A limit far below the fixpoint's depth ends the solve after that many iterations, not at the
    fixpoint (the closures: 4.5e8 and 1.8e9 tuples, half a second and more)."""
    query, make = DEEP[graph]
    s, d = map(to_gpu, make())
    opts = wg.make_options(max_iterations=12)
    times = []
    for _ in range(3):
        t = time.perf_counter()
        with pytest.raises(wg.WgError) as ei:
            engine.solve(query, s, d, opts)
        times.append(time.perf_counter() - t)
        assert ei.value.status == wg.WG_ERR_ITER_LIMIT
    assert min(times) < 0.015


@pytest.mark.parametrize("limit", [0, 1, 2])
@pytest.mark.parametrize("graph", sorted(SG))
def test_iteration_limit_at_the_fixpoint(engine, graph, limit):
    """The last iteration that is enough, and one fewer."""
    src, dst = SG[graph]()
    ref = oracle.sg(src, dst)
    if limit == 2:
        assert_same(*run(engine, "sg", src, dst, wg.make_options(max_iterations=2**64 - 1)), ref)
    elif limit == 1:
        assert_same(*run(engine, "sg", src, dst, wg.make_options(max_iterations=ref.iterations)), ref)
    elif ref.iterations > 1:
        with pytest.raises(wg.WgError) as ei:
            run(engine, "sg", src, dst, wg.make_options(max_iterations=ref.iterations - 1))
        assert ei.value.status == wg.WG_ERR_ITER_LIMIT


@pytest.mark.parametrize("scale,m", [(12, 40_000), (15, 100_000), (17, 60_000)])
def test_triangles(engine, scale, m):
    src, dst = inputs.rmat(scale, m, *inputs.RMAT_ABCD, seed=scale)
    src, dst = np.concatenate([src, src[:64]]), np.concatenate([dst, src[:64]])  # self-loops
    if scale == 17:  # a column for every vertex
        ids = np.arange(1 << scale, dtype=np.uint32)
        src, dst = np.concatenate([src, ids[:-1]]), np.concatenate([dst, ids[1:]])
    count, st = engine.triangles(to_gpu(src), to_gpu(dst))
    assert (count, st["join_candidates"]) == oracle.triangles(src, dst)
    assert by_forms(st)


@pytest.mark.parametrize("make", [
    lambda: inputs.grid_dag(150), lambda: inputs.erdos_renyi(200_000, 160_000, seed=5),
    lambda: inputs.erdos_renyi(600_000, 480_000, seed=4), lambda: inputs.erdos_renyi(700_000, 630_000, seed=4)],
    ids=["slabs_of_16", "queue_4_waves", "queue_16_waves", "thin_and_queue"])
def test_large_closures_equal_the_iterations(engine, make):
    """Routes whose graphs are too large for the oracle, against the iterations' launches."""
    import torch

    s, d = map(to_gpu, make())
    a_s, a_d, a = engine.solve("tc", s, d)
    b_s, b_d, b = engine.solve("tc", s, d, wg.make_options(batch_k=2))
    assert by_forms(a) and not by_forms(b)
    assert torch.equal(a_s.view(torch.int32), b_s.view(torch.int32)) and torch.equal(a_d.view(torch.int32), b_d.view(torch.int32))
    for key in ("iterations", "delta_sizes", "join_candidates"):
        assert a[key] == b[key], key
