"""The row-at-a-time closure's kernels on the CPU SIMT shim, against the oracle.

Every tier (thread, group, queue in both block widths, bits), the row offsets and both ways of
reading the result, with AddressSanitizer on: the tuples, every level's tuples and candidates and
the instances' offsets must be the oracle's, and rows must have gone through the tiers the graph
is made for.
"""

import os
import platform
import shutil
import subprocess

import numpy as np
import pytest

import oracle
from paper_2607_17571_amd import inputs

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SIMT = os.path.join(ROOT, "tests", "simt")
CSRC = os.path.join(ROOT, "paper_2607_17571_amd", "csrc")

pytestmark = pytest.mark.skipif(shutil.which("g++") is None or platform.machine() != "x86_64",
                                reason="needs g++ on x86-64 (the shim switches fibers in x86-64 assembly)")


@pytest.fixture(scope="module")
def harness(tmp_path_factory):
    exe = tmp_path_factory.mktemp("simt_reach") / "reach_harness"
    subprocess.run(["g++", "-std=c++20", "-O1", "-g", "-DSIMT_STACK=131072", "-fsanitize=address",
                    "-fno-omit-frame-pointer", f"-I{SIMT}", f"-I{CSRC}", f"-I{os.path.join(ROOT, 'include')}",
                    "-pthread", os.path.join(SIMT, "reach_harness.cpp"), "-o", str(exe)], check=True,
                   capture_output=True)
    return exe


def _run(harness, tmp_path, graphs, w=None, kb=4, grid=3, pool=1 << 20, slots=4096, start=0, hub=256, levels=4096):
    """Closure of one graph or a batch; returns the stop bits and the queued rows, after comparing
    everything else with the oracle (when nothing stopped it)."""
    w = w or max(1, max(int(max(s.max(), d.max())).bit_length() for s, d in graphs if len(s)))
    keys = [np.unique((np.uint64(i) << np.uint64(2 * w)) | (s.astype(np.uint64) << np.uint64(w)) | d.astype(np.uint64))
            for i, (s, d) in enumerate(graphs)]
    E = np.concatenate(keys)
    inp, out = tmp_path / "in.bin", tmp_path / "out.bin"
    with open(inp, "wb") as f:
        np.array([w, kb, len(graphs), E.size, hub, levels], dtype=np.uint64).tofile(f)
        E.tofile(f)
    r = subprocess.run([str(harness), str(inp), str(out), str(grid), "4", str(pool), str(slots), str(start)],
                       capture_output=True, text=True, timeout=900, env=dict(os.environ, ASAN_OPTIONS="detect_leaks=0"))
    assert r.returncode == 0, r.stdout + r.stderr[-3000:]
    got = np.fromfile(out, dtype=np.uint64)
    stop, used, queued = int(got[0]), int(got[1]), [int(x) for x in got[2:5]]
    if stop:
        return stop, used, queued
    refs = [oracle.tc(s, d) for s, d in graphs]
    L = int(got[5])
    lev = got[6:6 + 2 * L].reshape(L, 2)
    F = int(got[6 + 2 * L])
    pairs, flat, inst = np.split(got[7 + 2 * L:], [F, 2 * F])
    assert L == max(x.iterations for x in refs)
    want = np.zeros(L + 1, dtype=np.int64)
    for x in refs:
        want[:len(x.delta_sizes)] += np.asarray(x.delta_sizes, dtype=np.int64)
    assert lev[:, 0].tolist() == want[:L].tolist()
    assert int(lev[:, 1].sum()) == sum(x.candidates for x in refs)
    ref_pairs = np.concatenate([(x.src.astype(np.uint64) << np.uint64(32)) | x.dst for x in refs])
    np.testing.assert_array_equal(pairs, ref_pairs)
    ref_keys = np.concatenate([(np.uint64(i) << np.uint64(2 * w)) | (x.src.astype(np.uint64) << np.uint64(w))
                               | x.dst.astype(np.uint64) for i, x in enumerate(refs)])
    np.testing.assert_array_equal(flat, ref_keys)
    assert inst.tolist() == np.concatenate([[0], np.cumsum([x.src.size for x in refs])]).tolist()
    return stop, used, queued


def _star(deg):
    return np.zeros(deg, np.uint32), np.arange(1, deg + 1, dtype=np.uint32)


# sizes at the edges of the thread tier (15 edges, 16 tuples) and the group tier (128 tuples)
# and the queue tier (levels of 96 here)
@pytest.mark.parametrize("graph,group,wide", [
    (lambda: inputs.chain(17), 0, 0), (lambda: inputs.chain(18), 1, 0), (lambda: inputs.cycle(16), 0, 0),
    (lambda: inputs.cycle(17), 17, 0), (lambda: _star(15), 0, 0), (lambda: _star(16), 1, 0),
    (lambda: _star(128), 1, 0), (lambda: inputs.complete_dag(98), 82, 0), (lambda: _star(129), 1, 1), (lambda: inputs.cycle(128), 128, 0),
    (lambda: inputs.chain(130), 113, 1), (lambda: inputs.cycle(129), 129, 129),
    (lambda: (np.array([3], np.uint32), np.array([3], np.uint32)), 0, 0)])
def test_edges_of_the_tiers(harness, tmp_path, graph, group, wide):
    src, dst = graph()
    _, _, queued = _run(harness, tmp_path, [(src, dst)])
    assert queued == [group, wide, 1 if len(src) == 129 and src.max() == 0 else 0]


@pytest.mark.parametrize("kb,grid", [(4, 3), (8, 4)])
@pytest.mark.parametrize("graph", ["er", "rmat", "grid", "dense", "deep"])
def test_graphs(harness, tmp_path, kb, grid, graph):
    """Random graphs, hubs, a mesh, a dense graph whose levels outgrow the queue tier (96 ids here)
    and a chain deeper than the level table in LDS."""
    src, dst = {"er": lambda: inputs.erdos_renyi(400, 420, seed=3),
                "rmat": lambda: inputs.rmat(9, 460, *inputs.RMAT_ABCD, seed=9), "grid": lambda: inputs.grid_dag(14),
                "dense": lambda: inputs.erdos_renyi(300, 1500, seed=4), "deep": lambda: inputs.chain(400)}[graph]()
    _, _, queued = _run(harness, tmp_path, [(src, dst)], kb=kb, grid=grid)
    assert queued[0] > 0
    if graph != "er":
        assert queued[1] > 0
    if graph == "dense":
        assert queued[2] > 0


@pytest.mark.parametrize("start", [1, 2])
def test_tiers_entered_directly(harness, tmp_path, start):
    src, dst = inputs.erdos_renyi(200, 260, seed=5)
    _, _, queued = _run(harness, tmp_path, [(src, dst)], start=start)
    assert queued[0] == 0 and queued[start] > 0


def test_hubs_skip_tiers(harness, tmp_path):
    src, dst = inputs.rmat(9, 460, *inputs.RMAT_ABCD, seed=9)
    _, _, queued = _run(harness, tmp_path, [(src, dst)], hub=16)
    assert queued[2] > 0


def test_batches(harness, tmp_path):
    graphs = [inputs.erdos_renyi(60, 55, seed=1), inputs.cycle(40), (np.empty(0, np.uint32), np.empty(0, np.uint32)),
              inputs.complete_dag(24), inputs.chain(3), inputs.erdos_renyi(200, 320, seed=2)]
    empty = [i for i, (s, _) in enumerate(graphs) if not len(s)]
    assert empty == [2]
    _run(harness, tmp_path, graphs, kb=8)
    _run(harness, tmp_path, graphs, kb=4)


def test_too_small_buffers_are_reported(harness, tmp_path):
    """A pool or slots too small: the stop bits say so, and the pool's need has been counted."""
    src, dst = inputs.grid_dag(14)
    _, used, _ = _run(harness, tmp_path, [(src, dst)])
    stop, need, _ = _run(harness, tmp_path, [(src, dst)], pool=5000)
    assert stop == 1 and need == used
    src, dst = inputs.erdos_renyi(300, 1500, seed=4)
    stop, _, queued = _run(harness, tmp_path, [(src, dst)], slots=5)
    assert stop & 2 and queued[2] > 5
    stop, _, _ = _run(harness, tmp_path, [inputs.chain(400)], levels=300)
    assert stop == 8
