"""Same-generation on the renumbered graph: the kernels of both forms (pairs in a hash set, by rounds
and with the one-workgroup tail; bit matrices) on the CPU SIMT shim with AddressSanitizer, against
the oracle -- every tuple, every round's tuples and the candidates."""

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
ROUNDS, TAIL, MATRICES = 0, 1, 2


@pytest.fixture(scope="module")
def harness(tmp_path_factory):
    exe = tmp_path_factory.mktemp("simt_sg") / "sg_harness"
    subprocess.run(["g++", "-std=c++20", "-O1", "-g", "-DSIMT_STACK=131072", "-fsanitize=address,alignment",
                    "-fno-sanitize-recover=alignment",
                    "-fno-omit-frame-pointer", f"-I{SIMT}", f"-I{CSRC}", f"-I{os.path.join(ROOT, 'include')}",
                    "-pthread", os.path.join(SIMT, "sg_harness.cpp"), "-o", str(exe)], check=True,
                   capture_output=True)
    return exe


def _run(harness, tmp_path, graphs, form, w=None, kb=4, grid=3, slots=1 << 14, diagonal=True, levels=512):
    w = w or max(1, max(int(max(s.max(), d.max())).bit_length() for s, d in graphs if len(s)))
    keys = [np.unique((np.uint64(i) << np.uint64(2 * w)) | (s.astype(np.uint64) << np.uint64(w)) | d.astype(np.uint64))
            for i, (s, d) in enumerate(graphs)]
    E = np.concatenate(keys)
    span = ((len(graphs) << w) + 31) & ~31
    inp, out = tmp_path / "in.bin", tmp_path / "out.bin"
    with open(inp, "wb") as f:
        np.array([w, kb, len(graphs), E.size, levels, span], dtype=np.uint64).tofile(f)
        E.tofile(f)
    r = subprocess.run([str(harness), str(inp), str(out), str(grid), "4", str(form), str(slots), str(int(diagonal))],
                       capture_output=True, text=True, timeout=900, env=dict(os.environ, ASAN_OPTIONS="detect_leaks=0"))
    assert r.returncode == 0, (r.returncode, r.stdout + r.stderr[-3000:])
    got = np.fromfile(out, dtype=np.uint64)
    stop = int(got[0])
    if stop:
        return stop
    refs = [oracle.sg(s, d) for s, d in graphs]
    deg = np.concatenate([np.bincount(np.unique(k >> np.uint64(w), return_inverse=True)[1]) for k in keys if k.size])
    assert int(got[1]) == int((deg * (deg - 1)).sum()) and int(got[2]) == int(deg.max() > 64)
    R = int(got[3])
    lev = got[4:4 + 2 * (R + 1)].reshape(R + 1, 2)
    assert R == max(x.iterations for x in refs)
    want = np.zeros(R + 1, dtype=np.int64)
    for x in refs:
        want[:len(x.delta_sizes)] += np.asarray(x.delta_sizes, dtype=np.int64)
    assert lev[:, 0].tolist() == want.tolist()
    assert int(lev[1:, 1].sum()) == sum(x.candidates for x in refs)
    fin = refs if diagonal else [oracle.sg(s, d, irreflexive=True) for s, d in graphs]
    ref = np.concatenate([(np.uint64(i) << np.uint64(2 * w)) | (x.src.astype(np.uint64) << np.uint64(w))
                          | x.dst.astype(np.uint64) for i, x in enumerate(fin)])
    assert int(got[4 + 2 * (R + 1)]) == ref.size
    np.testing.assert_array_equal(got[5 + 2 * (R + 1):], ref)
    return 0


GRAPHS = {"er": lambda: inputs.erdos_renyi(200, 210, seed=3), "tree": lambda: inputs.binary_tree(5),
          "rmat": lambda: inputs.rmat(7, 110, *inputs.RMAT_ABCD, seed=4), "diamond": inputs.diamond,
          "cycles": lambda: (np.array([0, 0, 1, 2, 3, 4, 4, 9], np.uint32), np.array([1, 2, 3, 3, 0, 4, 0, 4], np.uint32)),
          "star": lambda: inputs.out_star(70), "none": lambda: inputs.chain(12)}


@pytest.mark.parametrize("form", [ROUNDS, TAIL, MATRICES])
@pytest.mark.parametrize("graph", sorted(GRAPHS))
def test_graphs(harness, tmp_path, graph, form):
    for kb, grid, diagonal in ((4, 3, True), (8, 2, False)):
        assert _run(harness, tmp_path, [GRAPHS[graph]()], form, kb=kb, grid=grid, diagonal=diagonal) == 0


def test_wide_frontier_leaves_the_tail(harness, tmp_path):
    """A tree whose last generations have more pairs than the tail takes: rounds and tails in turn."""
    assert _run(harness, tmp_path, [inputs.binary_tree(7)], TAIL, slots=1 << 16) == 0


@pytest.mark.parametrize("form", [ROUNDS, TAIL])
def test_batches(harness, tmp_path, form):
    graphs = [inputs.erdos_renyi(40, 44, seed=1), (np.empty(0, np.uint32), np.empty(0, np.uint32)), inputs.binary_tree(4),
              inputs.diamond(), inputs.erdos_renyi(90, 100, seed=2)]
    assert _run(harness, tmp_path, graphs, form, kb=4) == 0


def test_too_small_tables_are_reported(harness, tmp_path):
    src, dst = inputs.binary_tree(6)
    for form in (ROUNDS, TAIL):
        assert _run(harness, tmp_path, [(src, dst)], form, slots=1 << 8) & 3
        assert _run(harness, tmp_path, [inputs.binary_tree(6)], form, levels=4) & 4
