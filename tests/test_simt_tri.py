"""Triangle counting on the renumbered graph: the kernels of both ways (pairs looked up, bits) on the
CPU SIMT shim with AddressSanitizer, against the oracle."""

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
    exe = tmp_path_factory.mktemp("simt_tri") / "tri_harness"
    subprocess.run(["g++", "-std=c++20", "-O1", "-g", "-DSIMT_STACK=131072", "-fsanitize=address",
                    "-fno-omit-frame-pointer", f"-I{SIMT}", f"-I{CSRC}", f"-I{os.path.join(ROOT, 'include')}",
                    "-pthread", os.path.join(SIMT, "tri_harness.cpp"), "-o", str(exe)], check=True,
                   capture_output=True)
    return exe


def _loops(src, dst, k):
    ids = np.unique(src)[::k]
    return np.concatenate([src, ids]), np.concatenate([dst, ids])


def _both(n):  # every ordered pair, loops included
    a, b = np.divmod(np.arange(n * n, dtype=np.uint32), np.uint32(n))
    return a, b


GRAPHS = {
    "rmat": lambda: inputs.rmat(8, 1500, *inputs.RMAT_ABCD, seed=4),
    "rmat_loops": lambda: _loops(*inputs.rmat(9, 4000, *inputs.RMAT_ABCD, seed=5), 3),
    "er": lambda: inputs.erdos_renyi(300, 900, seed=3),
    "complete": lambda: _both(40),
    "hub": lambda: (np.concatenate([np.zeros(700, np.uint32), np.arange(1, 701, dtype=np.uint32), np.arange(1, 700, dtype=np.uint32)]),
                    np.concatenate([np.arange(1, 701, dtype=np.uint32), np.zeros(700, np.uint32), np.arange(2, 701, dtype=np.uint32)])),
    "cycle": lambda: inputs.cycle(3), "chain": lambda: inputs.chain(12),
    "one_loop": lambda: (np.array([5], np.uint32), np.array([5], np.uint32)),
}


@pytest.mark.parametrize("graph", sorted(GRAPHS))
def test_graphs(harness, tmp_path, graph):
    src, dst = GRAPHS[graph]()
    ref, two = oracle.triangles(src, dst)
    w = max(1, int(max(src.max(), dst.max())).bit_length())
    E = np.unique((src.astype(np.uint64) << np.uint64(w)) | dst.astype(np.uint64))
    for kb, grid in ((4, 3), (8, 2)):
        inp = tmp_path / "in.bin"
        with open(inp, "wb") as f:
            np.array([w, kb, E.size, ((1 << w) + 31) & ~31], dtype=np.uint64).tofile(f)
            E.tofile(f)
        r = subprocess.run([str(harness), str(inp), str(grid), "4"], capture_output=True, text=True, timeout=900,
                           env=dict(os.environ, ASAN_OPTIONS="detect_leaks=0"))
        assert r.returncode == 0, (r.returncode, r.stdout + r.stderr[-3000:])
        count, paths, pieces = map(int, r.stdout.split())
        assert (count, paths) == (ref, two)
        assert pieces > 0 or graph not in ("hub", "complete", "rmat_loops")
