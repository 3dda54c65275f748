"""The host's bound on a trie's stored nodes (csrc/node_bound.h, which sets launch shapes) against
the oracle's tries: never below the nodes that are stored, through collections, windows, loaded
states and pending ones; as tight as the window; and the limit given to captured calls covers every
later step.  Compiled with the host compiler (CPU only)."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

import oracle.trie as otrie

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2502_00085_amd", "csrc")
WRAP = """
#include "node_bound.h"
using namespace td;
extern "C" long bound(int n, int d, int f, int t, int b, int W, int G, int cap, int leaf) {
  return node_bound(NodeBound{n, d, f, t}, TrieShape{b, W, G, cap}, leaf);
}
extern "C" long limit(int n, int d, int f, int t, int b, int W, int G, int cap, int leaf) {
  return node_limit(NodeBound{n, d, f, t}, TrieShape{b, W, G, cap}, leaf);
}
extern "C" long keys(int n, int d, int f, int t, int b, int W, int G, int cap, int leaf, long nodes, int q) {
  return window_keys(NodeBound{n, d, f, t}, TrieShape{b, W, G, cap}, leaf, nodes, q);
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("node_bound")
    (d / "w.cpp").write_text(WRAP)
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC, str(d / "w.cpp"),
                    "-o", str(d / "w.so")], check=True)
    L = ctypes.CDLL(str(d / "w.so"))
    L.bound.restype = L.limit.restype = L.keys.restype = ctypes.c_long
    L.keys.argtypes = [ctypes.c_int] * 9 + [ctypes.c_long, ctypes.c_int]
    return L


def loaded(tr):
    """What td_load_state notes of a trie: nodes, leaf depth, first depth, end of the trunk."""
    full = (1 << tr.n_live) - 1
    n_shared = 0
    while n_shared < len(tr.order) and tr.masks[id(tr.order[n_shared])] == full:
        n_shared += 1
    trunk = tr.order[n_shared - 1].depth + 1 if n_shared else 0
    return len(tr.order), tr.leaf_depth, tr.order[0].depth, trunk


@pytest.mark.parametrize("P,b,W,G", [(1, 4, 0, 1), (20, 5, 0, 4), (20, 5, 7, 1), (3, 6, 9, 4), (40, 4, 12, 15), (9, 3, 30, 2)])
@pytest.mark.parametrize("alpha", [0.0, 2.0])
def test_bound_holds_and_is_as_tight_as_the_window(lib, P, b, W, G, alpha):
    g = np.random.default_rng(P + b + W + G)
    tr = otrie.Trie(g.integers(0, 50, P), None, None, b, W, G)
    starts = [(P, P - 1, 0, P)]
    cap, seen = 10 ** 6, []
    for s in range(90):
        w = 1.0 / (np.arange(tr.n_live) + 1.0) ** alpha
        tr.append(g.choice(tr.n_live, size=b, p=w / w.sum()), g.integers(0, 50, b), np.zeros(b, np.float32))
        if tr.gc_due():
            tr.garbage_collect()
        args = [(*st, b, W, G, cap, tr.leaf_depth) for st in starts]
        for a in args:
            assert len(tr.order) <= lib.bound(*a) <= lib.limit(*a)
            assert lib.bound(*a[:7], 30, a[8]) <= 30
        # a limit taken earlier covers this step; without a window it is the capacity
        assert all(lib.bound(*args[i]) <= lim for i, lim in seen)
        seen += [(i, lib.limit(*a)) for i, a in enumerate(args)]
        assert W or all(lib.limit(*a) == cap for a in args)
        if W and s + 1 >= G + W + P:
            assert all(lib.bound(*a) <= b * (W + G - 1) for a in args if tr.leaf_depth - a[1] >= G)
        if s in (11, 30, 31):
            starts.append(loaded(tr))
    if W == 0 and G == 1:  # exact at the start, b more per append
        assert lib.bound(P, P - 1, 0, P, b, 0, 1, cap, P - 1) == P
        assert lib.bound(P, P - 1, 0, P, b, 0, 1, cap, P + 9) == P + 10 * b


def test_window_keys(lib):
    # a chain: the window and the queries; a trie of 10 nodes per level: ten times the window
    assert lib.keys(1000, 999, 0, 1000, 8, 64, 1, 10 ** 6, 999, 1000, 33) == 64 + 33
    assert lib.keys(1000, 99, 0, 0, 10, 40, 1, 10 ** 6, 99, 1000, 33) == 400 + 33
    assert lib.keys(1000, 999, 0, 1000, 8, 0, 1, 10 ** 6, 999, 1000, 33) == 1000
    assert lib.keys(200, 999, 900, 0, 8, 190, 1, 10 ** 6, 999, 200, 33) == 200
