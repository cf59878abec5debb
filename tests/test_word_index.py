"""Algorithm 1's word index (csrc/word_index.hpp) on the host, compiled by itself, against the checker."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

from oracle import arcs_for_sequence
from paper_2306_15685_amd import binding as B
from paper_2306_15685_amd import synth

HERE = os.path.dirname(os.path.abspath(__file__))
SRC = os.path.join(HERE, "word_index_host.cpp")


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    lib = str(tmp_path_factory.mktemp("word_index") / "libword_index.so")
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-shared", "-fPIC", "-pthread", "-o", lib, SRC], check=True)
    L = C.CDLL(lib)
    L.word_index_make.restype = C.c_void_p
    L.word_index_make.argtypes = [C.c_int32, C.c_void_p, C.c_void_p, C.c_void_p]
    L.word_index_free.restype = None
    L.word_index_free.argtypes = [C.c_void_p]
    L.word_index_laid_out.restype = C.c_int32
    L.word_index_laid_out.argtypes = [C.c_void_p]
    L.word_index_lists.restype = C.c_int64
    L.word_index_lists.argtypes = [C.c_void_p, C.c_void_p, C.c_void_p, C.c_void_p, C.c_int32, C.c_void_p, C.c_int64, C.c_void_p]
    return L


class Index:
    def __init__(self, host, g):
        self.L, self.keep = host, [np.ascontiguousarray(x, np.int32) for x in (g.row_offsets, g.dst, g.olabel)]
        self.h = host.word_index_make(g.num_states, *(x.ctypes.data for x in self.keep))

    def lists(self, lists):
        words, offs = B.pack_lists([np.asarray(q, np.int32) for seqs in lists for q in seqs])
        lo = np.cumsum([0] + [len(x) for x in lists]).astype(np.int32)
        ao = np.zeros(len(lists) + 1, np.int64)
        arcs = np.empty(1 << 22, np.int32)
        n = self.L.word_index_lists(self.h, words.ctypes.data, offs.ctypes.data, lo.ctypes.data, len(lists),
                                    arcs.ctypes.data, arcs.size, ao.ctypes.data)
        assert n <= arcs.size
        return [arcs[ao[i]:ao[i + 1]].copy() for i in range(len(lists))]

    def laid_out(self):
        return bool(self.L.word_index_laid_out(self.h))

    def close(self):
        self.L.word_index_free(self.h)


GRAPHS = [(4, 0.0, 300), (0, 0.3, 40), (0, 0.0, 2_000)]


@pytest.mark.parametrize("period,loops,words", GRAPHS)
def test_word_0_stands_for_arcs_without_word(host, period, loops, words):
    """A 0 after the first word is followed like a word, through the arcs that carry none (as the checker does it); a
    sequence that begins with one contributes nothing, nor does an id below 0 or above the graph's."""
    g = synth.make_graph(300, 50, words, 0.1, seed_stream=(78, period), self_loop_frac=loops, word_period=period)
    rng = np.random.default_rng(6)
    seqs = []
    for q in synth.word_sequences_on_walks(g, 8, 3, rng):
        for at in range(len(q) + 1):
            seqs.append(q[:at] + [0] + q[at:])
            seqs.append(q[:at] + [int(rng.choice([-1, -2**31, words + 9, 2**31 - 1]))] + q[at:])
    seqs += [[0], [0, 0], [seqs[0][-1], 0, 0], []]
    want = [np.array(sorted(arcs_for_sequence(g, q)) if q and q[0] > 0 else [], np.int32) for q in seqs]
    assert sum(x.size for x, q in zip(want, seqs) if 0 in q) > 0
    index = Index(host, g)
    got = index.lists([[q] for q in seqs])
    index.close()
    for q, x, y in zip(seqs, want, got):
        assert np.array_equal(x, y), q


class Chain:
    """A ring of S states in random order, a word every `apart` states: the searches' paths have no branches."""
    def __init__(self, S, apart, words, rng):
        at = rng.permutation(S)
        self.num_states, self.src = S, np.arange(S)
        self.row_offsets, self.dst, self.olabel = np.arange(S + 1), np.zeros(S, np.int32), np.zeros(S, np.int32)
        self.dst[at] = np.roll(at, -1)
        self.olabel[at[::apart]] = 1 + rng.integers(0, words, at[::apart].size)


@pytest.mark.parametrize("graph", ["small", "several threads", "long chains"])
def test_layout_comes_when_it_pays_and_changes_nothing(host, graph):
    """A graph's first lists don't wait for the layout of the whole graph, a request that searches enough of it does, and
    the lists before, in and after that request equal the checker's.  Graphs above 65,536 states are laid out by several
    threads; chains of 40 states without word take more sweeps than the signatures are given."""
    rng = np.random.default_rng(8)
    g = (synth.make_graph(300, 50, 300, 0.1, seed_stream=(79, 4), word_period=4) if graph == "small" else
         Chain(70_001, 40 if graph == "long chains" else 4, 5_000, rng))
    if graph == "small":
        seqs = synth.word_sequences_on_walks(g, 60, 3, rng)
    else:
        seqs = []
        for s in rng.choice(np.flatnonzero(g.olabel), 400):
            q, s = [int(g.olabel[s])], g.dst[s]
            while len(q) < 3:
                if g.olabel[s]:
                    q.append(int(g.olabel[s]))
                s = g.dst[s]
            seqs.append(q)
    want = [np.array(sorted(arcs_for_sequence(g, q)), np.int32) for q in seqs]
    index = Index(host, g)
    assert np.array_equal(index.lists([[seqs[0]]])[0], want[0]) and not index.laid_out()
    requests = 0
    while not index.laid_out():
        for x, y in zip(index.lists([[q] for q in seqs]), want):
            assert np.array_equal(x, y)
        requests += 1
        assert requests < 50
    for x, y in zip(index.lists([[q] for q in seqs]), want):
        assert np.array_equal(x, y)
    assert np.array_equal(index.lists([seqs])[0], np.unique(np.concatenate(want)))
    index.close()
    index = Index(host, g)   # one list that searches enough of it, taken up again behind the layout
    assert np.array_equal(index.lists([seqs * 8])[0], np.unique(np.concatenate(want))) and index.laid_out()
    index.close()


def test_every_failing_allocation_is_reported(tmp_path):
    """Whatever allocation of a request fails, on whatever thread and after threads were started, the request ends in
    bad_alloc or is served by fewer threads or without the layout; the process lives on."""
    exe = str(tmp_path / "no_memory")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-DNO_MEMORY", "-pthread", "-o", exe, SRC], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, (r.returncode, r.stdout, r.stderr)
