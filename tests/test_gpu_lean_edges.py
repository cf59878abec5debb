"""GPU parity of lean frames where a wave's list of arcs, its tiles and its commit log end: graphs in which every state is
a token after a few frames, so that the sizes below decide how many tokens and arcs each of the sixteen waves has."""
import numpy as np
import pytest

from paper_2306_15685_amd import synth

from test_gpu_parity import run_batch, torch_cuda  # noqa: F401

pytestmark = pytest.mark.gpu


def full_graph(S, deg, eps_every, seed):
    """S states with `deg` emitting arcs each; every eps_every-th (0: none) has an epsilon-input arc to its successor."""
    rng = np.random.default_rng(seed)
    row, dst, ilabel = [0], [], []
    for s in range(S):
        d = [(s * deg + j + 1) % S for j in range(deg)]   # (together they reach every state)
        il = list(1 + rng.integers(0, 40, deg))
        if eps_every and s % eps_every == 0 and s + 1 < S:
            d.insert(1, s + 1)
            il.insert(1, 0)
        dst += d
        ilabel += il
        row.append(len(dst))
    A = len(dst)
    olabel = np.where(rng.random(A) < 0.25, 1 + rng.integers(0, 8, A), 0).astype(np.int32)
    return synth.Graph(S, A, 40, 9, 0, np.array(row, np.int32), np.array(dst, np.int32), np.array(ilabel, np.int32), olabel,
                       rng.uniform(0.1, 1.0, A).astype(np.float32))


# states, degree: arcs of a wave at one, two and more rounds of 64 lanes, tiles of 64 tokens and the remainder of one, the
# owner map's 256 positions, the commit log's 256 entries
@pytest.mark.parametrize("eps_every", [0, 3, 40])
@pytest.mark.parametrize("S,deg", [(3, 2), (16, 3), (17, 64), (100, 3), (157, 3), (160, 4), (161, 4), (189, 5), (256, 4), (272, 4),
                                   (320, 2), (512, 4), (517, 4), (1024, 2), (1031, 2), (1024, 4), (1045, 4)])
def test_sizes(torch_cuda, S, deg, eps_every):  # noqa: F811
    print("states", S, "degree", deg, "epsilon arcs every", eps_every, flush=True)
    g = full_graph(S, deg, eps_every, seed=S + deg)
    C, T = 2, 16
    L = synth.make_loglikes(C, T, g.num_pdfs, 2.0, seed_stream=(S, deg), device="cuda")
    listed = np.arange(0, g.num_arcs, 7, dtype=np.int32)[:50]
    s = run_batch(torch_cuda, g, L, [listed, listed[::2]], [-2.0, 1.5], beam=60.0, max_active=0, chunks=[5, 11])
    assert s["status"] == 0 and s["max_tokens"] >= 0.9 * S
    # Who decodes the frames in which all states are tokens: rows of 63 arcs or more, and waves that log more than 256 commits
    # (on average, so one of them does), go to the general code; the lean code takes all frames of sizes that stay clear of its
    # limits (256 commits, and 64 closure records in 128 arcs, by four and five standard deviations of a Poisson count).
    arcs = (S + 15) // 16 * deg
    closures, in_round = (arcs / eps_every, min(arcs, 128) / eps_every) if eps_every else (0, 0)
    print("lean frames", s["lean_frames"], "of", s["frames"], flush=True)
    if deg >= 63 or arcs + closures > 256:
        assert s["lean_frames"] < s["frames"]
    elif arcs + closures + 4 * closures ** 0.5 <= 256 and in_round + 5 * in_round ** 0.5 <= 64:
        assert s["lean_frames"] == s["frames"]


def boosted_graph(S, deg, short_every, listed_per_row, offset, beam, eps_every, seed):
    """As full_graph, every short_every-th state (0: none) with one arc less, and the list that goes with it: the last emitting
    arcs of every row, whose weights are lower than the others' by the list's offset.  Boosted, all arcs cost the same on
    average; any of them taken without the offset lies below all that are right by about as much."""
    rng = np.random.default_rng(seed)
    row, dst, ilabel, listed = [0], [], [], []
    for s in range(S):
        n = deg - 1 if short_every and s % short_every == 0 else deg
        d = [(s * deg + j + 1) % S for j in range(n)]
        il = list(1 + rng.integers(0, 40, n))
        last = list(range(max(0, n - listed_per_row), n))
        if eps_every and s % eps_every == 0 and s + 1 < S:
            d.insert(1, s + 1)
            il.insert(1, 0)
            last = [j + 1 if j >= 1 else j for j in last]
        listed += [row[-1] + j for j in last]
        dst += d
        ilabel += il
        row.append(len(dst))
    A = len(dst)
    weight = rng.uniform(0.0, 0.6 * beam, A).astype(np.float32)
    listed = np.array(listed, np.int32)
    weight[listed] -= np.float32(offset)
    olabel = np.where(rng.random(A) < 0.25, 1 + rng.integers(0, 8, A), 0).astype(np.int32)
    return synth.Graph(S, A, 40, 9, 0, np.array(row, np.int32), np.array(dst, np.int32), np.array(ilabel, np.int32), olabel,
                       weight), listed


# states, degree, short rows: 2, 62 to 64, 63, 64, 65, 126 to 128, 126, 128, 129 and 256 arcs per wave, and two tiles with
# one token in the second; the last: more listed arcs (2,752) than the copy of a list in LDS holds
@pytest.mark.parametrize("lookup_mode", [0, 1])
@pytest.mark.parametrize("S,deg,short_every,listed_per_row", [(16, 2, 0, 1), (256, 4, 16, 1), (144, 7, 0, 1), (256, 4, 0, 1),
                                                              (208, 5, 0, 1), (512, 4, 32, 1), (288, 7, 0, 1), (512, 4, 0, 1),
                                                              (688, 3, 0, 1), (1024, 4, 0, 1), (1040, 3, 0, 1), (688, 5, 0, 4)])
@pytest.mark.parametrize("of_beam,max_active", [(0.5, 0), (1.0, 0), (2.0, 0), (0.5, 3), (-0.5, 0)])
def test_positive_offsets(torch_cuda, S, deg, short_every, listed_per_row, lookup_mode, of_beam, max_active):  # noqa: F811
    """A wave's lanes beyond its last arc: that arc is listed in every row, and without its offset it would be the frame's best.
    Offsets below, at and above the beam, which is narrow enough for a cutoff that is off by the offset to drop tokens."""
    print("states", S, "degree", deg, "offset", of_beam, "of the beam, max-active", max_active, "lookup", lookup_mode, flush=True)
    beam = 6.0
    # (closures only where a wave's 256 log entries hold them beside its arcs)
    g, listed = boosted_graph(S, deg, short_every, listed_per_row, of_beam * beam, beam, 9 if S * deg <= 3200 else 0, S + deg)
    C, T = 2, 12
    L = synth.make_loglikes(C, T, g.num_pdfs, 0.4, seed_stream=(S, deg), device="cuda")
    s = run_batch(torch_cuda, g, L, [listed, listed], [of_beam * beam, of_beam * beam], beam=beam,
                  max_active=S // max_active if max_active else 0, chunks=[5, 7], lookup_mode=lookup_mode)
    assert s["status"] == 0 and s["lean_frames"] == s["frames"] == C * T


@pytest.mark.parametrize("lookup_mode", [0, 1])
def test_one_listed_arc_above_the_beam(torch_cuda, lookup_mode):  # noqa: F811
    """A chain of one arc per state, all listed at +20 where the beam is 10: each frame has one candidate, and keeps it."""
    T = 5
    g = synth.Graph(T + 1, T, 4, 9, 0, np.array([0, 1, 2, 3, 4, 5, 5], np.int32), np.arange(1, T + 1, dtype=np.int32),
                    np.ones(T, np.int32), np.arange(1, T + 1, dtype=np.int32), np.full(T, 0.5, np.float32))
    L = torch_cuda.zeros((1, T, 4), dtype=torch_cuda.float32, device="cuda")
    listed = np.arange(T, dtype=np.int32)
    s = run_batch(torch_cuda, g, L, [listed], [20.0], beam=10.0, max_active=0, chunks=[1] * T, lookup_mode=lookup_mode)
    assert s["status"] == 0 and s["frames"] == s["lean_frames"] == s["tokens"] == T
