"""Many biasing lists at once (cbd_context_lists_from_words) against the checker's plain statement of Algorithm 1."""
import numpy as np
import pytest

from paper_2306_15685_amd import binding as B
from paper_2306_15685_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("period,loops,words", [(4, 0.0, 300), (0, 0.3, 40), (0, 0.0, 2_000), (1, 0.0, 50)])
def test_lists_equal_the_checker(period, loops, words):
    """Word labels four arcs apart; no spacing and self-loops (one large component behind almost every state, all
    signatures full); many words (sparse signatures); every arc labelled (no searches).  1 list to more lists than
    threads, empty ones, unknown words, repeated sequences."""
    from oracle import arcs_for_sequences
    g = synth.make_graph(3_000, 50, words, 0.1, seed_stream=(77, period), self_loop_frac=loops, word_period=period)
    rng = np.random.default_rng(5)
    lists = []
    for i in range(70):
        seqs = synth.word_sequences_on_walks(g, i % 5, 1 + i % 4, rng)
        lists.append(seqs + ([[words + 7], []] if i % 7 == 0 else []) + seqs[:1])
    gh = B.cbd_graph_load(g.num_states, g.num_pdfs, g.start_state, g.row_offsets, g.dst, g.ilabel, g.olabel, g.weight)
    try:
        for n in (0, 1, 70):
            arcs, off = B.cbd_context_lists_from_words(gh, lists[:n])
            assert off.size == n + 1 and off[0] == 0 and off[-1] == arcs.size
            for i in range(n):
                assert np.array_equal(arcs[off[i]:off[i + 1]], arcs_for_sequences(g, lists[i])), f"list {i}"
    finally:
        B.cbd_graph_free(gh)


def test_report_of_lists_made():
    """What runner.contexts_from_words says of its work: lists, host time, sizes and the threads they were shared over."""
    from paper_2306_15685_amd import runner
    g = synth.make_graph(3_000, 50, 300, 0.1, seed_stream=(77, 4), word_period=4)
    seqs = synth.word_sequences_on_walks(g, 40, 2, np.random.default_rng(5))
    gh = B.cbd_graph_load(g.num_states, g.num_pdfs, g.start_state, g.row_offsets, g.dst, g.ilabel, g.olabel, g.weight)
    try:
        made, said = runner.contexts_from_words(gh, [([[q] for q in seqs], np.zeros(40, np.float32)), ([seqs], np.zeros(1, np.float32))])
        assert [len(lists) for lists, _ in made] == [40, 1] and said["lists"] == 41 and said["ms_per_list"] > 0
        assert said["arcs_per_list"] * 41 == sum(x.size for lists, _ in made for x in lists)
        assert said["threads"] == B.lib().cbd_context_lists_threads(40) and 1 <= said["threads"] <= 10
        assert runner.contexts_from_words(gh, [([seqs], np.zeros(1, np.float32))])[1]["threads"] == 1
        assert runner.contexts_from_words(gh, [])[1]["threads"] == 1
    finally:
        B.cbd_graph_free(gh)
