"""GPU parity of frames decoded by parts (graphs with long rows, frames that outgrow the LDS tables): shares of the states
from one to eight, long rows into states with and without closure lists, an unprepared mix of long and ordinary rows, pruning,
final costs, context swaps, frames that move between the LDS tables and the shares, frames whose queues are too small, and a
graph that the shares cannot take."""
import numpy as np
import pytest

import gpu_harness as GH
from paper_2306_15685_amd import binding as B
from paper_2306_15685_amd import synth

from test_gpu_parity import run_batch, torch_cuda  # noqa: F401

pytestmark = pytest.mark.gpu


def hub_graph(S, P, hubs, hub_arcs, mean_degree=3.0, eps=0.15, finals=False, seed=1, eps_hubs=0):
    """An HCLG-style random graph in which a few states, the start state among them, have long rows (each between 513 and
    hub_arcs emitting arcs more), and one arc in twenty leads to one of these.  A state with so many arcs has no stored
    closure list if any of them is an epsilon-input arc: eps_hubs of the long rows have one, the others none."""
    g = synth.make_graph(S, P, 500, eps, seed_stream=(seed, 7), mean_degree=mean_degree, with_finals=finals)
    rng = np.random.default_rng(seed)
    hub = np.concatenate([[g.start_state], 1 + rng.choice(S - 1, hubs - 1, replace=False)])
    dst = g.dst.copy()
    to_hub = (rng.random(g.num_arcs) < 0.05) & (g.ilabel > 0)
    dst[to_hub] = rng.choice(hub, int(to_hub.sum()))
    rows = [[dst[a:b], g.ilabel[a:b], g.olabel[a:b], g.weight[a:b]] for a, b in zip(g.row_offsets[:-1], g.row_offsets[1:])]
    for i, h in enumerate(hub):
        emitting = rows[h][1] > 0
        rows[h] = [x[emitting] for x in rows[h]]
        if i < eps_hubs:   # (epsilon-input arcs lead upwards: no cycle)
            rows[h] = [np.append(x, y).astype(x.dtype) for x, y in zip(rows[h], (rng.integers(h + 1, S), 0, 0, 0.5))]
        n = 513 if i == 1 else int(rng.integers(513, hub_arcs + 1))
        more = [rng.integers(0, S, n), rng.integers(1, P + 1, n), rng.integers(0, 500, n), rng.uniform(0.0, 3.0, n)]
        rows[h] = [np.concatenate(x) for x in zip(rows[h], more)]
    row = np.concatenate([[0], np.cumsum([len(r[0]) for r in rows])]).astype(np.int32)
    d, il, ol, w = (np.concatenate([r[k] for r in rows]) for k in range(4))
    return synth.Graph(S, int(row[-1]), P, 500, g.start_state, row, d.astype(np.int32), il.astype(np.int32),
                       ol.astype(np.int32), w.astype(np.float32), g.final_cost)


def inputs(torch, g, C, T, sigma, seed, arcs=200):
    L = synth.make_loglikes(C, T, g.num_pdfs, sigma, seed_stream=(seed,), device="cuda")
    rng = np.random.default_rng(seed)
    ctxs = [np.sort(rng.choice(g.num_arcs, size=arcs, replace=False)).astype(np.int32) for _ in range(C)]
    return L, ctxs, rng.uniform(-4.0, 2.0, C).astype(np.float32)


def by_parts(s, shares):
    """Most frames that outgrew the LDS tables were decoded by parts, with that many shares.  (Small LDS tables, or 256
    threads, leave little room for the list of closures: 4 to 29 of some 72 frames are given up for it.)"""
    p = s["parts"]
    print("parts", p, "slow", s["slow_frames"], "of", s["frames"], "max tokens", s["max_tokens"], flush=True)
    return p["shares"] == shares and s["slow_frames"] // 2 < p["frames"] <= s["slow_frames"] - p["given_up"]


@pytest.mark.parametrize("hash_log2,block,pdfs,shares", [
    (12, 1024, 64, 1), (13, 1024, 1_500, 2), (14, 1024, 64, 4), (15, 1024, 64, 8), (14, 960, 64, 4), (13, 512, 64, 4), (12, 256, 64, 4)])
def test_shares_and_long_rows(torch_cuda, hash_log2, block, pdfs, shares):  # noqa: F811
    """64 tokens of LDS tables leave some 2,900 slots with 1,024 threads, 830 with 256, 12 bytes each: as many shares as hold
    2^hash_log2 / 2 tokens in seven eighths of them.  Most frames hold more than 64 tokens and less than 2,048; rows of
    1,500 pdfs are read from device memory."""
    print("shares", hash_log2, block, flush=True)
    g = hub_graph(2_000, pdfs, 6, 1_500, seed=hash_log2)
    L, ctxs, offs = inputs(torch_cuda, g, 3, 24, 2.5, hash_log2)
    s = run_batch(torch_cuda, g, L, ctxs, offs, beam=7.0, max_active=0, chunks=[1, 6, 17], hash_log2=hash_log2, lookup_mode=hash_log2 & 1,
                  lds_token_cap=64, block_threads=block)
    assert s["slow_frames"] > s["frames"] // 2 and s["eps_arcs"] > 0 and s["max_tokens"] > 300
    assert by_parts(s, shares)


def test_closure_that_is_not_stored(torch_cuda):  # noqa: F811
    """One long row with an epsilon-input arc: such a state's closure has no list, which the shares need."""
    g = hub_graph(2_000, 64, 6, 1_500, seed=12, eps_hubs=1)
    L, ctxs, offs = inputs(torch_cuda, g, 3, 24, 2.5, 12)
    s = run_batch(torch_cuda, g, L, ctxs, offs, beam=7.0, max_active=0, chunks=[1, 6, 17], hash_log2=12, lds_token_cap=64)
    assert s["slow_frames"] > 0 and s["parts"] == {"shares": 0, "mostly": False, "frames": 0, "given_up": 0}


def test_pruning_finals_and_swap(torch_cuda):  # noqa: F811
    g = hub_graph(4_000, 96, 5, 900, finals=True, seed=3)
    L, ctxs, offs = inputs(torch_cuda, g, 4, 30, 2.0, 3)
    swap = (10, [c[::2] for c in ctxs], -offs)
    s = run_batch(torch_cuda, g, L, ctxs, offs, beam=8.0, max_active=150, chunks=[10, 20], hash_log2=14, use_final=True,
                  swap=swap, lds_token_cap=128)
    assert s["active_tokens"] < s["tokens"] and by_parts(s, 4)


def test_frames_move_between_the_tables(torch_cuda):  # noqa: F811
    """Around as many tokens as the LDS tables hold: frames go to the shares and come back."""
    g = hub_graph(6_000, 400, 3, 700, seed=5)
    L, ctxs, offs = inputs(torch_cuda, g, 4, 40, 4.0, 5)
    s = run_batch(torch_cuda, g, L, ctxs, offs, beam=9.0, max_active=0, chunks=[3, 17, 20], hash_log2=13, lds_token_cap=192)
    assert s["slow_frames"] < s["frames"] and by_parts(s, 2)


def test_queues_too_small(torch_cuda):  # noqa: F811
    """More candidates than a share's queue holds (640 emitting, 384 closure candidates) over a graph of 300 states, within
    the 512 tokens and 1,024 improvements of the general code, which decodes such frames."""
    g = hub_graph(300, 40, 2, 600, seed=9)
    L, ctxs, offs = inputs(torch_cuda, g, 2, 12, 1.0, 9, arcs=30)
    s = run_batch(torch_cuda, g, L, ctxs, np.abs(offs), beam=6.0, max_active=0, chunks=[5, 7], hash_log2=10, lds_token_cap=64)
    assert s["status"] == 0 and s["parts"]["shares"] == 1 and s["parts"]["given_up"] > 0
    assert s["parts"]["frames"] < s["slow_frames"]


def test_one_row_too_long_to_lay_out(torch_cuda):  # noqa: F811
    """The first long row, the start state's, alone exceeds what the shares' tables take; the others are laid out all the
    same (the key tables, four bytes per slot, are there), and all frames agree."""
    g = hub_graph(2_000, 64, 6, 600, seed=12)
    deg = np.diff(g.row_offsets)
    others, n = int(deg[deg > 512].sum() - deg[g.start_state]), 6_000
    rng = np.random.default_rng(4)
    at = g.row_offsets[g.start_state + 1]
    add = lambda x, y: np.insert(x, at, np.asarray(y, x.dtype))  # noqa: E731
    row = g.row_offsets.copy()
    row[g.start_state + 1:] += n
    big = synth.Graph(g.num_states, g.num_arcs + n, g.num_pdfs, g.num_words, g.start_state, row, add(g.dst, rng.integers(0, 2_000, n)),
                      add(g.ilabel, rng.integers(1, 65, n)), add(g.olabel, rng.integers(0, 500, n)), add(g.weight, rng.uniform(0, 3, n)), None)
    assert others < 2 * 2_880 // 2 < n
    plain = synth.make_graph(2_000, 64, 500, 0.15, seed_stream=(12, 7))
    L, ctxs, offs = inputs(torch_cuda, big, 3, 16, 2.5, 12)
    kw = dict(beam=7.0, max_active=0, chunks=[1, 15], hash_log2=13, lds_token_cap=64)
    s = run_batch(torch_cuda, big, L, ctxs, offs, **kw)
    base = run_batch(torch_cuda, plain, L, [c[c < plain.num_arcs] for c in ctxs], offs, **kw)
    extra = s["info"]["device_bytes"] - base["info"]["device_bytes"]
    print("too long", s["parts"], s["slow_frames"], extra, flush=True)
    assert s["parts"]["shares"] == 2 and s["parts"]["frames"] > 0 and extra > 4 * 2 * 2_880


@pytest.mark.parametrize("words,shares", [(600, 8), (6_000, 2)])
def test_lexicon_loop(torch_cuda, words, shares):  # noqa: F811
    """LDS tables of 256 tokens, and as large as LDS allows: eight shares of 3,500 slots and two of 11,700 for 16,384 tokens."""
    g = synth.make_lexicon_graph(48, words, seed_stream=(5, words))
    L = synth.make_loglikes(3, 25, 48, 2.0, seed_stream=(5,), device="cuda")
    w = synth.scaled(synth.WORKLOADS["e2e"], channels=3, config_id=71)
    ctxs, offs = synth.make_contexts(w, g)
    s = run_batch(torch_cuda, g, L, ctxs, offs, beam=10.0, max_active=800 if words > 600 else 100, chunks=[3, 10, 12], hash_log2=15,
                  lookup_mode=1, lds_token_cap=0 if words > 600 else 256)
    assert s["status"] == 0 and by_parts(s, shares)


@pytest.mark.parametrize("block", [1024, 960, 512, 256])
def test_kernel_for_frames_that_mostly_outgrow_lds(torch_cuda, block):  # noqa: F811
    """records_per_frame chooses between two kernels of the same results: more than the LDS tables hold, or not (equal to
    them, or not given)."""
    g = hub_graph(2_000, 64, 6, 1_500, seed=21)
    L, ctxs, offs = inputs(torch_cuda, g, 2, 16, 2.5, 21)
    for records, mostly in ((0, False), (64, False), (65, True), (2_000, True)):
        s = run_batch(torch_cuda, g, L, ctxs, offs, beam=7.0, max_active=0, chunks=[5, 11], hash_log2=12, lds_token_cap=64,
                      block_threads=block, max_frames=16 if records in (0, 2_000) else 400, records_per_frame=records)
        assert s["parts"]["mostly"] is mostly and s["parts"]["frames"] > s["frames"] // 4


def test_long_rows_beside_result_walks(torch_cuda):  # noqa: F811
    """A decoder whose calls fill the device in one round, on a graph with long rows: every chunk's partial result is
    requested before the next chunk is decoded, which then runs in the 120-register kernel.  Lean frames, general ones and
    frames by parts; partial results, final tables and paths are the checker's (every fifth channel)."""
    n_cu = torch_cuda.cuda.get_device_properties(0).multi_processor_count
    C, T = n_cu * 5 // 8, 30
    g = hub_graph(6_000, 400, 3, 700, seed=5)
    L, ctxs, offs = inputs(torch_cuda, g, C, T, 4.0, 5)
    dec = GH.GpuDecoder(g, C, 9.0, max_frames=T, hash_log2=13, lds_token_cap=192)
    try:
        some = range(0, C, 5)
        orcs = dict(zip(some, GH.oracle_channels(g, len(some), 9.0)))
        Lh = L[::5].cpu().numpy()
        dec.set_contexts(ctxs, offs)
        dec.reset()
        for c in some:
            orcs[c].set_context(ctxs[c], offs[c])
            orcs[c].reset()
        pending, want = None, None
        for t in range(0, T, 6):
            dec.advance(L, t, t + 6)
            if pending is not None:
                st, wl, al, cost, na, nw = B.cbd_best_paths_finish(dec.dh, pending)
                for c in some:
                    GH.assert_best_equal((int(st[c]), wl[c], al[c], float(cost[c])), want[c], f"partial t={t} ch={c}")
            pending = B.cbd_best_paths_begin(dec.dh, dec.all, False, 4 * T + 16)
            for i, c in enumerate(some):
                orcs[c].advance(Lh[i, t:t + 6])
            want = {c: orcs[c].best_path(False) for c in some}
        B.cbd_best_paths_finish(dec.dh, pending)
        for c in some:
            GH.assert_tables_equal(dec.tokens(c), orcs[c].tokens(), f"final table ch={c}")
            GH.assert_best_equal(dec.best(c), orcs[c].best_path(False), f"final ch={c}")
        p, s = B.cbd_get_parts(dec.dh), dec.stats()
        print("beside", p, s["lean_frames"], s["frames"], flush=True)
        assert p["shares"] > 0 and not p["mostly"] and p["frames"] > 0 and 0 < s["lean_frames"] < s["frames"]
    finally:
        dec.close()
