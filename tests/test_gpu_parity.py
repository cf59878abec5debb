"""GPU parity: the HIP library, called through its C ABI, against the CPU checker on the same
seeded inputs.  Integer results (states, arcs, words, counters) must be bit-exact; costs must
have the same fp32 bits (tolerance stated by the benchmark spec: 1e-3 absolute, also asserted)."""
import json
import os

import numpy as np
import pytest

from paper_2306_15685_amd import synth
from paper_2306_15685_amd import binding as B

import gpu_harness as GH
from oracle import OracleGraph, OracleChannel

pytestmark = pytest.mark.gpu
HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    torch.cuda.set_device(0)
    return torch


def test_wave_primitives_selftest(torch_cuda):
    """The DPP prefix sum / minimum the kernels rely on, against host loops."""
    B.cbd_selftest()


def tiny_inputs(torch, T=100, seed=(0,)):
    w = synth.WORKLOADS["tiny"]
    g = synth.graph_for(w)
    L = synth.make_loglikes(1, T, w.num_pdfs, w.sigma, seed_stream=seed, device="cuda")
    ctxs, offs = synth.make_contexts(w, g)
    return w, g, L, ctxs, offs


@pytest.mark.parametrize("table_location,block,lds_cap", [(1, 1024, 0), (2, 1024, 0), (1, 256, 0), (2, 512, 0),
                                                          (1, 1024, 192), (1, 512, 64), (1, 960, 0)])
def test_tiny_frame_by_frame(torch_cuda, table_location, block, lds_cap):
    """Config Tiny: every frame's token table, then words / path / cost / arc counter.  With a small
    LDS capacity most frames outgrow the LDS tables and are redone in device memory, and decoding
    moves back to LDS whenever the token list fits again."""
    torch = torch_cuda
    w, g, L, ctxs, offs = tiny_inputs(torch)
    Lh = L.cpu().numpy()
    dec = GH.GpuDecoder(g, 1, w.beam, w.max_active, max_frames=w.frames, table_location=table_location,
                        lds_token_cap=lds_cap, block_threads=block)
    info = B.cbd_decoder_info(dec.dh)
    assert info["tables_in_lds"] == (table_location == 1) and info["block_threads"] == block
    if lds_cap:
        assert info["lds_token_cap"] == lds_cap
    try:
        orc = GH.oracle_channels(g, 1, w.beam, w.max_active)[0]
        dec.set_contexts(ctxs, offs)
        orc.set_context(ctxs[0], offs[0])
        dec.reset(); orc.reset()
        GH.assert_tables_equal(dec.tokens(0), orc.tokens(), "after reset")
        for t in range(w.frames):
            dec.advance(L, t, t + 1)
            orc.advance(Lh[0, t:t + 1])
            GH.assert_tables_equal(dec.tokens(0), orc.tokens(), f"frame {t}")
        GH.assert_best_equal(dec.best(0), orc.best_path(), "final")
        st = dec.stats(0)
        assert st["emit_arcs"] == orc.emit_arcs and st["frames"] == w.frames
        assert st["tokens"] == orc.stat(1) and st["active_tokens"] == orc.stat(2) and st["max_tokens"] == orc.stat(3)
        if table_location == 2:
            assert st["slow_frames"] == w.frames
        elif lds_cap:
            assert 0 < st["slow_frames"] < w.frames   # both kinds of frames, and switches in both directions
        else:
            assert st["slow_frames"] == 0
    finally:
        dec.close()


def test_worked_example_on_gpu(torch_cuda):
    torch = torch_cuda
    with open(os.path.join(HERE, "golden", "worked_example.json")) as f:
        ex = json.load(f)
    g = synth.Graph(ex["num_states"], len(ex["dst"]), ex["num_pdfs"], 9, ex["start_state"],
                    np.array(ex["row_offsets"], np.int32), np.array(ex["dst"], np.int32),
                    np.array(ex["ilabel"], np.int32), np.array(ex["olabel"], np.int32),
                    np.array(ex["weight"], np.float32))
    L = torch.tensor(ex["loglikes"], dtype=torch.float32, device="cuda").unsqueeze(0).contiguous()
    for c in ex["cases"]:
        dec = GH.GpuDecoder(g, 1, c["beam"], 0, max_frames=8, hash_log2=6)
        try:
            dec.set_contexts([np.array(c["context"], np.int32)], [c["offset"]])
            dec.reset()
            for t in range(2):
                dec.advance(L, t, t + 1)
                rc, st, co, ar = dec.tokens(0)
                got = {str(int(s)): [float(x), int(a)] for s, x, a in zip(st, co, ar)}
                assert got == c["table_after_frame"][t], (c["name"], t)
            rc, words, arcs, cost = dec.best(0)
            assert rc == 0 and arcs.tolist() == c["best_arcs"] and words.tolist() == c["best_words"]
            assert cost == c["best_cost"]
        finally:
            dec.close()


def run_batch(torch, g, L, ctxs, offs, beam, max_active, chunks, lookup_mode=0, table_location=0, hash_log2=12,
              use_final=False, partial_check=True, swap=None, lds_token_cap=0, workgroups_per_cu=0,
              workgroups_per_channel=0, block_threads=0, max_frames=0, records_per_frame=0):
    """Decode all channels of L on the GPU and one by one on the checker; compare partial results
    after every chunk, final results, tables and counters.  swap = (frame, lists, offsets): replace
    all contexts before that frame (must be a chunk boundary)."""
    C, T, P = L.shape
    Lh = L.cpu().numpy()
    dec = GH.GpuDecoder(g, C, beam, max_active, max_frames=max_frames or T, lookup_mode=lookup_mode,
                        table_location=table_location, records_per_frame=records_per_frame, hash_log2=hash_log2, lds_token_cap=lds_token_cap, workgroups_per_cu=workgroups_per_cu,
                        workgroups_per_channel=workgroups_per_channel, block_threads=block_threads,
                        max_context_arcs=max(1, max(len(x) for x in ctxs),
                                                                  max((len(x) for x in swap[1]), default=1) if swap else 1))
    try:
        og = OracleGraph.from_graph(g)
        orcs = GH.oracle_channels(g, C, beam, max_active, og=og)
        dec.set_contexts(ctxs, offs)
        for c in range(C):
            orcs[c].set_context(ctxs[c], offs[c])
            orcs[c].reset()
        dec.reset()
        t = 0
        for n in chunks:
            if swap and swap[0] == t:
                dec.set_contexts(swap[1], swap[2])
                for c in range(C):
                    orcs[c].set_context(swap[1][c], swap[2][c])
            dec.advance(L, t, t + n)
            for c in range(C):
                orcs[c].advance(Lh[c, t:t + n])
            t += n
            if partial_check:
                st, wl, al, cost, na, nw = B.cbd_best_paths(dec.dh, dec.all, False, capacity=4 * T + 16)
                for c in range(C):
                    GH.assert_best_equal((int(st[c]), wl[c], al[c], float(cost[c])), orcs[c].best_path(False),
                                         f"partial t={t} ch={c}")
        for c in range(C):
            GH.assert_tables_equal(dec.tokens(c), orcs[c].tokens(), f"final table ch={c}")
            GH.assert_best_equal(dec.best(c, use_final), orcs[c].best_path(use_final), f"final ch={c}")
            s = dec.stats(c)
            assert s["emit_arcs"] == orcs[c].emit_arcs, f"ch={c} arcs expanded"
            assert s["tokens"] == orcs[c].stat(1) and s["active_tokens"] == orcs[c].stat(2)
        st = dec.stats(-1)
        st["info"] = B.cbd_decoder_info(dec.dh)
        st["parts"] = B.cbd_get_parts(dec.dh)
        return st
    finally:
        dec.close()


def mid_inputs(torch, C=6, T=48, S=60_000, P=500, sigma=4.0, eps=0.10, finals=False, seed=11, ctx_k=60):
    g = synth.make_graph(S, P, 2000, eps, seed_stream=(seed,), with_finals=finals)
    L = synth.make_loglikes(C, T, P, sigma, seed_stream=(seed,), device="cuda")
    w = synth.scaled(synth.WORKLOADS["large"], channels=C, ctx_min=ctx_k // 2, ctx_max=ctx_k, config_id=50 + seed)
    ctxs, offs = synth.make_contexts(w, g)
    return g, L, ctxs, offs


@pytest.mark.parametrize("table_location,lds_cap", [(1, 0), (2, 0), (1, 128)])
def test_multichannel_chunks_and_partials(torch_cuda, table_location, lds_cap):
    """Several channels with their own contexts, ragged chunking, partial traceback per chunk."""
    g, L, ctxs, offs = mid_inputs(torch_cuda)
    s = run_batch(torch_cuda, g, L, ctxs, offs, beam=13.0, max_active=0, chunks=[1, 7, 16, 24],
                  table_location=table_location, lds_token_cap=lds_cap)
    assert s["eps_arcs"] > 0 and s["improvements"] >= s["tokens"]
    if lds_cap:
        assert 0 < s["slow_frames"] < s["frames"]


@pytest.mark.parametrize("wgs", [1, 2, 4])
def test_shared_compute_units_and_unstaged_rows(torch_cuda, wgs):
    """Several channels per compute unit: smaller workgroups; with 6000 pdfs the log-likelihood row is read
    from device memory instead of LDS (rows of up to 1024 pdfs are staged: the other tests here)."""
    g, L, ctxs, offs = mid_inputs(torch_cuda, C=5, T=32, P=6000, seed=20)
    s = run_batch(torch_cuda, g, L, ctxs, offs, beam=13.0, max_active=0, chunks=[5, 27], workgroups_per_cu=wgs)
    assert s["info"]["block_threads"] == {1: 1024, 2: 512, 4: 256}[wgs]
    if wgs == 1:
        assert s["info"]["lds_bytes"] > 100_000     # big tables
    else:
        assert s["info"]["lds_bytes"] <= 163_840 // wgs


def test_decoding_beside_result_walks(torch_cuda):
    """A decoder whose calls fill the device in one round (more than half of the compute units) leaves room for
    result walks and decodes with the 120-register kernel while walks are in flight: every chunk's partial result
    is requested asynchronously, the next chunk is decoded before the request is finished, and every partial
    result, the final tables and the final paths are the checker's."""
    n_cu = torch_cuda.cuda.get_device_properties(0).multi_processor_count
    C = n_cu * 5 // 8
    g, L, ctxs, offs = mid_inputs(torch_cuda, C=C, T=40, S=40_000, P=400, seed=23, ctx_k=40)
    Lh = L.cpu().numpy()
    T = L.shape[1]
    dec = GH.GpuDecoder(g, C, 13.0, 0, max_frames=T, max_context_arcs=40, lookup_mode=1)
    try:
        assert B.cbd_decoder_info(dec.dh)["block_threads"] == 1024
        og = OracleGraph.from_graph(g)
        orcs = GH.oracle_channels(g, C, 13.0, 0, og=og)
        dec.set_contexts(ctxs, offs)
        for c in range(C):
            orcs[c].set_context(ctxs[c], offs[c])
            orcs[c].reset()
        dec.reset()
        pending = None   # (ticket, expected results)
        t = 0
        for n in (8, 8, 8, 8, 8):
            dec.advance(L, t, t + n)     # (from the second chunk on: with the previous chunk's walks in flight)
            if pending is not None:
                st, wl, al, cost, na, nw = B.cbd_best_paths_finish(dec.dh, pending[0])
                for c in range(C):
                    GH.assert_best_equal((int(st[c]), wl[c], al[c], float(cost[c])), pending[1][c], f"partial t={t - n} ch={c}")
            for c in range(C):
                orcs[c].advance(Lh[c, t:t + n])
            t += n
            pending = (B.cbd_best_paths_begin(dec.dh, dec.all, False, capacity=4 * T + 16),
                       [orcs[c].best_path(False) for c in range(C)])
        st, wl, al, cost, na, nw = B.cbd_best_paths_finish(dec.dh, pending[0])
        for c in range(C):
            GH.assert_best_equal((int(st[c]), wl[c], al[c], float(cost[c])), pending[1][c], f"last partial ch={c}")
        for c in range(0, C, 7):
            GH.assert_tables_equal(dec.tokens(c), orcs[c].tokens(), f"final table ch={c}")
    finally:
        dec.close()


def test_lexicon_loop_units_workload(torch_cuda):
    """Second workload (Sec. 6: end-to-end model units): a lexicon loop with a 3000-arc hub row, self-loops,
    thousands of tokens per frame, max-active pruning engaged,
    boosted epsilon-input word-end arcs."""
    torch = torch_cuda
    g = synth.make_lexicon_graph(48, 3000, seed_stream=(21,))
    L = synth.make_loglikes(3, 40, 48, 2.0, seed_stream=(21,), device="cuda")
    w = synth.scaled(synth.WORKLOADS["e2e"], channels=3, config_id=61)
    ctxs, offs = synth.make_contexts(w, g)
    assert all(np.all(g.ilabel[c] == 0) for c in ctxs)     # word-end arcs are epsilon-input arcs
    # once with the device-memory tables on every frame, once with whatever the LDS tables can carry
    s = run_batch(torch, g, L, ctxs, offs, beam=10.0, max_active=800, chunks=[3, 17, 20], hash_log2=14, lookup_mode=1,
                  table_location=2)
    assert s["slow_frames"] == s["frames"] and s["max_tokens"] > 2500
    assert s["active_tokens"] < 0.5 * s["tokens"]           # the histogram cut did most of the pruning
    s2 = run_batch(torch, g, L, ctxs, offs, beam=10.0, max_active=800, chunks=[3, 17, 20], hash_log2=14, lookup_mode=1)
    assert s2["tokens"] == s["tokens"] and s2["emit_arcs"] == s["emit_arcs"]
    # and with an LDS capacity that many frames exceed: tables move between LDS and device memory and back
    s3 = run_batch(torch, g, L, ctxs, offs, beam=10.0, max_active=800, chunks=[3, 17, 20], hash_log2=14, lookup_mode=1,
                   lds_token_cap=1024)
    assert 0 < s3["slow_frames"] and s3["tokens"] == s["tokens"]


def test_histogram_pruning_engages(torch_cuda):
    """max_active small enough that the 256-bin cut decides the survivors in most frames."""
    g, L, ctxs, offs = mid_inputs(torch_cuda, C=4, T=40, seed=12)
    s_off = run_batch(torch_cuda, g, L, ctxs, offs, beam=13.0, max_active=0, chunks=[40], partial_check=False)
    s_on = run_batch(torch_cuda, g, L, ctxs, offs, beam=13.0, max_active=60, chunks=[13, 27], partial_check=False)
    assert s_on["active_tokens"] < s_off["active_tokens"]


def test_hashed_bitmap_lookup_and_heavy_bias(torch_cuda):
    """lookup_mode 1 (bitmap filter + search) with a large list, including epsilon-input arcs."""
    torch = torch_cuda
    g, L, _, _ = mid_inputs(torch, C=4, T=40, seed=13)
    rng = np.random.default_rng(13)
    ctxs = [rng.choice(g.num_arcs, size=1000, replace=True).astype(np.int32) for _ in range(4)]  # duplicates too
    offs = np.array([-5.0, -2.0, 0.0, 3.0], np.float32)
    a = run_batch(torch, g, L, ctxs, offs, beam=12.0, max_active=0, chunks=[40], lookup_mode=1)
    b = run_batch(torch, g, L, ctxs, offs, beam=12.0, max_active=0, chunks=[40], lookup_mode=0)
    assert a["emit_arcs"] == b["emit_arcs"] and a["tokens"] == b["tokens"]


def test_context_lists_prepared_on_device_and_on_host(torch_cuda):
    """The list is a set (Sec. 4.2): given shuffled and with every entry three times it decodes like the plain
    list, whether the device sorts it (it fits its slot as given) or the host does (it fits only without repeats);
    list lengths on both sides of the powers of two the device sort pads to."""
    torch = torch_cuda
    g, L, _, offs = mid_inputs(torch, C=4, T=30, seed=15)
    rng = np.random.default_rng(15)
    ctxs = [np.sort(rng.choice(g.num_arcs, size=k, replace=False)).astype(np.int32) for k in (0, 1, 257, 512)]
    tripled = [rng.permutation(np.concatenate([x, x, x])).astype(np.int32) for x in ctxs]
    og = OracleGraph.from_graph(g)
    orcs = GH.oracle_channels(g, 4, 13.0, 0, og=og)
    Lh = L.cpu().numpy()
    for c in range(4):
        orcs[c].set_context(ctxs[c], offs[c]); orcs[c].reset(); orcs[c].advance(Lh[c])
    for lists, cap in ((ctxs, 512), (tripled, 1536), (tripled, 512)):
        dec = GH.GpuDecoder(g, 4, 13.0, 0, max_frames=30, max_context_arcs=cap)
        try:
            dec.set_contexts(lists, offs)
            dec.reset()
            dec.advance(L, 0, 30)
            for c in range(4):
                GH.assert_best_equal(dec.best(c), orcs[c].best_path(), f"cap {cap} ch {c}")
                GH.assert_tables_equal(dec.tokens(c), orcs[c].tokens(), f"cap {cap} ch {c}")
        finally:
            dec.close()


@pytest.mark.parametrize("lookup_mode", [0, 1])
def test_context_lists_longer_than_the_lds_copy(torch_cuda, lookup_mode):
    """Lists of more than 2,048 arcs stay in device memory and are searched there (Sec. 4.2's binary search, with
    and without the bitmap in front); 5,000 and 8,192 entries also reach the largest size the device sorts."""
    torch = torch_cuda
    g, L, _, _ = mid_inputs(torch, C=3, T=24, seed=16)
    rng = np.random.default_rng(16)
    ctxs = [rng.choice(g.num_arcs, size=k, replace=False).astype(np.int32) for k in (5000, 8192, 2049)]
    offs = np.array([-4.0, -1.5, -6.0], np.float32)
    s = run_batch(torch, g, L, ctxs, offs, beam=12.0, max_active=0, chunks=[5, 19], lookup_mode=lookup_mode)
    assert s["status"] == 0
    # one list beyond that size: the whole upload is then prepared on the host
    ctxs[1] = rng.choice(g.num_arcs, size=10000, replace=False).astype(np.int32)
    s = run_batch(torch, g, L, ctxs, offs, beam=12.0, max_active=0, chunks=[24], lookup_mode=lookup_mode)
    assert s["status"] == 0


def test_context_swap_mid_utterance_and_finals(torch_cuda):
    """Contexts replaced between chunks without a reset (Sec. 4.3); final costs pick the end token."""
    torch = torch_cuda
    g, L, ctxs, offs = mid_inputs(torch, C=4, T=40, seed=14, finals=True)
    w2 = synth.scaled(synth.WORKLOADS["dynamic"], channels=4, ctx_min=10, ctx_max=300, config_id=77)
    ctx2, off2 = synth.make_contexts(w2, g, segment=1)
    run_batch(torch, g, L, ctxs, offs, beam=12.0, max_active=500, chunks=[20, 20], use_final=True,
              swap=(20, ctx2, off2))


def test_preloaded_context_pool(torch_cuda):
    """Sec. 4.3: contexts loaded in advance, channels switch among them by id (also shared by several
    channels, also in mid-utterance), and can go back to their own uploaded list."""
    torch = torch_cuda
    g, L, ctxs, offs = mid_inputs(torch, C=4, T=36, seed=17)
    Lh = L.cpu().numpy()
    w2 = synth.scaled(synth.WORKLOADS["dynamic"], channels=3, ctx_min=20, ctx_max=400, config_id=78)
    pool_lists, pool_offs = synth.make_contexts(w2, g, segment=2)
    dec = GH.GpuDecoder(g, 4, 12.0, 0, max_frames=36, max_context_arcs=512, max_pool_contexts=3)
    try:
        ids = B.cbd_contexts_create(dec.dh, pool_lists, pool_offs)
        assert sorted(ids.tolist()) == [0, 1, 2]
        with pytest.raises(B.CbdError) as ei:   # pool is full
            B.cbd_contexts_create(dec.dh, pool_lists[:1], pool_offs[:1])
        assert ei.value.status == B.CBD_E_CAPACITY
        dec.set_contexts(ctxs, offs)            # the channels' own lists
        orcs = GH.oracle_channels(g, 4, 12.0, 0)
        # channels 0 and 1 share pool context 1, channel 2 uses pool context 0, channel 3 keeps its own list
        plan = {0: 1, 1: 1, 2: 0}
        B.cbd_use_contexts(dec.dh, np.array([0, 1, 2], np.int32), np.array([ids[1], ids[1], ids[0]], np.int32))
        for c in range(4):
            if c in plan:
                orcs[c].set_context(pool_lists[plan[c]], pool_offs[plan[c]])
            else:
                orcs[c].set_context(ctxs[c], offs[c])
            orcs[c].reset()
        dec.reset()
        dec.advance(L, 0, 18)
        for c in range(4):
            orcs[c].advance(Lh[c, :18])
        # mid-utterance: channel 0 goes back to its own list, channel 3 switches to pool context 2
        B.cbd_use_contexts(dec.dh, np.array([0, 3], np.int32), np.array([-1, ids[2]], np.int32))
        orcs[0].set_context(ctxs[0], offs[0])
        orcs[3].set_context(pool_lists[2], pool_offs[2])
        dec.advance(L, 18, 36)
        for c in range(4):
            orcs[c].advance(Lh[c, 18:])
            GH.assert_tables_equal(dec.tokens(c), orcs[c].tokens(), f"pool ch={c}")
            GH.assert_best_equal(dec.best(c), orcs[c].best_path(), f"pool ch={c}")
        with pytest.raises(B.CbdError):
            B.cbd_use_contexts(dec.dh, np.array([0], np.int32), np.array([7], np.int32))
        B.cbd_context_destroy(dec.dh, int(ids[0]))
        with pytest.raises(B.CbdError):
            B.cbd_use_contexts(dec.dh, np.array([1], np.int32), np.array([ids[0]], np.int32))
        assert B.cbd_contexts_create(dec.dh, pool_lists[:1], pool_offs[:1]).tolist() == [int(ids[0])]
    finally:
        dec.close()


def test_asynchronous_partial_results(torch_cuda):
    """Requests begun after a chunk and finished only after later chunks have been decoded (and a new
    utterance started) still describe the moment of the request (Sec. 2.2: intermediate results leave
    the GPU without interrupting the decoding)."""
    torch = torch_cuda
    g, L, ctxs, offs = mid_inputs(torch, C=5, T=40, seed=18)
    Lh = L.cpu().numpy()
    dec = GH.GpuDecoder(g, 5, 12.0, 0, max_frames=40)
    try:
        orcs = GH.oracle_channels(g, 5, 12.0, 0)
        dec.set_contexts(ctxs, offs)
        for c in range(5):
            orcs[c].set_context(ctxs[c], offs[c]); orcs[c].reset()
        dec.reset()
        want, tickets = [], []
        for k, (t0, t1) in enumerate([(0, 10), (10, 20), (20, 30), (30, 40)]):
            dec.advance(L, t0, t1)
            for c in range(5):
                orcs[c].advance(Lh[c, t0:t1])
            tickets.append(B.cbd_best_paths_begin(dec.dh, dec.all, False, capacity=200))
            want.append([orcs[c].best_path(False) for c in range(5)])
        with pytest.raises(B.CbdError) as ei:   # four requests are the limit
            B.cbd_best_paths_begin(dec.dh, dec.all, False, capacity=200)
        assert ei.value.status == B.CBD_E_CAPACITY
        dec.reset()                              # new utterance while the requests are still out
        dec.advance(L, 0, 5)
        for k in (2, 0, 3, 1):                   # any order
            st, wl, al, cost, na, nw = B.cbd_best_paths_finish(dec.dh, tickets[k])
            for c in range(5):
                GH.assert_best_equal((int(st[c]), wl[c], al[c], float(cost[c])), want[k][c], f"request {k} ch {c}")
        with pytest.raises(B.CbdError):
            B.cbd_best_paths_finish(dec.dh, tickets[0])   # already collected
        # the decoder went on meanwhile
        for c in range(5):
            orcs[c].reset(); orcs[c].advance(Lh[c, :5])
            GH.assert_best_equal(dec.best(c), orcs[c].best_path(), f"after requests ch {c}")
        # a request for the channels of the latest call walks from the tokens the decoding kernel left behind;
        # one for other channels, another order or with final costs takes its own snapshot: same answers
        sub = np.array([3, 0], np.int32)
        st, wl, al, cost, na, nw = B.cbd_best_paths_finish(dec.dh, B.cbd_best_paths_begin(dec.dh, sub, False, capacity=200))
        for i, c in enumerate(sub):
            GH.assert_best_equal((int(st[i]), wl[i], al[i], float(cost[i])), orcs[c].best_path(False), f"subset ch {c}")
        st, wl, al, cost, na, nw = B.cbd_best_paths_finish(dec.dh, B.cbd_best_paths_begin(dec.dh, dec.all, True, capacity=200))
        for c in range(5):
            GH.assert_best_equal((int(st[c]), wl[c], al[c], float(cost[c])), orcs[c].best_path(True), f"finals ch {c}")
        st, wl, al, cost, na, nw = B.cbd_best_paths_finish(dec.dh, B.cbd_best_paths_begin(dec.dh, dec.all, False, capacity=200))
        for c in range(5):
            GH.assert_best_equal((int(st[c]), wl[c], al[c], float(cost[c])), orcs[c].best_path(False), f"again ch {c}")
        # right after a reset the kernel-left token is the start token: empty path at cost 0
        dec.reset(sub)
        st, wl, al, cost, na, nw = B.cbd_best_paths_finish(dec.dh, B.cbd_best_paths_begin(dec.dh, sub, False, capacity=200))
        assert list(st) == [0, 0] and list(na) == [0, 0] and list(cost) == [0.0, 0.0]
    finally:
        dec.close()


def sample_word_sequences(g, n_seq, rng, max_len=4):
    """Word sequences read off random walks, so that they exist in the graph."""
    seqs = []
    for _ in range(n_seq):
        k = int(rng.integers(1, max_len + 1))
        s, words = int(rng.integers(0, g.num_states)), []
        for _ in range(400):
            if len(words) == k or g.row_offsets[s] == g.row_offsets[s + 1]:
                break
            a = int(rng.integers(g.row_offsets[s], g.row_offsets[s + 1]))
            if g.olabel[a]:
                words.append(int(g.olabel[a]))
            s = int(g.dst[a])
        if words:
            seqs.append(words)
    return seqs


def test_context_from_word_sequences(torch_cuda):
    """Algorithm 1 in the library against the checker's plain version, then a decode biased with the
    arcs it returns (unigrams, sequences, unknown words)."""
    from oracle import arcs_for_sequences
    torch = torch_cuda
    g, L, _, _ = mid_inputs(torch, C=2, T=30, S=20_000, seed=19)
    rng = np.random.default_rng(19)
    gh = B.cbd_graph_load(g.num_states, g.num_pdfs, g.start_state, g.row_offsets, g.dst, g.ilabel, g.olabel,
                          g.weight, g.final_cost)
    try:
        lists = []
        for c in range(2):
            seqs = sample_word_sequences(g, 25, rng) + [[int(rng.integers(1, 2000))], [999_999], []]
            got = B.cbd_context_from_words(gh, seqs)
            want = arcs_for_sequences(g, seqs)
            assert np.array_equal(got, want), f"list {c}: {got.size} arcs vs {want.size}"
            assert got.size > 25 and np.all(np.isin(g.olabel[got], np.concatenate([np.asarray(x) for x in seqs if x])))
            lists.append(got)
        offs = np.array([-2.0, -4.0], np.float32)   # the paper's discount factor, and a stronger one
        dec = GH.GpuDecoder(g, 2, 12.0, 0, max_frames=30, max_context_arcs=max(len(x) for x in lists), graph_handle=gh)
        try:
            orcs = GH.oracle_channels(g, 2, 12.0, 0)
            dec.set_contexts(lists, offs)
            Lh = L.cpu().numpy()
            for c in range(2):
                orcs[c].set_context(lists[c], offs[c]); orcs[c].reset()
            dec.reset(); dec.advance(L, 0, 30)
            for c in range(2):
                orcs[c].advance(Lh[c])
                GH.assert_best_equal(dec.best(c), orcs[c].best_path(), f"word-sequence context ch {c}")
        finally:
            dec.close()
    finally:
        B.cbd_graph_free(gh)


@pytest.mark.parametrize("beam,max_active", [(0.0, 0), (1.0e30, 0), (9.0, 1), (9.0, 7)])
def test_degenerate_beams(torch_cuda, beam, max_active):
    """Beam 0 (only the best token survives: greedy), a beam nothing exceeds, and max-active limits far below
    the table size (the histogram cut decides almost everything; with 1 even bin 0 overflows)."""
    g, L, ctxs, offs = mid_inputs(torch_cuda, C=3, T=20, S=3000, P=40, seed=31, ctx_k=20)
    s = run_batch(torch_cuda, g, L, ctxs, offs, beam=beam, max_active=max_active, chunks=[1, 9, 10], hash_log2=13)
    if beam == 0.0:
        assert s["active_tokens"] <= s["frames"] + 3


def test_largest_row_length_and_empty_calls(torch_cuda):
    """65535 pdfs, the most the arc record's label field can name: the row does not fit LDS and is read from
    device memory.  Calls with zero frames change nothing."""
    torch = torch_cuda
    P = 65535
    g = synth.make_graph(3000, P, 500, 0.10, seed_stream=(32,))
    assert int(g.ilabel.max()) > 60000
    L = synth.make_loglikes(2, 6, P, 4.0, seed_stream=(32,), device="cuda")
    w = synth.scaled(synth.WORKLOADS["large"], channels=2, ctx_min=5, ctx_max=20, config_id=82)
    ctxs, offs = synth.make_contexts(w, g)
    dec = GH.GpuDecoder(g, 2, 14.0, 0, max_frames=6, hash_log2=13)
    try:
        orcs = GH.oracle_channels(g, 2, 14.0, 0)
        Lh = L.cpu().numpy()
        dec.set_contexts(ctxs, offs)
        dec.reset()
        for c in range(2):
            orcs[c].set_context(ctxs[c], offs[c]); orcs[c].reset()
        dec.advance(L, 0, 0)                      # nothing to do
        for (t0, t1) in [(0, 1), (1, 1), (1, 6)]:
            dec.advance(L, t0, t1)
            for c in range(2):
                orcs[c].advance(Lh[c, t0:t1])
        for c in range(2):
            GH.assert_tables_equal(dec.tokens(c), orcs[c].tokens(), f"ch {c}")
            GH.assert_best_equal(dec.best(c), orcs[c].best_path(), f"ch {c}")
        assert dec.stats(-1)["frames"] == 12
    finally:
        dec.close()


def test_two_decoders_share_one_graph(torch_cuda):
    """The graph is immutable and shareable: two decoders with different beams and contexts, calls interleaved
    on one stream."""
    torch = torch_cuda
    g, L, ctxs, offs = mid_inputs(torch, C=2, T=30, seed=19)
    Lh = L.cpu().numpy()
    gh = B.cbd_graph_load(g.num_states, g.num_pdfs, g.start_state, g.row_offsets, g.dst, g.ilabel, g.olabel, g.weight,
                          g.final_cost)
    decs = [GH.GpuDecoder(g, 2, beam, 0, max_frames=30, graph_handle=gh) for beam in (11.0, 14.0)]
    try:
        og = OracleGraph.from_graph(g)
        orcs = [GH.oracle_channels(g, 2, beam, 0, og=og) for beam in (11.0, 14.0)]
        for k, dec in enumerate(decs):
            lists = ctxs if k == 0 else ctxs[::-1]
            o = offs if k == 0 else offs[::-1].copy()
            dec.set_contexts(lists, o)
            dec.reset()
            for c in range(2):
                orcs[k][c].set_context(lists[c], o[c]); orcs[k][c].reset()
        for (t0, t1) in [(0, 7), (7, 18), (18, 30)]:
            for k, dec in enumerate(decs):
                dec.advance(L, t0, t1)
                for c in range(2):
                    orcs[k][c].advance(Lh[c, t0:t1])
        for k, dec in enumerate(decs):
            for c in range(2):
                GH.assert_tables_equal(dec.tokens(c), orcs[k][c].tokens(), f"decoder {k} ch {c}")
                GH.assert_best_equal(dec.best(c), orcs[k][c].best_path(), f"decoder {k} ch {c}")
    finally:
        for dec in decs:
            dec.close()
        B.cbd_graph_free(gh)


def test_channel_subset_and_reuse_after_reset(torch_cuda):
    """A subset of channels advances while the others wait; a channel reset for a second utterance
    gives the same result as a fresh decoder."""
    torch = torch_cuda
    g, L, ctxs, offs = mid_inputs(torch, C=4, T=30, seed=15)
    Lh = L.cpu().numpy()
    dec = GH.GpuDecoder(g, 4, 12.0, 0, max_frames=30)
    try:
        orcs = GH.oracle_channels(g, 4, 12.0, 0)
        dec.set_contexts(ctxs, offs)
        for c in range(4):
            orcs[c].set_context(ctxs[c], offs[c]); orcs[c].reset()
        dec.reset()
        sub = np.array([3, 1], np.int32)
        Lsub = L[[3, 1]].contiguous()
        dec.advance(Lsub, 0, 30, channels=sub)
        for c in (3, 1):
            orcs[c].advance(Lh[c])
        for c in (3, 1):
            GH.assert_best_equal(dec.best(c), orcs[c].best_path(), f"subset ch={c}")
        for c in (0, 2):  # untouched channels still sit at their reset state
            GH.assert_tables_equal(dec.tokens(c), orcs[c].tokens(), f"idle ch={c}")
        # second utterance on channel 1 with channel 0's audio
        dec.reset(np.array([1], np.int32)); orcs[1].reset()
        dec.advance(L[[0]].contiguous(), 0, 30, channels=np.array([1], np.int32))
        orcs[1].advance(Lh[0])
        GH.assert_best_equal(dec.best(1), orcs[1].best_path(), "second utterance")
        assert dec.stats(1)["frames"] == 30
    finally:
        dec.close()


def test_error_states(torch_cuda):
    torch = torch_cuda
    # dead end -> NO_TOKENS; never-reset channel -> NO_TOKENS
    g = synth.Graph(2, 1, 1, 1, 0, np.array([0, 1, 1], np.int32), np.array([1], np.int32),
                    np.array([1], np.int32), np.array([1], np.int32), np.array([0.5], np.float32))
    L = torch.zeros((1, 3, 1), dtype=torch.float32, device="cuda")
    dec = GH.GpuDecoder(g, 2, 10.0, hash_log2=6)
    try:
        assert dec.best(1)[0] == B.CBD_E_NO_TOKENS
        dec.reset(np.array([0], np.int32))
        rc, words, arcs, cost = dec.best(0)
        assert rc == 0 and arcs.size == 0 and cost == 0.0
        dec.advance(L, 0, 3, channels=np.array([0], np.int32))
        assert dec.best(0)[0] == B.CBD_E_NO_TOKENS
        assert dec.stats(0)["status"] == B.CBD_E_NO_TOKENS
        dec.reset(np.array([0], np.int32))
        assert dec.best(0)[0] == 0
    finally:
        dec.close()
    # negative epsilon cycle after biasing -> EPS_DIVERGED, like the checker
    g = synth.Graph(2, 3, 1, 1, 0, np.array([0, 2, 3], np.int32), np.array([1, 0, 0], np.int32),
                    np.array([0, 1, 0], np.int32), np.array([0, 0, 0], np.int32),
                    np.array([0.5, 1.0, 0.5], np.float32))
    dec = GH.GpuDecoder(g, 1, 5.0, hash_log2=6, max_eps_iters=16)
    try:
        dec.reset()
        assert dec.best(0)[0] == 0  # positive cycle settles
        dec.set_contexts([np.array([0, 2], np.int32)], [-1.0])
        dec.reset()
        assert dec.best(0)[0] == B.CBD_E_EPS_DIVERGED
    finally:
        dec.close()
    # table too small -> CAPACITY (sticky until reset), never silent truncation
    w, gt, Lt, ctxs, offs = tiny_inputs(torch, T=40)
    for loc in (1, 2):
        dec = GH.GpuDecoder(gt, 1, w.beam, 0, hash_log2=7, table_location=loc, lds_token_cap=64)
        try:
            dec.reset()
            dec.advance(Lt, 0, 40)
            assert dec.best(0)[0] == B.CBD_E_CAPACITY
            dec.reset()
            assert dec.best(0)[0] == 0
        finally:
            dec.close()
    # invalid arguments are refused on the host
    dec = GH.GpuDecoder(gt, 2, w.beam, 0, max_context_arcs=8)
    try:
        with pytest.raises(B.CbdError):
            B.cbd_set_context(dec.dh, 0, np.array([gt.num_arcs], np.int32), -1.0)
        with pytest.raises(B.CbdError):
            B.cbd_set_context(dec.dh, 0, np.arange(9, dtype=np.int32), -1.0)
        B.cbd_set_context(dec.dh, 0, np.array([3, 3, 3, 3, 3, 3, 3, 3, 3, 3], np.int32), -1.0)  # 1 distinct arc
        with pytest.raises(B.CbdError):
            B.cbd_reset_channels(dec.dh, np.array([0, 0], np.int32))
        with pytest.raises(B.CbdError):
            B.cbd_reset_channels(dec.dh, np.array([2], np.int32))
        # small output buffer: sizes come back
        dec.reset(); dec.advance(Lt.expand(2, -1, -1).contiguous(), 0, 40)
        words = np.zeros(2, np.int32); arcs = np.zeros(2, np.int32)
        import ctypes as C
        nw, na, cost = C.c_int32(0), C.c_int32(0), C.c_float(0)
        rc = B.lib().cbd_best_path(dec.dh, 0, 0, words.ctypes.data_as(C.c_void_p), arcs.ctypes.data_as(C.c_void_p), 2,
                                   C.byref(nw), C.byref(na), C.byref(cost))
        assert rc == B.CBD_E_BUFFER and na.value >= 40
        rc2, w2, a2, c2 = dec.best(0)
        assert rc2 == 0 and a2.size == na.value and w2.size == nw.value
    finally:
        dec.close()


@pytest.mark.parametrize("table_location,block", [(1, 1024), (2, 1024), (1, 256)])
def test_repeated_decodes_match_checker(torch_cuda, table_location, block):
    """The same utterance many times over, one frame per call: counters and the final table must
    match the checker every time (lanes of different waves race for the same states; a lane can
    create a state's entry and still lose the minimum to another wave)."""
    torch = torch_cuda
    w, g, L, ctxs, offs = tiny_inputs(torch)
    Lh = L.cpu().numpy()
    orc = GH.oracle_channels(g, 1, w.beam, w.max_active)[0]
    orc.set_context(ctxs[0], offs[0]); orc.reset(); orc.advance(Lh[0])
    want = orc.tokens()
    dec = GH.GpuDecoder(g, 1, w.beam, w.max_active, max_frames=w.frames, table_location=table_location,
                        block_threads=block)
    try:
        dec.set_contexts(ctxs, offs)
        for rep in range(60):
            dec.reset()
            for t in range(w.frames):
                dec.advance(L, t, t + 1)
            st = dec.stats(0)
            assert st["tokens"] == orc.stat(1) and st["emit_arcs"] == orc.emit_arcs, f"repeat {rep}"
            GH.assert_tables_equal(dec.tokens(0), want, f"repeat {rep}")
    finally:
        dec.close()


def test_determinism_repeat(torch_cuda):
    """Two runs give identical tables (thread order must not matter)."""
    torch = torch_cuda
    g, L, ctxs, offs = mid_inputs(torch, C=3, T=30, seed=16)
    outs = []
    for rep in range(2):
        dec = GH.GpuDecoder(g, 3, 13.0, 200, max_frames=30)
        try:
            dec.set_contexts(ctxs, offs); dec.reset(); dec.advance(L, 0, 30)
            outs.append([tuple(x.tobytes() for x in dec.tokens(c)[1:]) + (dec.best(c)[2].tobytes(),) for c in range(3)])
        finally:
            dec.close()
    assert outs[0] == outs[1]
