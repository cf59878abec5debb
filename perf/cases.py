"""What a user of the decoder has it do, as timed passes: sizes, inputs, one pass, and the work it cannot do without.

A pass is what a recognition server does with one batch of utterances through the public entry points
(`paper_2306_15685_amd.binding`, and `runner.contexts_from_words` where biasing lists come as words): contexts set or
switched, utterances started, chunks of log-likelihoods decoded, intermediate results where the caller shows them, the
final best paths with their arcs.  Graphs, decoders and log-likelihoods are on the GPU before the pass; word lists, arc
lists and results are host data, as at the C boundary.

Kinds of case:
  hclg      HCLG-style graphs (10 % epsilon-input arcs, a quarter of the arcs with words), one workgroup per channel
  lexicon   lexicon loop over end-to-end units (a hub with an arc per word, thousands of tokens per frame)
  words     biasing lists arrive as word sequences: Algorithm 1, pre-loaded contexts, a first chunk under them
  long      long utterances whose back-pointer records are compacted as decoding goes, results in two parts
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

from paper_2306_15685_amd import binding as B
from paper_2306_15685_amd import runner, synth

DEV = "cuda"


def _hclg(name, states, pdfs, words, channels, frames, chunk, beam, max_active, sigma, ctx_min, ctx_max, offset_lo,
          offset_hi, lookup, partial, segments=1, eps=0.10, finals=False):
    """partial: "" = final results only, "wait" = the caller waits for a result after every chunk (a live caption),
    "beside" = requests are begun after a chunk and collected after the next one (a server that must not stall)."""
    c = dict(kind="hclg", states=states, pdfs=pdfs, words=words, channels=channels, frames=frames, chunk=chunk, beam=beam,
             max_active=max_active, sigma=sigma, ctx_min=ctx_min, ctx_max=ctx_max, offset_lo=offset_lo, offset_hi=offset_hi,
             lookup=lookup, partial=partial, segments=segments, eps=eps, finals=finals)
    return dict(c, name=name) if name else c


def _lexicon(name, units, words, channels, frames, chunk, beam, max_active, sigma, ctx_min, ctx_max, team, partial):
    c = dict(kind="lexicon", pdfs=units, words=words, channels=channels, frames=frames, chunk=chunk, beam=beam,
             max_active=max_active, sigma=sigma, ctx_min=ctx_min, ctx_max=ctx_max, offset_lo=-2.0, offset_hi=-2.0, lookup=1,
             team=team, partial=partial, segments=1)
    return dict(c, name=name) if name else c


def _words(name, states, pdfs, words, channels, frames, beam, seqs_min, seqs_max):
    c = dict(kind="words", states=states, pdfs=pdfs, words=words, channels=channels, frames=frames, beam=beam, max_active=10000,
             sigma=4.0, seqs_min=seqs_min, seqs_max=seqs_max, lookup=1)
    return dict(c, name=name) if name else c


def _long(name, states, pdfs, channels, frames, chunk, compact_every, beam, max_active, sigma, ctx):
    c = dict(kind="long", states=states, pdfs=pdfs, words=20000, channels=channels, frames=frames, chunk=chunk,
             compact_every=compact_every, beam=beam, max_active=max_active, sigma=sigma, ctx=ctx, lookup=0)
    return dict(c, name=name) if name else c


def listed():
    return [
        # a command or a short utterance on a small grammar, decoded in one call: launch and host latency count
        _hclg("command", 2_000, 200, 600, 1, 100, 100, 10.0, 0, 3.0, 20, 20, -3.0, -3.0, 0, "", eps=0.15, finals=True),
        # one live stream: 0.3 s chunks, the caption updated after each (the caller waits for every result)
        _hclg("live", 1_000_000, 3_000, 20_000, 1, 60, 10, 13.0, 7_000, 4.0, 50, 50, -5.0, -5.0, 0, "wait"),
        # 10-second recordings handed over whole, fewer channels than compute units
        _hclg("recordings", 1_000_000, 3_000, 20_000, 32, 333, 333, 13.0, 7_000, 4.0, 50, 50, -5.0, -5.0, 0, ""),
        # a mid-size server over a small graph: tight max-active (the histogram cut acts), an odd row length, final costs
        _hclg("pruned", 100_003, 1_021, 5_000, 100, 151, 17, 14.0, 200, 3.5, 10, 300, -6.0, -2.0, 0, "beside", finals=True),
        # an online server: 256 streams in 1.5 s chunks with intermediate results per chunk
        _hclg("server", 10_000_000, 6_000, 200_000, 256, 500, 50, 15.0, 10_000, 4.0, 100, 500, -5.0, -5.0, 1, "beside"),
        # short utterances, each with a fresh context (air-traffic style), twice as many channels as compute units
        _hclg("utterances", 10_000_000, 6_000, 200_000, 512, 100, 100, 15.0, 10_000, 4.0, 10, 1_000, -8.0, -2.0, 1, "",
              segments=4),
        # two thousand clients with thousand-entry lists at a wide beam
        _hclg("clients", 10_000_000, 6_000, 200_000, 2_048, 100, 50, 16.0, 20_000, 4.0, 1_000, 1_000, -5.0, -5.0, 1, ""),
        # end-to-end units, a 20,000-word loop: teams of four workgroups per channel
        _lexicon("units", 96, 20_000, 64, 100, 50, 10.0, 2_500, 2.0, 100, 300, 4, "beside"),
        # the same task with more channels than teams fit: one workgroup per channel
        _lexicon("units_many", 96, 20_000, 160, 40, 40, 10.0, 2_500, 2.0, 100, 300, 1, ""),
        # a smaller vocabulary, few channels
        _lexicon("units_small", 64, 3_000, 8, 100, 50, 10.0, 1_500, 2.0, 30, 100, 4, ""),
        # biasing lists arrive as word sequences for every channel of a server: arc lists made, loaded, used
        _words("word_lists", 2_000_000, 4_000, 50_000, 128, 25, 15.0, 3, 15),
        # minutes-long recordings with the records compacted every 100 frames
        _long("long", 1_000_000, 3_000, 8, 1_000, 50, 2, 13.0, 7_000, 4.0, 50),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["hclg"] * 6 + ["lexicon"] * 2 + ["words", "long"])
    if kind == "hclg":
        pdfs = _log_int(rng, 100, 6_000)
        channels = _log_int(rng, 1, 2_048)
        # at most the channel-frames and log-likelihood bytes of the largest listed case
        frames = _log_int(rng, 10, max(10, min(600, 200_000 // channels)))
        chunk = max(_log_int(rng, 5, 100), (frames + 15) // 16)
        lo = rng.randint(1, 500)
        return _hclg("", _log_int(rng, 2_000, 10_000_000), pdfs, _log_int(rng, 500, 200_000), channels, frames,
                     min(chunk, frames), round(rng.uniform(9.0, 16.0), 2), rng.choice([0, 200, 2_000, 10_000]), 4.0, lo,
                     lo + rng.randint(0, 500), round(rng.uniform(-8.0, -4.0), 2), round(rng.uniform(-4.0, -1.0), 2),
                     rng.choice([0, 1]), rng.choice(["", "wait", "beside"]), finals=rng.random() < 0.5)
    if kind == "lexicon":
        channels = _log_int(rng, 1, 160)
        frames = _log_int(rng, 10, max(10, min(200, 6_400 // channels)))
        words = _log_int(rng, 500, 20_000)
        lo = rng.randint(10, 150)
        team = 4 if channels * 4 <= 256 else (2 if channels * 2 <= 256 else 1)
        return _lexicon("", rng.randint(40, 200), words, channels, frames, min(_log_int(rng, 10, 100), frames), 10.0,
                        _log_int(rng, 300, 2_500), 2.0, lo, lo + rng.randint(0, 150), team, rng.choice(["", "beside"]))
    if kind == "words":
        lo = rng.randint(1, 8)
        states = _log_int(rng, 200_000, 2_000_000)
        # (at least a hundredth as many words as states: a list then stays within the decoder's 2,048 arcs)
        return _words("", states, _log_int(rng, 500, 4_000), _log_int(rng, max(5_000, states // 100), 50_000),
                      _log_int(rng, 4, 128), rng.randint(5, 25), round(rng.uniform(11.0, 15.0), 2), lo, lo + rng.randint(0, 7))
    return _long("", _log_int(rng, 100_000, 1_000_000), _log_int(rng, 500, 3_000), _log_int(rng, 1, 16),
                 _log_int(rng, 300, 1_000), rng.randint(30, 60), rng.randint(2, 4), round(rng.uniform(11.0, 13.0), 2), 7_000, 4.0,
                 rng.randint(10, 200))


# ---- graphs: what a server loads once and keeps ----------------------------------------------------------------------


class _Graph:
    """A decoding graph: the library's handle, and what the input drawing needs of it on the device."""

    def __init__(self, S, P, row, dst, ilabel, olabel, weight, final):
        h = lambda t: None if t is None else t.cpu().numpy()  # noqa: E731
        self.S, self.A = S, int(dst.numel())
        self.row, self.dst, self.olabel = row.to(torch.int64), dst, olabel
        self.handle = B.cbd_graph_load(S, P, 0, h(row), h(dst), h(ilabel), h(olabel), h(weight), h(final))

    def __del__(self):
        if getattr(self, "handle", None) is not None:
            B.cbd_graph_free(self.handle)


@functools.lru_cache(maxsize=12)
def _random_graph(states, pdfs, words, eps, finals, period):
    """Out-degree Poisson(3) at least 1; epsilon-input arcs lead upwards; weights -ln U(0.05, 1); the recipe of
    synth.make_graph, drawn on the device.  period > 0: words that many arcs apart, as in a composed graph."""
    g = torch.Generator(device=DEV)
    g.manual_seed(1_000_003 * period + states)
    rand = lambda n: torch.rand(n, generator=g, device=DEV, dtype=torch.float64)  # noqa: E731
    S = states
    deg = torch.poisson(torch.full((S,), 3.0, device=DEV), generator=g).clamp_(min=1).to(torch.int64)
    row = torch.zeros(S + 1, dtype=torch.int64, device=DEV)
    torch.cumsum(deg, 0, out=row[1:])
    src = torch.repeat_interleave(torch.arange(S, device=DEV), deg)
    A = int(src.numel())
    is_eps = (rand(A) < eps) & (src < S - 1)
    up = (src + 1 + (rand(A) * (S - 1 - src)).to(torch.int64)).clamp_(max=S - 1)
    dst = torch.where(is_eps, up, (rand(A) * S).to(torch.int64).clamp_(max=S - 1))
    word = 1 + (rand(A) * words).to(torch.int64).clamp_(max=words - 1)
    if period > 0:
        want = (src + 1) % period
        moved = dst - dst % period + want
        moved = torch.where(is_eps & (moved <= src), moved + period, moved)
        fits = moved < S
        is_eps &= fits
        dst = torch.where(fits, moved, want)
        olabel = torch.where(dst % period == 0, word, 0)
    else:
        olabel = torch.where(rand(A) < 0.25, word, 0)
    ilabel = torch.where(is_eps, 0, 1 + (rand(A) * pdfs).to(torch.int64).clamp_(max=pdfs - 1))
    weight = (-torch.log(0.05 + 0.95 * rand(A))).to(torch.float32)
    final = (-torch.log(0.05 + 0.95 * rand(S))).to(torch.float32) if finals else None
    i32 = torch.int32
    return _Graph(S, pdfs, row.to(i32), dst.to(i32), ilabel.to(i32), olabel.to(i32), weight, final)


@functools.lru_cache(maxsize=4)
def _lexicon_graph(units, words):
    g = synth.make_lexicon_graph(units, words)
    t = lambda a: torch.from_numpy(a).to(DEV)  # noqa: E731
    return _Graph(g.num_states, units, t(g.row_offsets), t(g.dst), t(g.ilabel), t(g.olabel), t(g.weight), None)


def _graph(case):
    if case["kind"] == "lexicon":
        return _lexicon_graph(case["pdfs"], case["words"])
    return _random_graph(case["states"], case["pdfs"], case["words"], case.get("eps", 0.10), case.get("finals", False),
                         4 if case["kind"] == "words" else 0)


# ---- inputs ----------------------------------------------------------------------------------------------------------


def _loglikes(case, gen, frames):
    """Scores as an acoustic model leaves them: log-softmax over pdfs."""
    x = torch.randn((case["channels"], frames, case["pdfs"]), generator=gen, device=DEV, dtype=torch.float32)
    x.mul_(case["sigma"])
    return torch.log_softmax(x, dim=-1)


def _walks(g, n, steps, gen):
    """The arcs that n random walks from random states cross: [n, steps]."""
    cur = torch.randint(0, g.S, (n,), generator=gen, device=DEV)
    out = torch.empty((n, steps), dtype=torch.int64, device=DEV)
    for k in range(steps):
        first, deg = g.row[cur], g.row[cur + 1] - g.row[cur]
        a = first + (torch.rand(n, generator=gen, device=DEV) * deg).to(torch.int64).minimum(deg - 1)
        out[:, k] = a
        cur = g.dst[a].to(torch.int64)
    return out


def _contexts(case, g, rng, gen, lo, hi):
    """Per channel lo..hi word arcs along connected walks (in a lexicon loop: any word ends), as Algorithm 1 returns them
    -> (arc_idx, list_offsets), offsets."""
    C = case["channels"]
    want = rng.integers(lo, hi + 1, C)
    if case["kind"] == "lexicon":
        wa = torch.nonzero(g.olabel > 0).flatten()
        lists = [np.sort(rng.choice(wa.numel(), size=min(int(k), wa.numel()), replace=False)) for k in want]
        idx, off = B.pack_lists(lists)
        return (wa[torch.from_numpy(idx.astype(np.int64)).to(DEV)].to(torch.int32).cpu().numpy(), off)
    per_walk, steps = 10, 40
    n_walks = (want + per_walk - 1) // per_walk + 1
    owner = np.repeat(np.arange(C), n_walks)
    arcs = _walks(g, int(owner.size), steps, gen)
    is_word = g.olabel[arcs] > 0
    keep = (is_word & (torch.cumsum(is_word, 1) <= per_walk)).cpu().numpy()
    flat, own = arcs.cpu().numpy()[keep].astype(np.int32), np.broadcast_to(owner[:, None], keep.shape)[keep]
    first = np.searchsorted(own, np.arange(C))
    take = np.arange(own.size) - first[own] < want[own]
    off = np.zeros(C + 1, np.int32)
    np.cumsum(np.bincount(own[take], minlength=C), out=off[1:])
    return np.ascontiguousarray(flat[take]), off


def _sequences(case, g, rng, gen):
    """Per channel a list of sequences of 1 to 3 words that occur in the graph."""
    C = case["channels"]
    n = rng.integers(case["seqs_min"], case["seqs_max"] + 1, C)
    arcs = _walks(g, int(n.sum()), 16, gen)
    words = g.olabel[arcs].cpu().numpy()
    seqs = [[int(x) for x in w[w > 0][:1 + i % 3]] for i, w in enumerate(words)]
    cut = np.concatenate([[0], np.cumsum(n)])
    return [[q for q in seqs[cut[i]:cut[i + 1]] if q] for i in range(C)]


class _Results:
    """Host arrays for k result requests of n channels; request i writes into row i."""

    def __init__(self, k, n, capacity, arcs, tails=False):
        self.words = np.zeros((k, n, capacity), np.int32)
        self.arcs = np.zeros((k, n, capacity), np.int32) if arcs else None
        self.n_words, self.n_arcs, self.status = (np.zeros((k, n), np.int32) for _ in range(3))
        self.cost = np.zeros((k, n), np.float32)
        self.fixed = np.zeros((k, 2, n), np.int32)
        self.tails = tails
        self.buffers = []
        for i in range(k):
            b = B.BestPathBuffers(n, 1, want_arcs=False)
            b.capacity = capacity
            b.words, b.n_words, b.n_arcs, b.cost, b.status = self.words[i], self.n_words[i], self.n_arcs[i], self.cost[i], self.status[i]
            b.arcs = self.arcs[i] if arcs else None
            b.n_fixed_words, b.n_fixed_arcs = self.fixed[i]
            self.buffers.append(b)

    def outputs(self):
        out = dict(words=self.words, n_words=self.n_words, n_arcs=self.n_arcs, cost=self.cost, status=self.status)
        if self.arcs is not None:
            out["arcs"] = self.arcs
        if self.tails:
            out["fixed"] = self.fixed
        return out


class _State:
    """A decoder and the inputs of one pass."""

    def __init__(self, case, seed):
        self.case = c = case
        self.g = g = _graph(c)
        rng = np.random.default_rng([seed, 1])
        gen = torch.Generator(device=DEV)
        gen.manual_seed(seed)
        kind, C, T = c["kind"], c["channels"], c["frames"]
        self.channels = np.arange(C, dtype=np.int32)
        self.decoder = None
        stream = torch.cuda.current_stream().cuda_stream
        segments = c.get("segments", 1)
        self.loglikes = [_loglikes(c, gen, T) for _ in range(segments)]
        capacity = 2 * T + 64
        if kind == "words":
            self.sequences = _sequences(c, g, rng, gen)
            self.offsets = rng.uniform(-6.0, -2.0, C).astype(np.float32)
            self.final = _Results(1, C, capacity, True)
            self.list_arcs = np.zeros(C * 2_048, np.int32)   # the arc lists back to back
            # (a word labels some thirty arcs, so fifteen sequences stay within 2,048; the pool holds one list a channel)
            self.decoder = B.cbd_decoder_create(g.handle, C, c["beam"], c["max_active"], T, 2_048, c["lookup"], 14,
                                                records_per_frame=runner.DEFAULT_RECORDS_PER_FRAME, max_pool_contexts=C,
                                                hip_stream=stream)
            return
        if kind == "long":
            self.contexts = [_contexts(c, g, rng, gen, c["ctx"], c["ctx"])]
            self.offsets = [np.full(C, -5.0, np.float32)]
            n = (T + c["chunk"] - 1) // c["chunk"]
            self.partial = _Results(n, C, capacity, False, tails=True)
            self.final = _Results(1, C, capacity, True)
            self.decoder = B.cbd_decoder_create(g.handle, C, c["beam"], c["max_active"], 400, max(c["ctx"], 1), c["lookup"], 14,
                                                records_per_frame=runner.DEFAULT_RECORDS_PER_FRAME, hip_stream=stream)
            return
        self.contexts = [_contexts(c, g, rng, gen, c["ctx_min"], c["ctx_max"]) for _ in range(segments)]
        self.offsets = [rng.uniform(c["offset_lo"], c["offset_hi"], C).astype(np.float32) for _ in range(segments)]
        n = (T + c["chunk"] - 1) // c["chunk"]
        self.partial = _Results(segments * (n - 1), C, capacity, False) if c["partial"] and n > 1 else None
        self.final = _Results(segments, C, capacity, True)
        if kind == "lexicon":
            log2 = max(12, math.ceil(math.log2(3.2 * c["words"])))
            self.decoder = B.cbd_decoder_create(g.handle, C, c["beam"], c["max_active"], T, c["ctx_max"], c["lookup"], log2,
                                                records_per_frame=5 * c["words"] // 4, workgroups_per_channel=c["team"],
                                                hip_stream=stream)
        else:
            self.decoder = B.cbd_decoder_create(g.handle, C, c["beam"], c["max_active"], T, c["ctx_max"], c["lookup"], 14,
                                                records_per_frame=runner.DEFAULT_RECORDS_PER_FRAME, hip_stream=stream)

    def __del__(self):
        if self.decoder is not None:
            B.cbd_decoder_free(self.decoder)


def prepare(case, seed):
    return _State(case, seed)


# ---- one pass --------------------------------------------------------------------------------------------------------


def _advance(s, L, t, n):
    C, T, P = L.shape
    B.cbd_advance(s.decoder, s.channels, L.data_ptr() + 4 * t * P, T * P, n)


def _run_decode(s):
    c, d, ch = s.case, s.decoder, s.channels
    T, cap = c["frames"], 2 * c["frames"] + 64
    k = 0
    for seg, L in enumerate(s.loglikes):
        B.cbd_set_contexts(d, ch, None, s.offsets[seg], packed=s.contexts[seg])
        B.cbd_reset_channels(d, ch)
        pending = None
        for t in range(0, T, c["chunk"]):
            n = min(c["chunk"], T - t)
            _advance(s, L, t, n)
            if s.partial is None or t + n >= T:
                continue
            if c["partial"] == "wait":
                B.cbd_best_paths(d, ch, False, cap, want_arcs=False, buffers=s.partial.buffers[k], as_lists=False)
            else:
                if pending is not None:
                    B.cbd_best_paths_finish(d, pending[0], buffers=s.partial.buffers[pending[1]], as_lists=False)
                pending = (B.cbd_best_paths_begin(d, ch, False, cap, want_arcs=False), k)
            k += 1
        if pending is not None:
            B.cbd_best_paths_finish(d, pending[0], buffers=s.partial.buffers[pending[1]], as_lists=False)
        B.cbd_best_paths(d, ch, True, cap, want_arcs=True, buffers=s.final.buffers[seg], as_lists=False)
    out = {"final": s.final.outputs()}
    if s.partial is not None:
        out["partial"] = s.partial.outputs()
    return out


def _run_words(s):
    c, d, ch = s.case, s.decoder, s.channels
    made, _ = runner.contexts_from_words(s.g.handle, [(s.sequences, s.offsets)])
    packed = B.pack_lists(made[0][0])
    ids = B.cbd_contexts_create(d, None, s.offsets, packed=packed)
    B.cbd_use_contexts(d, ch, ids)
    B.cbd_reset_channels(d, ch)
    _advance(s, s.loglikes[0], 0, c["frames"])
    B.cbd_best_paths(d, ch, True, 2 * c["frames"] + 64, want_arcs=True, buffers=s.final.buffers[0], as_lists=False)
    B.cbd_use_contexts(d, ch, np.full(ch.size, -1, np.int32))
    for i in ids:
        B.cbd_context_destroy(d, i)
    s.list_arcs[:packed[0].size] = packed[0]
    return {"final": s.final.outputs(), "list_arcs": s.list_arcs, "list_offsets": packed[1]}


def _run_long(s):
    c, d, ch, L = s.case, s.decoder, s.channels, s.loglikes[0]
    T, cap = c["frames"], 2 * c["frames"] + 64
    B.cbd_set_contexts(d, ch, None, s.offsets[0], packed=s.contexts[0])
    B.cbd_reset_channels(d, ch)
    for k, t in enumerate(range(0, T, c["chunk"])):
        _advance(s, L, t, min(c["chunk"], T - t))
        if (k + 1) % c["compact_every"] == 0:
            B.cbd_compact_records(d, ch)
        B.cbd_best_tails(d, ch, False, cap, want_arcs=False, buffers=s.partial.buffers[k], as_lists=False)
    B.cbd_best_paths(d, ch, True, cap, want_arcs=True, buffers=s.final.buffers[0], as_lists=False)
    return {"final": s.final.outputs(), "partial": s.partial.outputs()}


def run(state):
    kind = state.case["kind"]
    return (_run_words if kind == "words" else _run_long if kind == "long" else _run_decode)(state)


# ---- what a pass cannot do without -----------------------------------------------------------------------------------


def _tokens(case):
    """Tokens of a channel-frame that are expanded, on average (as counted on these inputs)."""
    if case["kind"] == "lexicon":
        return min(0.95 * case["max_active"], 1.5 * case["words"])
    by_beam = 350.0 * math.exp(1.44 * (case["beam"] / case["sigma"] - 3.75))
    return min(by_beam, case["max_active"] or by_beam, 0.3 * case["states"])


def work(case):
    """Bytes: the log-likelihood rows, a 12-byte arc per expansion (three of a token's, or the hub's row), an 8-byte record
    per token, the lists and the paths.  Operations: two additions and a comparison per arc."""
    frames = case["channels"] * case["frames"] * case.get("segments", 1)
    tokens = _tokens(case)
    arcs = (2.2 * tokens + case["words"] if case["kind"] == "lexicon" else 3.3 * tokens) * frames
    records = (case["words"] if case["kind"] == "lexicon" else tokens) * frames
    lists = case["channels"] * case.get("segments", 1) * (case.get("ctx_min", case.get("ctx", 300)) + case.get("ctx_max", case.get("ctx", 300))) / 2
    return {"bytes": 4 * case["pdfs"] * frames + 12 * arcs + 8 * records + 4 * lists + 8 * frames, "flops": 3 * arcs}


def tolerance(case):
    # (cost, arc) keys are exact and every choice is independent of thread order
    return "exact"
