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
