"""GPU parity of the lean frames' list lookup (two arcs per lane, steps counted by the list's length): list lengths
around the powers of two and the length the LDS copy ends at, listed arcs at both ends of the arc numbering, rows
that are staged in LDS and rows that are not."""
import numpy as np
import pytest

from test_gpu_parity import mid_inputs, run_batch, torch_cuda  # noqa: F401

pytestmark = pytest.mark.gpu

LENGTHS = (0, 1, 2, 3, 4, 5, 63, 64, 65, 1023, 1024, 1025, 2047, 2048, 2049)


@pytest.mark.parametrize("lookup_mode", [0, 1])
@pytest.mark.parametrize("pdfs", [500, 1500])
def test_list_lengths(torch_cuda, lookup_mode, pdfs):  # noqa: F811
    C = len(LENGTHS)
    g, L, _, _ = mid_inputs(torch_cuda, C=C, T=20, S=3_000, P=pdfs, seed=31)
    rng = np.random.default_rng(31)
    ctxs = []
    for i, k in enumerate(LENGTHS):
        lo, hi = ((0, g.num_arcs), (0, g.num_arcs // 2), (g.num_arcs // 2, g.num_arcs))[i % 3]
        ends = [0, g.num_arcs - 1] if k > 1 else []   # of the numbering
        inner = np.arange(max(lo, 1), min(hi, g.num_arcs - 1))
        x = np.sort(np.concatenate([ends, rng.choice(inner, size=k - len(ends), replace=False)]).astype(np.int32))
        assert np.unique(x).size == k
        ctxs.append(x)
    offs = rng.uniform(-6.0, 2.0, C).astype(np.float32)
    s = run_batch(torch_cuda, g, L, ctxs, offs, beam=12.0, max_active=0, chunks=[7, 13], lookup_mode=lookup_mode)
    assert s["status"] == 0 and s["tokens"] > 0
