"""GPU parity of frames that the lean code gives up behind its second barrier, when the next frame's staged
log-likelihood row is already in LDS or on its way there: the redone frame reads its own row, the frame after it the next."""
import pytest

from test_gpu_parity import mid_inputs, run_batch, torch_cuda  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("block", [256, 1024])
@pytest.mark.parametrize("pdfs,beam", [(3, 5.0), (64, 13.0), (257, 13.0), (1021, 13.0), (1024, 13.0)])
def test_frames_redone_with_the_next_row_staged(torch_cuda, pdfs, beam, block):  # noqa: F811
    """Row lengths that are copied 4 and 16 bytes per lane, by one wave and by all, up to the longest staged one.  Between
    a tenth and two thirds of the frames make more than the 128 tokens that the LDS tables hold, which is counted behind
    that barrier."""
    g, L, ctxs, offs = mid_inputs(torch_cuda, C=4, T=24, S=20_000, P=pdfs, seed=33)
    s = run_batch(torch_cuda, g, L, ctxs, offs, beam=beam, max_active=0, chunks=[1, 9, 14], lds_token_cap=128,
                  block_threads=block)
    assert 0 < s["slow_frames"] < s["frames"]
