"""The fp32 path's products and attention at sizes where their tiling can go
wrong: a K that is not a whole number of stages (24 n_mels), row counts on
both sides of the rule that picks the tile shape, and query blocks of both
sizes with a remainder.  The encoder output of the same clip must be the same
bits however many clips share the batch, whichever tile shape that takes."""
import numpy as np
import pytest

from paper_2603_11273_amd import synth

from gpu_util import TOL, cpu_params, make_context, needs_gpu, oracle_encode, rel_err

pytestmark = [pytest.mark.gpu, needs_gpu]


@pytest.mark.parametrize("n_mels,n_head,d_ffn", [(8, 1, 64), (40, 6, 1536), (128, 3, 320)])
def test_f32_encoder_small_shapes(n_mels, n_head, d_ffn):
    shape = synth.ModelShape("odd", n_mels, 64 * n_head, 2, 0, n_head, d_ffn, 0, "f32")
    seed = 20260360 + n_mels
    lengths = [16000, 480000, 333, 70001, 5000]
    ctx = make_context(shape, seed, max_slots=0, max_prefill=len(lengths), max_decode=0)
    clips = [synth.pcm_clip(seed, i, n) for i, n in enumerate(lengths)]
    ctx.set_encoder_streams(1)
    all_at_once = ctx.debug_encode(clips)
    P = cpu_params(shape, seed)
    for i in (0, 2):
        assert rel_err(all_at_once[i], oracle_encode(clips[i], P, shape)) <= TOL["f32"]
    for n in range(1, len(clips)):
        assert np.array_equal(ctx.debug_encode(clips[:n]), all_at_once[:n]), n
