"""bf16 encoder products of a few clips: widths whose K has fewer tiles than a
product has LDS stages (d = 128: two), whose rows and columns leave remainders,
and batch sizes on both sides of the tile rules.  A clip's encoder output is the
same bits in every batch, whichever kernels its products took, and matches the
oracle."""
import numpy as np
import pytest

from paper_2603_11273_amd import synth

from gpu_util import TOL, cpu_params, make_context, needs_gpu, oracle_encode, rel_err

pytestmark = [pytest.mark.gpu, needs_gpu]


@pytest.mark.parametrize("n_mels,n_head,d_ffn,n", [
    (128, 2, 128, 3), (80, 4, 1152, 6), (128, 10, 2560, 9), (96, 6, 384, 4), (64, 20, 5120, 5),
    (96, 20, 1280, 5),
])
def test_clip_is_the_same_in_every_batch(n_mels, n_head, d_ffn, n):
    shape = synth.ModelShape("small-batch", n_mels, 64 * n_head, 2, 0, n_head, d_ffn, 0, "bf16")
    seed = 20260380 + n_head
    lengths = [16000 + 37000 * i for i in range(n)]
    ctx = make_context(shape, seed, max_slots=0, max_prefill=n, max_decode=0)
    clips = [synth.pcm_clip(seed, i, x) for i, x in enumerate(lengths)]
    ctx.set_encoder_streams(1)
    together = ctx.debug_encode(clips)
    ref = oracle_encode(clips[n - 1], cpu_params(shape, seed), shape)
    assert rel_err(together[n - 1], ref) <= TOL["bf16"]
    for k in range(1, n):
        assert np.array_equal(ctx.debug_encode(clips[:k]), together[:k]), k
    for g in (2, 3):
        ctx.set_encoder_streams(g)
        assert np.array_equal(ctx.debug_encode(clips), together), g


def test_log_mel_clip_is_the_same_in_every_batch():
    """The normalisation gives a thread 1 to 16 vectors by the batch's size: one
    up to 8 clips of 80 filters, two from 9 and three at 17, and none of that
    changes a value."""
    shape = synth.ModelShape("small-batch-mel", 80, 128, 1, 0, 2, 128, 0, "bf16")
    ctx = make_context(shape, 20260391, max_slots=0, max_prefill=17, max_decode=0)
    clips = [synth.pcm_clip(20260391, i, 800 + 27000 * i) for i in range(17)]
    together = ctx.debug_logmel(clips)
    for k in (1, 8, 9):
        assert np.array_equal(ctx.debug_logmel(clips[-k:]), together[-k:]), k
