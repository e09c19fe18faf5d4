"""A decode row's logits do not depend on the rows beside it: the same rows,
alone, in small batches and in batches past the 32 rows of a block (which take
other block shapes), give the same bits, and the single rows match the oracle.
Batches on both sides of the lines at which the LayerNorms (8 rows) and the merge
of the cross attention's key chunks (2) become kernels of their own and the
float32 vocabulary product changes its tiles (32), and rows from every block of
32.  The widths reach the products' limits: a K of fewer
chunks than a block has waves, the widest rows, an MLP that is not a power of
two."""
import numpy as np
import pytest

from oracle import whisper as OW
from paper_2603_11273_amd import synth

from gpu_util import TOL, cpu_params, make_context, needs_gpu, rel_err

pytestmark = [pytest.mark.gpu, needs_gpu]


@pytest.mark.parametrize("n_head,d_ffn,vocab,dtype,batches", [
    (1, 64, 40000, "f32", [2, 5, 32, 33]), (6, 1536, 500, "f32", [2, 3, 8, 9, 34, 128]),
    (20, 1344, 500, "f32", [4, 17, 40]),
    (2, 128, 500, "bf16", [2, 31, 65]), (12, 3072, 500, "bf16", [2, 3, 4, 5, 8, 9, 32, 33, 128]),
    (20, 5120, 500, "bf16", [3, 5, 40]), (32, 1920, 500, "bf16", [2, 5, 8, 36]),
    (32, 128, 500, "f32", [8, 9]),
])
def test_rows_do_not_depend_on_the_batch(n_head, d_ffn, vocab, dtype, batches):
    d = 64 * n_head
    shape = synth.ModelShape("rows", 80, d, 0, 2, n_head, d_ffn, vocab, dtype)
    seed = 20260370 + n_head
    B = max(batches)
    ctx = make_context(shape, seed, max_slots=B, max_prefill=8, max_decode=B)
    E = [synth.encoder_output(seed, b % 3, d).numpy() for b in range(B)]
    kv = [synth.self_kv_prefix(seed, b, 2, n_head).numpy() for b in range(3)]
    lengths = [(7 * b) % 440 for b in range(B)]
    toks = synth.token_ids(seed, B, shape.vocab)
    for b0 in range(0, B, 8):
        part = list(range(b0, min(B, b0 + 8)))
        ctx.debug_set_encoder_out(part, [-1] * len(part), [40] * len(part),
                                  np.stack([E[b] for b in part]))

    def step(rows):
        for b in rows:
            ctx.debug_set_self_kv(b, kv[b % 3], lengths[b])
        return ctx.step(slots=rows, tokens=[int(toks[b]) for b in rows], want_logits=True)["logits"]

    some = [0, 1, 2, 4, 7, 8, 31, 32, 33, 63, 64, 95, 96, B - 1]
    alone = {b: step([b])[0] for b in some if b < B}
    for n in batches:
        got = step(list(range(n)))
        for b in some:
            if b < n:
                assert np.array_equal(got[b], alone[b]), (n, b)
    P = cpu_params(shape, seed)
    for b in some[:2]:
        ckv = OW.cross_kv(E[b], P, 2)
        pre = kv[b % 3][:, :, :, :lengths[b]].transpose(0, 1, 3, 2, 4).reshape(2, 2, lengths[b], d)
        st = OW.DecoderState(2, d, pre[:, 0], pre[:, 1])
        ref = OW.decoder_step(int(toks[b]), st, ckv, P, 2, n_head)
        assert rel_err(alone[b], ref) <= TOL[dtype]


@pytest.mark.parametrize("vocab,dtype", [(1, "f32"), (33, "f32"), (289, "f32"), (70001, "f32"),
                                         (40, "bf16"), (65569, "bf16")])
def test_argmax_over_tile_counts_and_nan_rows(vocab, dtype):
    """One tile, a last tile of one entry, tile counts that leave a part of a
    block over, and more tiles than a block reads in one pass; a NaN row makes the
    step fail, and only the step that holds it."""
    shape = synth.ModelShape("argmax", 80, 128, 0, 1, 2, 128, vocab, dtype)
    ctx = make_context(shape, 20260392, max_slots=3, max_prefill=3, max_decode=3)
    E = np.stack([synth.encoder_output(20260392, b, 128).numpy() for b in range(3)])
    E[1, 7, 5] = np.nan
    ctx.debug_set_encoder_out([0, 1, 2], [-1] * 3, [40] * 3, E)
    for slots in ([0], [2, 0]):
        r = ctx.step(slots=slots, tokens=[0] * len(slots), want_logits=True)
        assert np.array_equal(r["argmax"], r["logits"].argmax(1))
    with pytest.raises(Exception, match="NaN logit"):
        ctx.step(slots=[0, 1, 2], tokens=[0] * 3)
    r = ctx.step(slots=[0, 2], tokens=[0] * 2, want_logits=True)
    assert np.array_equal(r["argmax"], r["logits"].argmax(1))
