"""The cross K/V product of bf16 contexts, as it stands in the slots' caches: every
layer, head and dim equals the oracle's, and a clip's cache is the same bits
however many clips share the product.  The sizes take each tile shape that the
product has: 128 x 64 tiles, whose waves own half a head (up to 128 tiles of
128 x 128), 128 x 128 tiles of four and of two LDS stages, and the persistent
kernel."""
import numpy as np
import pytest

from oracle import whisper as OW
from paper_2603_11273_amd import synth

from gpu_util import TOL, cpu_params, make_context, needs_gpu, rel_err

pytestmark = [pytest.mark.gpu, needs_gpu]


@pytest.mark.parametrize("n_head,n_dec,batches", [
    (8, 1, [1, 2, 6]),       # 96, 192 and 568 tiles of 128 x 128
    (10, 1, [1]),            # 120
    (4, 2, [1, 3]),          # 96, 288
    (2, 1, [1, 3, 8]),       # 24, 72, 188
    (20, 2, [1, 8]),         # 480; 940 tiles of 256 x 256
])
def test_cross_cache(n_head, n_dec, batches):
    d, n = 64 * n_head, max(batches)
    shape = synth.ModelShape("cross", 80, d, 0, n_dec, n_head, 128, 100, "bf16")
    seed = 20260400 + n_head
    ctx = make_context(shape, seed, max_slots=n, max_prefill=n, max_decode=1)
    E = np.stack([synth.encoder_output(seed, b, d).numpy() for b in range(n)])
    P = cpu_params(shape, seed)
    ref = [np.stack([np.stack([x.reshape(1500, n_head, 64).transpose(1, 0, 2) for x in layer])
                     for layer in OW.cross_kv(E[b], P, n_dec)]) for b in range(min(n, 3))]
    first = {}
    for k in batches:
        slots = list(range(n))[::-1][:k]                  # clip b in slot n - 1 - b
        ctx.debug_set_encoder_out(slots, [-1] * k, [40] * k, E[:k])
        for b in range(k):
            got = ctx.debug_get_kv(slots[b], 1)
            if b not in first:
                first[b] = got
            assert np.array_equal(got, first[b]), (k, b)
            if b < len(ref):
                for layer in range(n_dec):
                    for kv in range(2):
                        assert rel_err(got[layer, kv], ref[b][layer, kv]) <= TOL["bf16"], (k, b, layer, kv)
