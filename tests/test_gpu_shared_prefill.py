"""Prompts that share a prefill pass: every key and value the cache holds is bit for bit what the prompt's
own prefill writes, in every layer, whatever it shares the pass with: short prompts (their own narrow
pass), ragged ones around a token tile, one that needs a second pass, more rows than a pass holds.
"""
import numpy as np
import pytest

from gpu_common import decoder, say
from paper_2609_36590_amd import synth

pytestmark = pytest.mark.gpu

GROUPED = dict(hidden=96, n_heads=4, n_kv_heads=2, head_dim=128, ffn=160, vocab=256, n_layers=3, n_dec_layers=1)
ODD_GROUP = dict(GROUPED, n_heads=3, n_kv_heads=1, head_dim=64)   # the pass kernel does not take it: nothing is shared


@pytest.mark.parametrize("dtype", [synth.F32, synth.BF16])
@pytest.mark.parametrize("shape,lens", [
    (GROUPED, (70, 200, 40, 131, 66, 1, 67)),
    (GROUPED, (300, 4140, 90, 2000, 2100)),
    (ODD_GROUP, (70, 200, 40, 131)),
], ids=["ragged", "several-passes", "unshared"])
def test_cache_equals_the_prompt_alone(shape, lens, dtype):
    cfg = synth.C1_TINY.replace(name="shared-prefill", dtype=dtype, **shape)
    w = synth.make_weights(cfg, seed=2)
    g = np.random.default_rng(4)
    prompts = [g.integers(0, cfg.vocab, n).astype(np.int32) for n in lens]
    ctx = max(lens) + 8
    dec = decoder(cfg, w, max_batch=len(lens), max_ctx=ctx, max_draft=2)
    try:
        say(f"[gpu] shared prefill {dtype} lens={lens}")
        dec.prefill(prompts)
        together = [[dec.read_kv(b, layer, 0, n - 1) for layer in range(cfg.n_layers)] for b, n in enumerate(lens)]
        for b, n in enumerate(lens):
            dec.prefill([prompts[b]])
            for layer in range(cfg.n_layers):
                k, v = dec.read_kv(0, layer, 0, n - 1)
                np.testing.assert_array_equal(together[b][layer][0], k)
                np.testing.assert_array_equal(together[b][layer][1], v)
    finally:
        dec.close()
