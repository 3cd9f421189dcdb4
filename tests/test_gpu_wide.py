"""The tiled GEMM of passes of more than 64 rows (wide.hip) at the edges of its tiles, against the
oracle: row counts one around a token tile, a workgroup's 64 rows and the narrow passes' 64-row limit;
one, two and odd numbers of k-tiles (one k-tile cannot split K); and, with more rows and features, every
number of n-tiles per wave that the launch rule picks, in feature counts that leave a wave or a workgroup partly
empty (test_dispatch.py checks that these shapes pick them all), with a ragged second block of 1024 rows.
With n_dec = l the drafting objective's pass with one block over the sequence is the full causal model, so
its logits go through every projection and the LM head of both wide passes (the prefill and the objective's
own). Tolerances are those of the logits everywhere: 1e-4 fp32, 2e-2 bf16.
"""
import numpy as np
import pytest

from gpu_common import decoder, oracle_model, say
from oracle import seed as os_
from paper_2609_36590_amd import synth

pytestmark = pytest.mark.gpu

BASE = synth.C1_TINY.replace(n_layers=2, n_dec_layers=2, k=2)
SHAPES = {
    "one-k-tile": dict(hidden=32, n_heads=1, n_kv_heads=1, head_dim=64, ffn=32, vocab=16),
    "odd": dict(hidden=96, n_heads=3, n_kv_heads=1, head_dim=64, ffn=160, vocab=592),
    "grouped": dict(hidden=224, n_heads=4, n_kv_heads=2, head_dim=128, ffn=352, vocab=2320),
}

# hidden, query heads, KV heads, ffn, vocabulary, rows of the pass (heads of 64)
MANY_TILES = ((928, 8, 4, 224, 2688, 2500), (224, 2, 1, 544, 336, 2090), (1408, 2, 2, 832, 656, 2500),
              (32, 1, 1, 3008, 4000, 1037), (32, 4, 1, 3424, 1408, 1500), (32, 1, 1, 320, 5040, 2090),
              (2080, 2, 1, 288, 112, 2500))


@pytest.mark.parametrize("hidden,heads,kv,ffn,vocab,rows", MANY_TILES)
def test_every_width_of_a_wave(hidden, heads, kv, ffn, vocab, rows):
    cfg = BASE.replace(name="wide-tiles", dtype=synth.BF16, hidden=hidden, n_heads=heads, n_kv_heads=kv, head_dim=64,
                       ffn=ffn, vocab=vocab)
    w = synth.make_weights(cfg, seed=3)
    x = synth.make_prompts(cfg.replace(prompt_len=rows + 1), seed=5)[0]
    ref, _ = os_.spec_forward(oracle_model(cfg, w), x, rows + 1)
    dec = decoder(cfg, w, max_batch=1, max_ctx=rows + 8, max_draft=2)
    try:
        say(f"[gpu] wide pass of {rows} rows, hidden {hidden} ffn {ffn} vocab {vocab}")
        lg, _, _ = dec.spec_forward(x, rows + 1)
        err = float(np.abs(lg - ref).max())
        say(f"[gpu]   max |logits - oracle| = {err:.3g}")
        assert np.all(np.isfinite(lg)) and err <= 2e-2
    finally:
        dec.close()


@pytest.mark.parametrize("dtype,tol", [(synth.F32, 1e-4), (synth.BF16, 2e-2)], ids=["f32", "bf16"])
@pytest.mark.parametrize("shape", SHAPES)
def test_wide_pass_edges(shape, dtype, tol):
    cfg = BASE.replace(name="wide-" + shape, dtype=dtype, **SHAPES[shape])
    w = synth.make_weights(cfg, seed=3)
    m = oracle_model(cfg, w)
    sizes = (66, 67, 81, 129, 130, 194)
    x = synth.make_prompts(cfg.replace(prompt_len=max(sizes)), seed=5)[0]
    dec = decoder(cfg, w, max_batch=1, max_ctx=max(sizes) + 8, max_draft=2)
    try:
        for n in sizes:   # n tokens: passes of n - 1 rows
            say(f"[gpu] wide pass {shape} {dtype} rows={n - 1}")
            ref, _ = os_.spec_forward(m, x[:n], n)
            lg, _, _ = dec.spec_forward(x[:n], n)
            err = float(np.abs(lg - ref).max())
            say(f"[gpu]   max |logits - oracle| = {err:.3g}")
            assert np.all(np.isfinite(lg)) and err <= tol
    finally:
        dec.close()


def test_logits_of_any_alignment():
    """Logits go out 16 bytes at a time when the caller's buffer allows it, else 4."""
    import torch

    from paper_2609_36590_amd import binding

    cfg = BASE.replace(name="wide-odd", dtype=synth.BF16, **SHAPES["odd"])
    w = synth.make_weights(cfg, seed=3)
    x = synth.make_prompts(cfg.replace(prompt_len=90), seed=5)[0]
    dec = decoder(cfg, w, max_batch=1, max_ctx=100, max_draft=2)
    try:
        ref, _, _ = dec.spec_forward(x, 4)
        skv = torch.empty(binding.seed_spec_kv_bytes(dec.cfg), dtype=torch.uint8, device="cuda")
        buf = torch.full((89 * cfg.vocab + 8,), float("nan"), device="cuda")
        binding.seed_spec_forward(dec.ctx, x, 4, skv.data_ptr(), buf.data_ptr() + 4, None, False)
        got = buf.cpu().numpy()
        np.testing.assert_array_equal(got[1:1 + 89 * cfg.vocab].reshape(89, -1), ref)
        assert np.all(np.isnan(got[1 + 89 * cfg.vocab:])) and np.isnan(got[0])
    finally:
        dec.close()
