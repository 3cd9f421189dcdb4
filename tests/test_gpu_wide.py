"""The tiled GEMM of passes of more than 64 rows (wide.hip) at the edges of its tiles, against the
oracle: row counts one around a token tile, a workgroup's 64 rows and the narrow passes' 64-row limit;
feature counts that leave n-tiles of a wave or workgroup empty; one, two and odd numbers of k-tiles (one
k-tile cannot split K). With n_dec = l the drafting objective's pass with one block over the sequence is the
full causal model, so its logits go through every projection and the LM head of both wide passes (the
prefill and the objective's own). Tolerances are those of the logits everywhere: 1e-4 fp32, 2e-2 bf16.
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
