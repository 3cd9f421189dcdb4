"""The attention of wide single-sequence passes (prefill and the drafting objective's decoder pass)
against the oracle, at its edges: row counts around a workgroup's row-block and a stage of 64 positions;
query groups of 1, 4, 8 and 32 heads; head sizes 64 and 128; enough row-blocks for the 128-vector
workgroups; a second pass whose positions are split over workgroups and merged (prompts longer than a
4096-row pass), with objective blocks that straddle the two passes. The objective's logits depend on both
variants: on the prefill's causal attention through the deep keys and values, and on the block-causal
one. Tolerances are those of the logits everywhere: 1e-4 fp32, 2e-2 bf16.
"""
import numpy as np
import pytest

from gpu_common import decoder, oracle_model, say
from oracle import seed as os_
from paper_2609_36590_amd import synth

pytestmark = pytest.mark.gpu

BASE = synth.C1_TINY.replace(n_layers=3, n_dec_layers=2, hidden=64, ffn=64, vocab=64, k=2)
TOL = {synth.F32: 1e-4, synth.BF16: 2e-2}


def _check(cfg, sizes, block):
    w = synth.make_weights(cfg, seed=11)
    m = oracle_model(cfg, w)
    x = synth.make_prompts(cfg.replace(prompt_len=max(sizes)), seed=13)[0]
    dec = decoder(cfg, w, max_batch=1, max_ctx=max(sizes) + 8, max_draft=2)
    try:
        for n in sizes:
            say(f"[gpu] pass attention {cfg.name} {cfg.dtype} rows={n - 1} block={block}")
            ref, _ = os_.spec_forward(m, x[:n], block)
            lg, _, _ = dec.spec_forward(x[:n], block)
            err = float(np.abs(lg - ref).max())
            say(f"[gpu]   max |logits - oracle| = {err:.3g}")
            assert np.all(np.isfinite(lg)) and err <= TOL[cfg.dtype]
    finally:
        dec.close()


@pytest.mark.parametrize("dtype", [synth.F32, synth.BF16])
@pytest.mark.parametrize("heads,kv,hd", [(2, 2, 64), (8, 2, 64), (8, 1, 128), (32, 1, 64)])
def test_row_blocks_and_stages(heads, kv, hd, dtype):
    cfg = BASE.replace(name=f"pass-{heads}-{kv}-{hd}", n_heads=heads, n_kv_heads=kv, head_dim=hd, dtype=dtype)
    _check(cfg, (66, 80, 81, 129, 130, 193), 7)


@pytest.mark.parametrize("hd", [64, 128])
def test_workgroups_of_128_vectors(hd):
    # 2 heads per KV head: 64 rows per workgroup, 32 row-blocks and a ragged one x 16 KV heads = 528
    cfg = BASE.replace(name=f"pass-wide-{hd}", n_layers=2, n_dec_layers=1, n_heads=32, n_kv_heads=16, head_dim=hd,
                       dtype=synth.BF16)
    _check(cfg, (2090,), 33)


@pytest.mark.parametrize("dtype", [synth.F32, synth.BF16])
def test_second_pass_splits_positions(dtype):
    # passes of 4096 and 103 rows; blocks of 30 cross row 4096
    cfg = BASE.replace(name="pass-split", n_layers=2, n_dec_layers=1, n_heads=4, n_kv_heads=1, head_dim=64, dtype=dtype)
    _check(cfg, (4200,), 30)


@pytest.mark.parametrize("dtype", [synth.F32, synth.BF16])
@pytest.mark.parametrize("heads,kv,n,at", [(4, 1, 200, 120), (32, 16, 2090, 1085)], ids=["64-vectors", "128-vectors"])
def test_rows_before_a_token_that_overflows(heads, kv, n, at, dtype):
    """A token whose embedding is not finite spoils its own row and what attends to it, and no earlier block of 16
    positions, although those rows share its 64-position stage (and, with 2 heads per KV head, its row-block of 64):
    their keys, values and logits are what the prompt has with any other token there. (fp32 row-blocks stream whole
    tiles up to their own last row: 32 rows with 2 heads per KV head.)"""
    cfg = BASE.replace(name="pass-overflow", n_heads=heads, n_kv_heads=kv, head_dim=64, dtype=dtype)
    w = synth.make_weights(cfg, seed=11)
    w["embed"][5] = np.float32("nan") if dtype == synth.F32 else 0x7FC0
    g = np.random.default_rng(3)
    x = g.integers(6, cfg.vocab, n).astype(np.int32)
    bad = x.copy()
    bad[at] = 5
    clean = at // 32 * 32 if dtype == synth.F32 and heads == 32 else at // 16 * 16
    dec = decoder(cfg, w, max_batch=1, max_ctx=n + 8, max_draft=2)
    try:
        got = []
        for t in (x, bad):
            say(f"[gpu] a token that overflows, {n} tokens, {dtype}")
            lg, _, _ = dec.spec_forward(t, 16)
            got.append([np.delete(lg[:clean], 5, axis=1)] + [dec.read_kv(0, i, 0, clean) for i in range(cfg.n_layers)])
        assert np.all(np.isfinite(got[0][0]))
        np.testing.assert_array_equal(got[0][0], got[1][0])
        for i in range(1, cfg.n_layers + 1):
            np.testing.assert_array_equal(got[0][i][0], got[1][i][0])
            np.testing.assert_array_equal(got[0][i][1], got[1][i][1])
    finally:
        dec.close()
