"""The linear kernels of decode passes (rows.hip, head.hip) at the edges of their tiles, against the oracle:
row counts around each token tile up to 64; features that leave n-tiles of a workgroup empty; K of one
k-tile, of odd numbers of them, and long enough that its ranges go to several workgroups (an odd number
of ranges among them); the head of small vocabularies and of ones from 32768 tokens on (rows staged
whole, and in chunks). Every verification's logits against the full forward of prompt and drafts.
Tolerances are those of the logits everywhere: 1e-4 fp32, 2e-2 bf16. And, bit for bit, every row of a
verification against the row computed alone by plain greedy decoding, across both activation layouts and every
variant and split of the kernels.
"""
import numpy as np
import pytest

from gpu_common import decoder, oracle_model, say
from oracle import model as om
from paper_2609_36590_amd import synth

pytestmark = pytest.mark.gpu

BASE = synth.C1_TINY.replace(n_layers=2, n_dec_layers=1)
SHAPES = {
    "one-k-tile": dict(hidden=32, n_heads=1, n_kv_heads=1, head_dim=64, ffn=32, vocab=16),
    # down: 145 k-tiles in 9 ranges; gate/up: 580 n-tiles
    "long-k": dict(hidden=96, n_heads=3, n_kv_heads=1, head_dim=64, ffn=4640, vocab=592),
    # QKV: 272 n-tiles of 9 k-tiles, O: 128 k-tiles; a head of 2049 n-tiles
    "heads": dict(hidden=288, n_heads=32, n_kv_heads=1, head_dim=128, ffn=8192, vocab=32784),
    # QKV (20 n-tiles) and gate/up (12) of 145 k-tiles: long K into a narrow N outside the residual projections
    "narrow-long-k": dict(hidden=4640, n_heads=3, n_kv_heads=1, head_dim=64, ffn=96, vocab=64),
}
ROWS = ((1, 0), (1, 4), (1, 15), (17, 0), (8, 3), (11, 2), (12, 3), (7, 6), (16, 3))   # sequences, drafts


@pytest.mark.parametrize("dtype,tol", [(synth.F32, 1e-4), (synth.BF16, 2e-2)], ids=["f32", "bf16"])
@pytest.mark.parametrize("shape", SHAPES)
def test_verification_rows(shape, dtype, tol):
    cfg = BASE.replace(name="rows-" + shape, dtype=dtype, **SHAPES[shape])
    w = synth.make_weights(cfg, seed=6)
    m = oracle_model(cfg, w)
    g = np.random.default_rng(8)
    for batch, k in ROWS:
        prompts = [g.integers(0, cfg.vocab, 2 + b % 5).astype(np.int32) for b in range(batch)]
        drafts = g.integers(0, cfg.vocab, (batch, k)).astype(np.int32)
        dec = decoder(cfg, w, max_batch=batch, max_ctx=32, max_draft=k)
        try:
            say(f"[gpu] rows {shape} {dtype} {batch} x {k + 1}")
            dec.prefill(prompts)
            _, _, lg = dec.verify(k, drafts=drafts if k else None, logits=True)
            err = 0.0
            for b in range(batch):
                ref = om.full_forward(m, np.concatenate([prompts[b], drafts[b]]))[len(prompts[b]) - 1:]
                err = max(err, float(np.abs(lg[b] - ref).max()))
            say(f"[gpu]   max |logits - oracle| = {err:.3g}")
            assert np.all(np.isfinite(lg)) and err <= tol
        finally:
            dec.close()


# shapes beyond those for the bit-for-bit comparison: a small vocabulary's head in 8 k-ranges (64 KB of partial sums
# at 64 rows); 5 n-tiles per workgroup in gate/up and in a down projection whose ranges go to several workgroups;
# the head with 5 n-tiles per wave
MORE = {
    "small-head": dict(hidden=288, n_heads=4, n_kv_heads=2, head_dim=64, ffn=800, vocab=1040),
    "five-tiles": dict(hidden=2400, n_heads=4, n_kv_heads=1, head_dim=64, ffn=8224, vocab=592),
    "wide-vocab": dict(hidden=64, n_heads=1, n_kv_heads=1, head_dim=64, ffn=64, vocab=81936),
}


@pytest.mark.parametrize("dtype", [synth.F32, synth.BF16])
@pytest.mark.parametrize("shape", list(SHAPES) + list(MORE))
def test_rows_equal_the_row_alone(shape, dtype):
    cfg = BASE.replace(name="rows-" + shape, dtype=dtype, **{**SHAPES, **MORE}[shape])
    w = synth.make_weights(cfg, seed=6)
    g = np.random.default_rng(9)
    prompts = [g.integers(0, cfg.vocab, 2 + b % 5).astype(np.int32) for b in range(17)]
    drafts = [g.integers(0, cfg.vocab, 15).astype(np.int32) for _ in range(17)]
    one = decoder(cfg, w, max_batch=1, max_ctx=32, max_draft=0)
    alone = {}

    def row(b, r):   # plain greedy decoding's step after prompt b and r of its drafts
        if (b, r) not in alone:
            one.prefill([np.concatenate([prompts[b], drafts[b][:r]])])
            alone[b, r] = one.verify(0, logits=True)[2][0, 0]
        return alone[b, r]

    try:
        for batch, k in ((1, 4), (1, 15), (17, 0), (8, 4), (16, 3)):   # 5, 16, 17, 40 and 64 rows
            dec = decoder(cfg, w, max_batch=batch, max_ctx=32, max_draft=k)
            try:
                say(f"[gpu] rows alone {shape} {dtype} {batch} x {k + 1}")
                dec.prefill(prompts[:batch])
                d = np.stack([drafts[b][:k] for b in range(batch)])
                _, _, lg = dec.verify(k, drafts=d if k else None, logits=True)
                for b in range(batch):
                    for r in range(k + 1):
                        np.testing.assert_array_equal(lg[b, r], row(b, r), err_msg=f"sequence {b} row {r}")
            finally:
                dec.close()
    finally:
        one.close()


@pytest.mark.parametrize("vocab", [16, 32784, 262160])
def test_argmax_over_many_groups(vocab):
    """Partial maxima of 1, 257 and 2049 vocabulary groups (one more than one pass over them holds); every
    13 tokens share their logits bit for bit, so the lowest id has to win across groups."""
    cfg = BASE.replace(name=f"argmax-{vocab}", hidden=32, n_heads=1, n_kv_heads=1, head_dim=64, ffn=32, vocab=vocab)
    w = synth.make_weights(cfg, seed=7)
    w["embed"] = np.ascontiguousarray(w["embed"][np.arange(vocab) % 13])
    dec = decoder(cfg, w, max_batch=2, max_ctx=32, max_draft=4)
    try:
        say(f"[gpu] argmax over {vocab} tokens")
        dec.prefill([np.arange(3, dtype=np.int32), np.arange(7, dtype=np.int32)])
        d, lg = dec.draft(4, logits=True)
        assert d.max() < 13
        assert np.array_equal(d, lg.argmax(-1))
    finally:
        dec.close()
