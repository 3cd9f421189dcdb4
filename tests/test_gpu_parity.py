"""GPU parity of the SEED decode path against the CPU oracle (tiny models: every round).

fp32 model: logits within 1e-4 max-abs of the oracle; bf16 model (bf16 weights and KV cache):
within 2e-2. Tokens and acceptance lengths must match wherever the oracle's top-2 logit gap
exceeds twice the tolerance (elsewhere two answers are both within rounding)."""
import numpy as np
import pytest

from gpu_common import check_round, decoder, first_ambiguous, oracle_model, say
from oracle import seed as os_
from paper_2609_36590_amd import synth

pytestmark = pytest.mark.gpu

K = 4
WIDE = synth.C1_TINY.replace(name="wide-4L-h256-f8192", ffn=8192, n_heads=32, n_kv_heads=8, head_dim=128)
CASES = {
    # name: (config, enc_out_scale, tolerance)
    "tiny-f32": (synth.C1_TINY, 1.0, 1e-4),
    "tiny-f32-damped": (synth.C1_TINY, 0.1, 1e-4),
    "tiny-bf16": (synth.C1_TINY.replace(name="tiny-4L-h256-bf16", dtype=synth.BF16), 1.0, 2e-2),
    "tiny-bf16-damped": (synth.C1_TINY.replace(name="tiny-4L-h256-bf16", dtype=synth.BF16), 0.1, 2e-2),
    # a wide FFN and 32 query heads: a down projection of 16 k-ranges, which go to several workgroups and are
    # added by a second kernel, at 1, 5 and 7 rows
    "wide-f32": (WIDE, 1.0, 1e-4),
    "wide-bf16": (WIDE.replace(name="wide-4L-h256-f8192-bf16", dtype=synth.BF16), 1.0, 2e-2),
}


@pytest.fixture(scope="module", params=list(CASES))
def case(request):
    cfg, scale, tol = CASES[request.param]
    w = synth.make_weights(cfg, seed=0, enc_out_scale=scale)
    prompt = synth.make_prompts(cfg)[0]
    m = oracle_model(cfg, w)
    toks, rounds = os_.generate(m, prompt, K, cfg.gen_len, record=True)
    dec = decoder(cfg, w, max_batch=1, max_ctx=len(prompt) + cfg.gen_len + 2 * 6 + 2, max_draft=6)
    yield dict(name=request.param, cfg=cfg, w=w, prompt=prompt, toks=toks, rounds=rounds, tol=tol, dec=dec)
    dec.close()


def test_every_round_matches_oracle(case):
    """Teacher-forced from the oracle's own decode: each round's draft and verify logits."""
    worst_d = worst_v = 0.0
    for rd in case["rounds"]:
        say(f"[gpu] {case['name']} round p={rd.p}")
        dmax, vmax = check_round(case["dec"], case["prompt"], case["toks"], rd, case["tol"], K)
        worst_d, worst_v = max(worst_d, dmax), max(worst_v, vmax)
    say(f"[gpu] {case['name']}: max |draft - oracle| = {worst_d:.3g}, max |verify - oracle| = {worst_v:.3g}")
    assert worst_d <= case["tol"] and worst_v <= case["tol"]


def test_generate_matches_oracle_stream(case):
    rounds = case["rounds"]
    cfg = case["cfg"]
    n_ok = first_ambiguous(rounds, case["tol"])
    say(f"[gpu] {case['name']} generate k={K}; oracle rounds unambiguous: {n_ok}/{len(rounds)}")
    out, counts, st = case["dec"].generate([case["prompt"]], K, cfg.gen_len, log_cap=4 * cfg.gen_len)
    assert counts[0] == cfg.gen_len
    # tokens committed by the unambiguous oracle rounds must agree
    upto = (rounds[n_ok].p + 1 - len(case["prompt"])) if n_ok < len(rounds) else cfg.gen_len
    np.testing.assert_array_equal(out[0, :upto], case["toks"][:upto])
    log = st["n_accept_log"][:, 0]
    for i in range(n_ok):
        assert log[i] == rounds[i].n_accept, (i, log[i], rounds[i].n_accept)
    if upto == cfg.gen_len:
        assert st["rounds"] == len(rounds)


def test_speculative_equals_plain_greedy_bit_exact(case):
    """SEED (k=4) and plain greedy (k=0) through the same verify kernels give identical tokens."""
    cfg = case["cfg"]
    say(f"[gpu] {case['name']} k=0 vs k=4 vs k=6")
    g0, _, _ = case["dec"].generate([case["prompt"]], 0, cfg.gen_len)
    g4, _, _ = case["dec"].generate([case["prompt"]], 4, cfg.gen_len)
    g6, _, _ = case["dec"].generate([case["prompt"]], 6, cfg.gen_len)
    np.testing.assert_array_equal(g4, g0)
    np.testing.assert_array_equal(g6, g0)


def test_draft_is_idempotent(case):
    dec = case["dec"]
    dec.prefill([case["prompt"]])
    d1, q1 = dec.draft(K, logits=True)
    d2, q2 = dec.draft(K, logits=True)
    np.testing.assert_array_equal(d1, d2)
    np.testing.assert_array_equal(q1, q2)
