"""GPU parity at the full workload sizes, in the launch configuration the benchmark times.

* 28L-h2048 (prompt 512) and 4B-36L-h2560 (prompt 1024): the first draft-verify round against the
  oracle, every draft and verify logit row within 2e-2 max-abs (bf16 weights and KV cache), the
  drafted tokens, n_accept and the bonus token where the oracle's top-2 gap exceeds twice that;
  then the speculative decode (k=4) is bit-exact to the GPU's own plain greedy decode (k=0).
* 4B at batch 8 with ragged prompt lengths (uniform in [256, 2048]): every sequence's first round
  against the oracle inside the batch (one batched draft and one batched verification of the
  oracle's drafts, 40 rows), and every sequence's batched decode bit-exact to the same sequence
  decoded alone and to plain greedy decoding.
* 28L-h2048 and 4B-36L-h2560, three consecutive rounds from one prefill (the second with drafts
  forced to the oracle's greedy continuation, so it accepts all four and the third round's drafter
  reads decoder-layer keys/values that a verification wrote): every round's draft and verify
  logits against the oracle, which commits what the GPU committed (teacher forcing).
* 4B with a 16384-token prompt, first round against the oracle's stored round
  (tests/golden/c5_first_round.npz, written by tests/golden/make_c5_first_round.py, which calls
  only the oracle and the seeded generators): draft logits and verify logits of the oracle's drafts
  element by element within 2e-2, n_accept and bonus where the top-2 gaps allow.
* 4B with a 16384-token prompt: the oracle cannot follow a 16k-token prefill through all 36
  layers within a test's time. It forms the first two layers' keys/values at sampled positions one
  position at a time (layer 1's need one row of layer 0 attending to the whole prefix), and
  those are compared with the GPU's cache after prefill and one verification: prefill rows and
  the verification rows at positions 16383..16387, whose layer-1 entries pass through the
  decode attention over the 16k-token cache. Beyond that, properties that hold at any size:
  the speculative decode equals plain greedy decoding bit for bit, and every verify logit is
  finite. The batch-8 case gets the same sampled cache check for its longest sequence.

The oracle runs in float32 on the host; its inputs come from ``synth`` only.
"""
import hashlib
import os

import numpy as np
import pytest

from gpu_common import GPU_ROWS, compare_kv, decoder, oracle_model, say, top2_gap
from oracle import model as om
from oracle import seed as os_
from paper_2609_36590_amd import synth

pytestmark = [pytest.mark.gpu, pytest.mark.slow]

K = 4
TOL = 2e-2
N_NEW = 24


@pytest.fixture(scope="module")
def weights_4b():
    say("[gpu] generating 4B-36L-h2560 weights (seed 0)")
    w = synth.make_weights(synth.C3_4B, seed=0)
    yield w


def oracle_first_round(cfg, w, prompt, m=None):
    say(f"[gpu] oracle prefill {cfg.name} over {len(prompt)} tokens")
    m = m if m is not None else oracle_model(cfg, w)
    st = os_.prefill(m, prompt, capacity=len(prompt) + K + 2)
    drafts, qlog = os_.draft(st, K)
    plog = os_.verify(st, drafts)
    n, bonus = os_.accept(drafts, plog)
    say(f"[gpu] oracle round: drafts {drafts.tolist()} n_accept {n} bonus {bonus}")
    return os_.Round(st.p, drafts, qlog, plog, n, bonus)


def compare_round(rd, d, qlog, na, bo, vlog):
    """GPU round (drafts d [K], draft logits [K, V], verify logits [K+1, V] from the oracle's drafts)
    against the oracle round rd."""
    derr = float(np.abs(qlog[0] - rd.draft_logits[0]).max())
    for i in range(1, K):
        if not np.array_equal(d[:i], rd.drafts[1:i + 1]):
            break
        derr = max(derr, float(np.abs(qlog[i] - rd.draft_logits[i]).max()))
    for i in range(K):
        if top2_gap(rd.draft_logits[i]) > 2 * TOL and np.array_equal(d[:i], rd.drafts[1:i + 1]):
            assert d[i] == rd.drafts[i + 1], (i, d, rd.drafts)
    verr = float(np.abs(vlog - rd.verify_logits).max())
    say(f"[gpu] max |draft - oracle| = {derr:.3g}, max |verify - oracle| = {verr:.3g}")
    assert derr <= TOL and verr <= TOL
    if np.all(top2_gap(rd.verify_logits) > 2 * TOL):
        assert na == rd.n_accept and bo == rd.bonus, (na, rd.n_accept, bo, rd.bonus)


def check_sampled_kv(cfg, w, dec, b, tokens, positions, m=None):
    """Layers 0 and 1 of sequence b's cache at ``positions`` against the oracle's, formed one
    position at a time from ``tokens`` (the committed prefix and the verified drafts)."""
    m = m if m is not None else oracle_model(cfg, w)
    say(f"[gpu] oracle layer-0/1 keys/values at {len(positions)} positions of {len(tokens)} tokens")
    ref = om.sampled_kv_first_layers(m, tokens, positions)
    for layer in (0, 1):
        got_k = np.stack([dec.read_kv(b, layer, j, 1)[0][0] for j in positions])
        got_v = np.stack([dec.read_kv(b, layer, j, 1)[1][0] for j in positions])
        compare_kv(got_k, ref[2 * layer], True, what=f"layer {layer} keys")
        compare_kv(got_v, ref[2 * layer + 1], True, what=f"layer {layer} values")


def spec_equals_greedy(dec, prompts):
    out4, c4, _ = dec.generate(prompts, K, N_NEW, use_graph=True)
    out0, c0, _ = dec.generate(prompts, 0, N_NEW, use_graph=True)
    assert np.all(c4 == N_NEW) and np.all(c0 == N_NEW)
    np.testing.assert_array_equal(out4, out0)
    return out4


@pytest.mark.timeout(900)
@pytest.mark.parametrize("cfg", [synth.C2_28L, synth.C3_4B], ids=["28L-h2048", "4B-36L-h2560"])
def test_first_round_matches_oracle_at_full_size(cfg, request):
    w = request.getfixturevalue("weights_4b") if cfg is synth.C3_4B else synth.make_weights(cfg, seed=0)
    prompt = synth.make_prompts(cfg)[0]
    assert len(prompt) == cfg.prompt_len
    dec = decoder(cfg, w, max_batch=1, max_ctx=cfg.prompt_len + cfg.gen_len + 2 * K + 2, max_draft=K)
    try:
        dec.prefill([prompt])
        d, qlog = dec.draft(K, logits=True)
        rd = oracle_first_round(cfg, w, prompt)
        dec.prefill([prompt])
        na, bo, vlog = dec.verify(K, drafts=np.asarray(rd.drafts[1:], dtype=np.int32)[None], logits=True)
        compare_round(rd, d[0], qlog[0], int(na[0]), int(bo[0]), vlog[0])
        say(f"[gpu] {cfg.name}: generate {N_NEW} tokens, k={K} vs k=0")
        out = spec_equals_greedy(dec, [prompt])
        # the first round commits n_accept drafts and the bonus token
        if np.all(top2_gap(rd.verify_logits) > 2 * TOL):
            first = list(rd.drafts[1:rd.n_accept + 1]) + [rd.bonus]
            np.testing.assert_array_equal(out[0, :len(first)], first)
    finally:
        dec.close()


def greedy_continuation(st, n):
    """The next n tokens of plain greedy decoding from the oracle state st (each from one more
    verification pass; the state's committed tokens are left as they are)."""
    out = []
    for _ in range(n):
        plog = os_.verify(st, np.asarray([st.tokens[-1]] + out + [0] * (n - len(out)), dtype=np.int64))
        out.append(int(np.argmax(plog[len(out)])))
    st.cache.truncate(st.t - 1)
    return out


@pytest.mark.timeout(900)
@pytest.mark.parametrize("cfg", [synth.C2_28L, synth.C3_4B], ids=["28L-h2048", "4B-36L-h2560"])
def test_three_rounds_match_oracle_at_full_size(cfg, request):
    w = request.getfixturevalue("weights_4b") if cfg is synth.C3_4B else synth.make_weights(cfg, seed=0)
    prompt = synth.make_prompts(cfg)[0]
    dec = decoder(cfg, w, max_batch=1, max_ctx=cfg.prompt_len + 3 * (K + 1) + 2 * K + 2, max_draft=K)
    m = oracle_model(cfg, w)
    try:
        say(f"[gpu] oracle prefill {cfg.name} over {len(prompt)} tokens")
        st = os_.prefill(m, prompt, len(prompt) + 3 * (K + 1) + K + 2)
        dec.prefill([prompt])
        accepted = []
        for r in range(3):
            d, qlog = dec.draft(K, logits=True)
            drafts, qref = os_.draft(st, K)
            if r == 1:
                drafts = np.asarray([st.tokens[-1]] + greedy_continuation(st, K), dtype=np.int64)
            plog = os_.verify(st, drafts)
            n, bonus = os_.accept(drafts, plog)
            na, bo, vlog = dec.verify(K, drafts=np.asarray(drafts[1:], dtype=np.int32)[None], logits=True)
            say(f"[gpu] {cfg.name} round {r} at p={st.p}: drafts {drafts[1:].tolist()} n_accept {int(na[0])} "
                f"(oracle {n}), bonus {int(bo[0])} (oracle {bonus})")
            # draft rows compare with the oracle drafter's own drafts; the verify rows, n_accept and
            # bonus with the verification of the drafts actually verified
            own = np.asarray([st.tokens[-1]] + [int(x) for x in np.argmax(qref, axis=1)], dtype=np.int64)
            compare_round(os_.Round(st.p, own, qref, plog, n, bonus), d[0], qlog[0], int(na[0]), int(bo[0]), vlog[0])
            if r == 1 and np.all(top2_gap(plog) > 2 * TOL):
                assert int(na[0]) == K     # the greedy continuation is accepted whole
            os_.commit(st, drafts, int(na[0]), int(bo[0]))   # the oracle commits what the GPU committed
            accepted.append(int(na[0]))
        np.testing.assert_array_equal(dec.tokens(0), st.tokens)
        say(f"[gpu] {cfg.name}: accepted per round {accepted}")
    finally:
        dec.close()


GOLDEN_C5 = os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden", "c5_first_round.npz")


@pytest.mark.timeout(900)
def test_long_context_first_round_matches_stored_oracle(weights_4b):
    cfg = synth.C5_4B_LONG
    g = np.load(GOLDEN_C5)
    prompt = synth.make_prompts(cfg)[0]
    assert str(g["config"]) == cfg.name
    assert hashlib.sha256(np.asarray(prompt, dtype=np.int32).tobytes()).hexdigest() == str(g["prompt_sha256"])
    rd = os_.Round(int(g["p"]), g["drafts"], g["draft_logits"], g["verify_logits"], int(g["n_accept"]), int(g["bonus"]))
    assert rd.p == len(prompt) - 1
    dec = decoder(cfg, weights_4b, max_batch=1, max_ctx=len(prompt) + N_NEW + 2 * K + 2, max_draft=K)
    try:
        say("[gpu] 16k prefill, first round against the stored oracle round")
        dec.prefill([prompt])
        d, qlog = dec.draft(K, logits=True)
        dec.prefill([prompt])
        na, bo, vlog = dec.verify(K, drafts=np.asarray(rd.drafts[1:], dtype=np.int32)[None], logits=True)
        compare_round(rd, d[0], qlog[0], int(na[0]), int(bo[0]), vlog[0])
    finally:
        dec.close()


@pytest.mark.timeout(900)
def test_batch8_ragged_matches_alone_greedy_and_oracle(weights_4b):
    cfg = synth.C4_4B_B8
    lens = synth.make_prompt_lengths(cfg)
    prompts = synth.make_prompts(cfg, lengths=lens)
    say(f"[gpu] batch of {len(prompts)} ragged prompts, lengths {lens}")
    ctx = max(lens) + N_NEW + 2 * K + 2
    dec = decoder(cfg, weights_4b, max_batch=cfg.batch, max_ctx=ctx, max_draft=K)
    try:
        # every sequence's first round, inside the batch, against the oracle: one batched draft,
        # then (after a fresh prefill) one batched verification of the oracle's drafts
        dec.prefill(prompts)
        d, qlog = dec.draft(K, logits=True)
        m = oracle_model(cfg, weights_4b)
        rds = [oracle_first_round(cfg, weights_4b, p, m) for p in prompts]
        dec.prefill(prompts)
        drafts = np.stack([rd.drafts[1:] for rd in rds]).astype(np.int32)
        na, bo, vlog = dec.verify(K, drafts=drafts, logits=True)
        for b, rd in enumerate(rds):
            say(f"[gpu] sequence {b} (len {lens[b]}) first round against the oracle")
            compare_round(rd, d[b], qlog[b], int(na[b]), int(bo[b]), vlog[b])
        bl = int(np.argmax(lens))
        pl = lens[bl] - 1
        check_sampled_kv(cfg, weights_4b, dec, bl, np.concatenate([prompts[bl], drafts[bl]]),
                         [0, 17, pl // 2, pl - 1] + list(range(pl, pl + K + 1)), m=m)
        del m
        say(f"[gpu] batch generate {N_NEW} tokens each, k={K}")
        out_b, cnt, _ = dec.generate(prompts, K, N_NEW, use_graph=True)
        assert np.all(cnt == N_NEW)
    finally:
        dec.close()
    solo = decoder(cfg, weights_4b, max_batch=1, max_ctx=ctx, max_draft=K)
    try:
        for i, p in enumerate(prompts):
            say(f"[gpu] sequence {i} alone (len {len(p)}): k={K} and k=0")
            out_s = spec_equals_greedy(solo, [p])
            np.testing.assert_array_equal(out_b[i], out_s[0])
    finally:
        solo.close()


@pytest.mark.timeout(900)
def test_long_context_16k_spec_equals_greedy(weights_4b):
    cfg = synth.C5_4B_LONG
    prompt = synth.make_prompts(cfg)[0]
    assert len(prompt) == 16384
    dec = decoder(cfg, weights_4b, max_batch=1, max_ctx=len(prompt) + N_NEW + 2 * K + 2, max_draft=K)
    try:
        say("[gpu] 16k prefill + first round")
        dec.prefill([prompt])
        d, _ = dec.draft(K)
        _, _, vlog = dec.verify(K, logits=True)
        assert np.all(np.isfinite(vlog))
        p = len(prompt) - 1
        check_sampled_kv(cfg, weights_4b, dec, 0, np.concatenate([prompt, d[0]]),
                         [0, 15, 16, 4095, 8192, 12289, p - 1] + list(range(p, p + K + 1)))
        say(f"[gpu] 16k: generate {N_NEW} tokens, k={K} vs k=0")
        spec_equals_greedy(dec, [prompt])
    finally:
        dec.close()


@pytest.mark.timeout(900)
def test_spec_forward_28l_matches_oracle():
    """Forward pass of the speculative drafting objective (Algorithm 1) on the 28-layer model, a
    512-token sequence, block size 4: every row's drafter logits within 2e-2 of the oracle."""
    cfg = synth.C2_28L
    w = synth.make_weights(cfg, seed=0)
    x = synth.make_prompts(cfg)[0]
    dec = decoder(cfg, w, max_batch=1, max_ctx=len(x) + 8, max_draft=K)
    try:
        lg, nll, loss = dec.spec_forward(x, 4)
    finally:
        dec.close()
    say(f"[gpu] oracle spec forward {cfg.name} over {len(x)} tokens")
    ref, ref_loss = os_.spec_forward(oracle_model(cfg, w), x, 4)
    err = float(np.abs(lg - ref).max())
    say(f"[gpu] max |logits - oracle| = {err:.3g}; L_spec {loss:.6g} vs {ref_loss:.6g}")
    assert err <= TOL
    assert abs(loss - ref_loss) <= 2 * TOL * (len(x) - 1)


@pytest.mark.timeout(900)
def test_tree_round_matches_oracle_at_full_size(weights_4b):
    """Dynamic drafting and tree verification on the 4B model after the 1024-token prefill: the
    first step's drafter logits and p0 against the oracle's, the drafted tree where no decision is
    near a boundary; then a 31-node tree (depth 3, fan-out 10: the row kernels of two token tiles and
    the chunked head) verified by the GPU, every node's logits within 2e-2 of the oracle's tree verification,
    path and bonus where the visited nodes' top-2 gaps leave no doubt; finally tree decoding commits
    the GPU's plain greedy tokens."""
    from oracle import tree as ot
    from paper_2609_36590_amd import binding
    cfg = synth.C3_4B
    w = weights_4b
    prompt = synth.make_prompts(cfg)[0]
    dec = decoder(cfg, w, max_batch=1, max_ctx=len(prompt) + N_NEW + 2 * 65 + 2, max_draft=K)
    m = oracle_model(cfg, w)
    try:
        dec.prefill([prompt])
        toks, par, p0, dlog = dec.draft_tree(binding.tree_opts(K), logits=True)
        say(f"[gpu] oracle prefill {cfg.name} over {len(prompt)} tokens")
        st = os_.prefill(m, prompt, len(prompt) + 70)
        tree = ot.draft_tree(st, 0.7, K, max_nodes=GPU_ROWS)
        derr = float(np.abs(dlog[0] - tree.draft_logits[0]).max())
        say(f"[gpu] step 1: p0 {p0[0]:.4g} vs {tree.p0[0]:.4g}, max |draft - oracle| = {derr:.3g}, "
            f"{len(toks)} vs {len(tree.tokens)} nodes")
        assert derr <= TOL and abs(p0[0] - tree.p0[0]) <= 4 * TOL * tree.p0[0] + 1e-6
        top = np.sort(tree.draft_logits[0].astype(np.float64))[::-1][:11]
        if len(tree.p0) == 1 and np.all(-np.diff(top) > 2 * TOL) and min(
                abs(tree.p0[0] - x) for x in (0.95, 0.8, 0.5, 0.7)) > 4 * TOL:
            assert toks == tree.tokens and par == tree.parents
        # a wide tree through the GPU's verification (drafting again from the committed prefix)
        st.cache.truncate(st.t - 1)
        wide = ot.draft_tree(st, 0.0, 3, max_nodes=GPU_ROWS)
        assert len(wide.tokens) == 31
        logits, _ = ot.verify_tree(st, wide)
        path, bonus = ot.accept_tree(wide, logits)
        dec.prefill([prompt])
        gpath, gbonus, glog = dec.verify_tree(wide.tokens, wide.parents, logits=True)
        verr = float(np.abs(glog - logits).max())
        say(f"[gpu] 31-node tree: max |verify - oracle| = {verr:.3g}; path {gpath} vs {path}")
        assert verr <= TOL
        visited = [0] + list(path)
        if np.all(top2_gap(logits[visited]) > 2 * TOL):
            assert gpath == path and gbonus == bonus
        say(f"[gpu] {cfg.name}: tree decoding of {N_NEW} tokens vs plain greedy")
        out0, _, _ = dec.generate([prompt], 0, N_NEW, use_graph=True)
        out_t, _ = dec.generate_tree(prompt, binding.tree_opts(K), N_NEW, use_graph=True)
        np.testing.assert_array_equal(out_t, out0[0])
    finally:
        dec.close()
