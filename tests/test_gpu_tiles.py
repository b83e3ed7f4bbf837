"""GEMM tile choice: a row's result does not depend on the tile its batch
size selects.

One question alone runs on the smallest tiles, the same question inside a
batch on larger ones, and every tile adds the same products in the same order,
so the scores agree bit for bit. Prefix lengths sit at and around tile edges;
the widths give K loops of a few steps (one too short for some tiles' rings)
and column remainders. The batch is checked against the fp64 oracle.
"""
import numpy as np
import pytest

import jet_synth
import oracle
from paper_2609_33874_amd import jet as J

pytestmark = pytest.mark.gpu

DENSE = dict(arch="dense", n_layers=2, n_heads=6, n_kv_heads=2, head_dim=128, vocab=1100, max_ctx=1024)
CASES = {
    "f16": (dict(DENSE, dtype="bf16", d_model=768, ffn=1088), J.JET_F16),
    "f16_short_k": (dict(DENSE, dtype="bf16", d_model=320, ffn=448), J.JET_F16),
    # 256x256 tiles: two and three K steps of 64 columns, residual add, RoPE, SwiGLU
    "f16_wide": (dict(DENSE, dtype="bf16", d_model=4096, ffn=128), J.JET_F16),
    "f16_wide_ffn": (dict(DENSE, dtype="bf16", d_model=192, ffn=2112), J.JET_F16),
    "bf16_pair_wide": (dict(DENSE, dtype="bf16", d_model=4096, ffn=128), J.JET_BF16),
    "bf16_pair_wide_ffn": (dict(DENSE, dtype="bf16", d_model=192, ffn=2112), J.JET_BF16),
    "f16_pair_wide": (dict(DENSE, dtype="bf16", d_model=4096, ffn=128), J.JET_F16P),
    "bf16_pair": (dict(DENSE, dtype="bf16", d_model=768, ffn=1088), J.JET_BF16),
    "f16_pair": (dict(DENSE, dtype="bf16", d_model=768, ffn=1088), J.JET_F16P),
    "q8": (dict(DENSE, dtype="q8", d_model=768, ffn=1024), J.JET_F16),
    "q4": (dict(DENSE, dtype="q4", d_model=768, ffn=1024), J.JET_F16),
    # the narrowest block-quantized models: no fused QKV tile runs K = 128
    "q8_narrow": (dict(DENSE, dtype="q8", d_model=128, ffn=192), J.JET_F16),
    "q4_narrow": (dict(DENSE, dtype="q4", d_model=128, ffn=192), J.JET_F16),
    # the attention kernel of the smaller heads: items of 64 and of 128 query slots
    "f16_head64": (dict(DENSE, dtype="bf16", d_model=256, ffn=320, head_dim=64), J.JET_F16),
    "f16_head32": (dict(DENSE, dtype="bf16", d_model=256, ffn=320, head_dim=32), J.JET_F16),
    "bf16_single_head64": (dict(DENSE, dtype="bf16", d_model=256, ffn=320, head_dim=64), J.JET_BF16_SINGLE),
    "hybrid_pair": (dict(DENSE, arch="hybrid", n_layers=4, dtype="bf16", d_model=640, ffn=832, gdn_heads=5,
                         gdn_dk=128, gdn_dv=128, conv_kernel=4), J.JET_BF16),
    # the stepwise recurrence over prefixes (chunks of 32 steps)
    "hybrid_fp32": (dict(DENSE, arch="hybrid", n_layers=4, dtype="f32", d_model=256, ffn=320, gdn_heads=2,
                         gdn_dk=128, gdn_dv=128, conv_kernel=4), J.JET_FP32),
    # routed experts: segments of a few rows, of tens and of hundreds (the
    # oracle is left out: a rounding difference may swap experts of equal logit)
    "experts": (dict(DENSE, dtype="bf16", d_model=512, ffn=512, n_experts=16, top_k=2, moe_ffn=512, shared_ffn=512),
                J.JET_F16),
    # ... and a gate/up product on the 256-row tiles of four waves
    "experts_wide": (dict(DENSE, dtype="bf16", d_model=1024, ffn=512, n_experts=16, top_k=2, moe_ffn=512,
                          shared_ffn=512), J.JET_F16),
    # 128x128 and 256x256 tiles of int8 / int4 weights where no small tile runs K
    "q8_odd_k": (dict(DENSE, dtype="q8", d_model=384, ffn=960), J.JET_F16),
    "q4_odd_k": (dict(DENSE, dtype="q4", d_model=384, ffn=960), J.JET_F16),
    "experts_hybrid": (dict(DENSE, arch="hybrid", n_layers=4, dtype="bf16", d_model=512, ffn=512, n_experts=16,
                            top_k=2, moe_ffn=512, shared_ffn=512, gdn_heads=2, gdn_dk=128, gdn_dv=128,
                            conv_kernel=4), J.JET_F16),
}
PREFIX = [1, 2, 15, 16, 17, 31, 33, 63, 64, 65, 127, 129, 200, 257, 300]


@pytest.mark.parametrize("case", list(CASES))
def test_scores_do_not_depend_on_the_tile(case, tmp_path):
    spec, mode = CASES[case]
    path = str(tmp_path / "m.jetm")
    jet_synth.write_model(path, spec)
    g = np.random.Generator(np.random.Philox(key=[3, len(case)]))
    pre = [g.integers(0, spec["vocab"], n).astype(np.int32) for n in PREFIX]
    cand = [[g.integers(0, spec["vocab"], m).astype(np.int32) for m in (1, 1 + q % 5, 9)] for q in range(len(pre))]
    few = jet_synth.from_lists(pre, cand)
    # the same questions again with 60 more, so that the batch has many tiles
    more = [g.integers(0, spec["vocab"], 280).astype(np.int32) for _ in range(60)]
    many = jet_synth.from_lists(pre + more, cand + [[y[:7] for y in more[q:q + 1]] for q in range(60)])
    m = J.jet_model_load(path, dtype=mode)
    try:
        def score(w):
            p = J.jet_prefill_prefix(m, w.prefix_offsets, w.prefix_tokens)
            out = J.jet_score_candidates(m, p, w.q_cand_offsets, w.cand_tok_offsets, w.cand_tokens)
            J.jet_prefix_free(p)
            return out

        tok, tot = score(few)
        tok_many, tot_many = score(many)
        np.testing.assert_array_equal(tok, tok_many[:len(tok)])
        np.testing.assert_array_equal(tot, tot_many[:len(tot)])
        for q in range(len(pre)):
            t1, s1 = score(jet_synth.from_lists(pre[q:q + 1], cand[q:q + 1]))
            c0, c1 = few.q_cand_offsets[q], few.q_cand_offsets[q + 1]
            np.testing.assert_array_equal(t1, tok[few.cand_tok_offsets[c0]:few.cand_tok_offsets[c1]], err_msg=f"{PREFIX[q]}")
            np.testing.assert_array_equal(s1, tot[c0:c1])
    finally:
        J.jet_model_free(m)
    if spec.get("n_experts"):
        return
    ref_tok, ref_sum = oracle.score_unshared(path, few)
    # the modes' tolerance per token and per candidate (of at most 9 tokens).
    # The (hi, lo) bf16 mode is held to fp32's: its error here is that of 32-bit
    # sums, and without the lo planes it would be bf16's, 3e-3 and more.
    precise = mode in (J.JET_FP32, J.JET_BF16)
    t_tol, s_tol = (1e-4, 9e-4) if precise else (2e-2, 5e-2)
    err = np.max(np.abs(tok - ref_tok))
    print(f"[tiles] {case}: max|d tok|={err:.3e}", flush=True)
    assert err <= t_tol
    assert np.max(np.abs(tot - ref_sum)) <= s_tol


# Candidates' own rows in tiles of 64 (one row short of, exactly, and past a
# tile and two), the short ones beside them; many: questions whose rows with one
# query head per KV head fill items of 128 query slots past row 64.
OWN = [1, 64, 65, 66, 2, 129, 130, 9, 200]


@pytest.mark.parametrize("heads,kv_heads", [(4, 4), (6, 2)])
@pytest.mark.parametrize("mode", [J.JET_F16, J.JET_BF16_SINGLE, J.JET_BF16])
def test_long_candidates(heads, kv_heads, mode, tmp_path):
    spec = dict(DENSE, dtype="bf16", d_model=256, ffn=320, n_heads=heads, n_kv_heads=kv_heads)
    path = str(tmp_path / "m.jetm")
    jet_synth.write_model(path, spec)
    g = np.random.Generator(np.random.Philox(key=[5, heads]))
    pre = [g.integers(0, spec["vocab"], n).astype(np.int32) for n in [1, 63, 65, 130] * 8]
    cand = [[g.integers(0, spec["vocab"], m).astype(np.int32) for m in OWN[q % 9:] + OWN[:q % 9]]
            for q in range(len(pre))]
    rows = sum(len(y) - 1 for c in cand for y in c)
    assert rows * heads >= 128 * 128 and rows // len(pre) >= 96  # what items of 128 slots take
    m = J.jet_model_load(path, dtype=mode)
    try:
        def score(w):
            p = J.jet_prefill_prefix(m, w.prefix_offsets, w.prefix_tokens)
            out = J.jet_score_candidates(m, p, w.q_cand_offsets, w.cand_tok_offsets, w.cand_tokens)
            J.jet_prefix_free(p)
            return out

        wl = jet_synth.from_lists(pre, cand)
        tok, tot = score(wl)
        alone = []
        for q in range(4):  # one question: items of 64 slots; one candidate: one item per KV head
            t1, s1 = score(jet_synth.from_lists(pre[q:q + 1], cand[q:q + 1]))
            c0, c1 = wl.q_cand_offsets[q], wl.q_cand_offsets[q + 1]
            np.testing.assert_array_equal(t1, tok[wl.cand_tok_offsets[c0]:wl.cand_tok_offsets[c1]], err_msg=str(q))
            np.testing.assert_array_equal(s1, tot[c0:c1])
            alone.append(t1)
            for c in range(len(OWN)):
                t2, _ = score(jet_synth.from_lists(pre[q:q + 1], [cand[q][c:c + 1]]))
                a, b = wl.cand_tok_offsets[c0 + c], wl.cand_tok_offsets[c0 + c + 1]
                np.testing.assert_array_equal(t2, tok[a:b], err_msg=f"question {q}, {len(cand[q][c])} tokens")
    finally:
        J.jet_model_free(m)
    ref_tok, _ = oracle.score_unshared(path, jet_synth.from_lists(pre[:4], cand[:4]))
    err = np.max(np.abs(np.concatenate(alone) - ref_tok))
    print(f"[long] heads {heads}/{kv_heads} mode {mode}: max|d tok|={err:.3e}", flush=True)
    assert err <= (1e-4 if mode == J.JET_BF16 else 2e-2)


@pytest.mark.parametrize("mode,d,vocab", [
    (J.JET_F16, 320, 1100), (J.JET_BF16, 256, 1100),
    # 83 vocabulary splits: 700 rows are dealt to the XCDs in even bands
    (J.JET_F16, 320, 21000),
    # above 128 rows: tiles of eight waves up to 256 workgroups, of four from there
    (J.JET_F16, 2048, 40000), (J.JET_BF16_SINGLE, 2048, 40000)])
def test_lm_head_does_not_depend_on_the_rows(mode, d, vocab, tmp_path):
    """One-token candidates: the call is the LM head alone, one row each. 35,
    105, 210, 315 and 700 rows take its 64-, 128- and 256-row tiles."""
    path = str(tmp_path / "m.jetm")
    jet_synth.write_model(path, dict(arch="dense", dtype="bf16", n_layers=1, n_heads=1, n_kv_heads=1, head_dim=64,
                                     d_model=d, ffn=64, vocab=vocab, max_ctx=64))
    g = np.random.Generator(np.random.Philox(key=[7, d]))
    pre = [g.integers(0, vocab, 3 + q % 4).astype(np.int32) for q in range(20)]
    cand = [[y for y in g.integers(0, vocab, (35, 1)).astype(np.int32)] for _ in pre]
    m = J.jet_model_load(path, dtype=mode)
    try:
        def score(n):
            w = jet_synth.from_lists(pre[:n], cand[:n])
            p = J.jet_prefill_prefix(m, w.prefix_offsets, w.prefix_tokens)
            tok, _ = J.jet_score_candidates(m, p, w.q_cand_offsets, w.cand_tok_offsets, w.cand_tokens)
            J.jet_prefix_free(p)
            return tok

        tok = score(20)
        for n in (1, 3, 6, 9):
            np.testing.assert_array_equal(score(n), tok[:35 * n], err_msg=f"{35 * n} rows")
    finally:
        J.jet_model_free(m)
    ref, _ = oracle.score_unshared(path, jet_synth.from_lists(pre[:2], cand[:2]))
    assert np.max(np.abs(tok[:70] - ref)) <= (1e-4 if mode == J.JET_BF16 else 2e-2)
