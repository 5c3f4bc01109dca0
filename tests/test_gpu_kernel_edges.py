"""Edges of single kernels, each against the CPU oracle through a whole step of a small shape.  `-m gpu`, MI355X."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

from oracle import cerberus_oracle as orc
from paper_2410_13344_amd import binding as B
from paper_2410_13344_amd import synth
from tests import harness as H


def _step_matches(pair, dtype, n_prompt, tol=None):
    cfg = pair.cfg
    taps, st = pair.taps(), pair.engine.new_state()
    ost = orc.prefill(cfg, pair.W, synth.make_token_ids(n_prompt, cfg["vocab"], seed=3).numpy(), capacity=pair.kv_capacity)
    ost["flag"] = 0
    H.round_oracle_kv(ost, dtype)
    H.upload_sequence(st, 0, ost, dtype)
    out = pair.oracle_step(ost)
    pair.engine.verify_step(st, 1)
    torch.cuda.synchronize()
    assert int(st.status[0]) == 0
    rep = H.compare_step(cfg, out, st, taps, 0, pair.T, dtype, ost, tol=tol)
    assert not rep.failures, "; ".join(rep.failures)


@pytest.mark.parametrize("tree,n_prompt,over", [
    ("root", 1, dict(d_ffn=8, vocab=16, topk=4)),                              # K of 8: fewer 16-column units than waves
    ("chain4", 15, dict(d_ffn=40, vocab=48)),                                  # K a multiple of 8, not of 16; one column tile past two
    ("rand17s1k4", 16, dict(d_model=64, n_heads=1, head_dim=64, d_ffn=264)),   # 17 rows: a row tile of one row; one head
    ("rand33s2k4", 63, dict(n_heads=2, head_dim=128, d_ffn=1000)),             # head size 128: two keys per wave
])
def test_fp32_kernels_at_the_edges_of_their_tiles(tree, n_prompt, over):
    print(f"fp32 step, tree {tree}, {n_prompt} committed rows, {over}", flush=True)
    if tree == "root":
        over = dict(over, n_cerb_heads=1, special_block=-1)
    pair = H.Pair("tiny", B.CERBERUS_F32, tree, seed=11, max_batch=1, kv_capacity=128, **over)
    _step_matches(pair, B.CERBERUS_F32, n_prompt)
    pair.engine.close()


@pytest.mark.parametrize("n_prompt,L0", [(193, 0), (256, 700), (384, 5), (385, 0), (420, 7), (576, 1), (700, 130), (1152, 0), (1153, 3)])
@pytest.mark.parametrize("dtype,attn_mfma", [(B.CERBERUS_F32, 0), (B.CERBERUS_BF16, 1), (B.CERBERUS_BF16, 0)])
def test_long_prompts_run_several_pieces_per_pass(dtype, attn_mfma, n_prompt, L0):
    """A prompt of more than one piece of 192 tokens goes through the layers in passes of up to six pieces: the cache
    rows, the pending token, the gate, the heads and the tapped rows (the last piece's, from slot 0) against the same prompt
    handed over piece by piece (each call a pass of its own).  Then the same with a cache that has room for the first half
    of the prompt and 24 rows (at least a piece): the pieces before the first one that does not fit are committed and nothing else, also where
    the prompt's last piece would fit, in the same pass or in a later one.  The pieces' operands are the same either way and only
    sums change order: fp32 5e-5; bf16 within the bars of a prompt of two passes (a different last bit flips the bf16
    rounding of a cached row now and then)."""
    print(f"prompt of {n_prompt} after {L0} rows, dtype={dtype}, attn_mfma={attn_mfma}", flush=True)
    P = B.CERBERUS_MAX_TREE
    tol = H.TOL_F32 if dtype == B.CERBERUS_F32 else H.TOL_BF16
    tokens = synth.make_token_ids(n_prompt, 1024, seed=5)
    pair = H.Pair("tiny", dtype, "p63", seed=2, max_batch=2, kv_capacity=1280, topk=6, entropy_threshold=float("inf"))
    pair.engine.set_param("attn_mfma", attn_mfma)
    base = pair.T                                      # taps: T rows per sequence, sequence 1
    n_last = (n_prompt - 1) % P + 1
    kept = ("root_token", "gate_flag", "entropy", "cand")

    def run(start, n_tokens, pieces):
        taps, st = pair.taps(), pair.engine.new_state()
        g = torch.Generator(device="cuda")
        g.manual_seed(1)
        for layer in st.kv:
            layer.normal_(0.0, 1.0, generator=g)
        st.kv_len.copy_(torch.tensor([17, start], dtype=torch.int32))
        st.gate_flag[:] = 1
        st.root_token[:], st.entropy[:], st.cand[:] = 7, 0.25, 9
        taps.node_token[:] = -5
        before = {k: getattr(st, k).clone() for k in kept}
        for i in range(0, n_tokens, pieces or n_tokens):
            pair.engine.prefill(st, 2, 1, tokens[i:min(i + (pieces or n_tokens), n_tokens)].cuda())
        torch.cuda.synchronize()
        return st, taps, before

    for start in (L0, 1280 - min(n_prompt - 1, max(P, n_prompt // 2 + 24))):
        fit = n_prompt if start + n_prompt <= 1280 else (1280 - start) // P * P     # rows of the pieces that fit
        got, gt, before = run(start, n_prompt, None)
        want, wt, _ = run(start, fit, P)
        n = start + fit
        assert (fit == n_prompt) == (start == L0) and 0 < fit
        assert got.kv_len.tolist() == want.kv_len.tolist() == [17, n]
        assert int(got.status[0]) == (0 if fit == n_prompt else B.CERBERUS_DEV_KV_OVERFLOW)
        assert torch.equal(got.kv[:, :, 0], want.kv[:, :, 0]) and torch.equal(got.kv[:, :, 1, :, n:], want.kv[:, :, 1, :, n:])
        mm = H.kv_mismatch(got.kv[:, :, 1, :, :n].double().cpu().numpy(), want.kv[:, :, 1, :, :n].double().cpu().numpy(), tol)
        assert mm is None, mm
        # the token of a slot is that of the latest piece which has a row there
        tail = n_last if fit == n_prompt else 0
        expect = [int(tokens[fit - tail + i]) if i < tail else int(tokens[fit - tail - P + i]) for i in range(pair.T)]
        assert gt.node_token.tolist() == [-5] * base + expect
        if fit < n_prompt:
            for name in kept:
                assert torch.equal(getattr(got, name), before[name]), name
            continue
        k = min(n_last, pair.T)
        assert float((gt.logits[base:base + k] - wt.logits[base:base + k]).abs().max()) <= tol.logits
        assert float((gt.h_last[base:base + k] - wt.h_last[base:base + k]).abs().max()) <= tol.hidden
        assert float((gt.head_logits[1] - wt.head_logits[1]).abs().max()) <= tol.logits
        assert abs(float(got.entropy[1]) - float(want.entropy[1])) <= tol.entropy
        assert got.gate_flag.tolist() == [1, 0] and torch.equal(got.cand[0], before["cand"][0])
        if k == n_last:                                # the last row is tapped
            top = wt.logits[base + k - 1].sort().values
            if float(top[-1] - top[-2]) > 2 * tol.logits:
                assert int(got.root_token[1]) == int(want.root_token[1])
    pair.engine.close()


@pytest.mark.parametrize("fused,team", [(1, 3), (0, 3), (0, 0)])   # the tile kernel, the team kernel, 64-row blocks
@pytest.mark.parametrize("n_prompt", [193, 256, 384, 385, 640, 1024, 1152])
def test_cache_rows_of_a_long_prompt_are_as_close_to_the_oracle_as_piece_by_piece(n_prompt, fused, team):
    """One layer of the 7B width (K = 4096): the cache rows are the QKV projection of the embeddings, whose products are exact
    in the hi and lo planes, so an element differs from the rounded oracle where the error of its fp32 sum crosses a
    rounding boundary, in proportion to that error.  In a pass of several pieces there are to be no more of them than where
    every piece runs on its own: 500 to 3269 of 1.6 to 9 million, whose independent draws differ by 2.5 to 6 % (one standard
    deviation); bar 10 %.  Planes that sum over three quarters of K have 17 % more, over all of K 27 %."""
    print(f"prompt of {n_prompt}, gemm_fused {fused}, gemm_team {team}", flush=True)
    pair = H.Pair("7b", B.CERBERUS_BF16, "root", seed=3, kv_capacity=1152, n_layers=1, d_ffn=256, vocab=1024, n_cerb_heads=1, special_block=-1)
    pair.engine.set_param("gemm_fused", fused)
    pair.engine.set_param("gemm_team", team)
    tokens = synth.make_token_ids(n_prompt, 1024, seed=8)
    kv = orc.new_kv(pair.cfg, n_prompt)
    orc.decoder_rows(pair.cfg, pair.W, tokens.numpy(), np.arange(n_prompt), np.tril(np.ones((n_prompt, n_prompt), dtype=bool)), kv, 0)
    want = torch.stack([torch.from_numpy(m).to(torch.bfloat16) for m in kv[0]])
    differ = {}
    for piece in (n_prompt, B.CERBERUS_MAX_TREE):
        st = pair.engine.new_state()
        for i in range(0, n_prompt, piece):
            pair.engine.prefill(st, 1, 0, tokens[i:i + piece].cuda())
        torch.cuda.synchronize()
        assert int(st.status[0]) == 0
        differ[piece] = int((st.kv[0, :, 0, :, :n_prompt].cpu() != want).sum())
    print(differ, flush=True)
    assert 100 < differ[B.CERBERUS_MAX_TREE] and differ[n_prompt] <= 1.1 * differ[B.CERBERUS_MAX_TREE], differ
    pair.engine.close()


@pytest.mark.parametrize("dtype,n_prompt,fused", [(B.CERBERUS_F32, 700, 1), (B.CERBERUS_BF16, 230, 1), (B.CERBERUS_BF16, 384, 1), (B.CERBERUS_BF16, 700, 1),
                                                  (B.CERBERUS_BF16, 1153, 1), (B.CERBERUS_BF16, 384, 0), (B.CERBERUS_BF16, 1153, 0)])
def test_long_prompts_match_the_oracle(dtype, n_prompt, fused):
    """Six layers of width 1024, passes of several pieces against the oracle's causal forward over pieces of 192 tokens, its
    cache rounded to the storage type between them: every cache row, the tapped rows, entropy, the heads' logits, the
    pending token; the layers on the tile kernel (gate/up of this width on the team kernel) and, with gemm_fused 0, on the team
    kernel and the 64-row blocks, QKV with its sums limited."""
    print(f"prompt of {n_prompt}, dtype {dtype}, gemm_fused {fused}", flush=True)
    P = B.CERBERUS_MAX_TREE
    tol = H.TOL_F32 if dtype == B.CERBERUS_F32 else H.TOL_BF16
    pair = H.Pair("tiny", dtype, "p63", seed=6, kv_capacity=1280, topk=6, n_layers=6, d_model=1024, n_heads=8, head_dim=128, d_ffn=1000,
                  entropy_threshold=float("inf"))
    pair.engine.set_param("gemm_fused", fused)
    cfg = pair.cfg
    tokens = synth.make_token_ids(n_prompt, cfg["vocab"], seed=9)
    ost = {"kv": orc.new_kv(cfg, n_prompt)}
    for off in range(0, n_prompt, P):
        n = min(P, n_prompt - off)
        if off:
            H.round_oracle_kv(ost, dtype)
        h_last, logits = orc.decoder_rows(cfg, pair.W, tokens.numpy()[off:off + n], np.arange(off, off + n),
                                          np.tril(np.ones((n, n), dtype=bool)), ost["kv"], off)
    taps, st = pair.taps(), pair.engine.new_state()
    st.gate_flag[:] = 1
    pair.engine.prefill(st, 1, 0, tokens.cuda())
    torch.cuda.synchronize()
    assert int(st.status[0]) == 0 and int(st.kv_len[0]) == n_prompt and int(st.gate_flag[0]) == 0
    for l, (K, V) in enumerate(ost["kv"]):
        for kvi, ref in enumerate((K, V)):
            mm = H.kv_mismatch(st.kv[l, kvi, 0, :, :n_prompt].double().cpu().numpy(), ref, tol)
            assert mm is None, (l, kvi, mm)
    k = min(n, pair.T)
    heads = np.stack(orc.cerberus_heads(cfg, pair.W["heads"], h_last[-1]))
    err = [float(np.max(np.abs(got.double().cpu().numpy() - ref))) for got, ref in
           ((taps.logits[:k], logits[:k]), (taps.h_last[:k], h_last[:k]), (taps.head_logits[0], heads))]
    print("errors of logits, h_last, heads' logits: %.2e %.2e %.2e" % tuple(err), flush=True)
    assert err[0] <= tol.logits and err[1] <= tol.hidden and err[2] <= tol.logits
    assert abs(float(st.entropy[0]) - orc.entropy_bits(h_last[-1])) <= tol.entropy
    top = np.sort(logits[-1])
    if top[-1] - top[-2] > 2 * tol.logits:
        assert int(st.root_token[0]) == int(orc.argmax_lowest(logits[-1]))
    pair.engine.close()


@pytest.mark.parametrize("one_token", [(), (0, 2, 3, 5, 6, 7, 9, 10, 12, 13, 15), tuple(range(16)), tuple(range(1, 16)),
                                       tuple(range(15)), (0, 1, 2, 4, 5, 6, 7, 9, 10, 11, 13, 14, 15)])
@pytest.mark.parametrize("fused", [0, 1])
def test_down_projection_of_a_large_batch(fused, one_token):
    """16 sequences of a 192-node tree at d = 1024: the down projection runs on the tile kernel, or with gemm_fused 0 on the team
    kernel (two column blocks, from 10 teams at the bound to 16 with few rows), with all 3072 rows, with 971, 589 and 207 of them and with 16, where every sequence
    brings one; the consumer sums as many planes as the launch took.  One workgroup per (item, head) of sequences of many lengths in
    attention.  Every row of every sequence against the oracle; the bars are those of the 7B shape, whose sums are longer."""
    print(f"down projection, one-token sequences {one_token}, gemm_fused {fused}", flush=True)
    pair = H.Pair("tiny", B.CERBERUS_BF16, "bfs4x192", seed=4, max_batch=16, kv_capacity=512, d_model=1024, n_heads=8, head_dim=128, d_ffn=1000)
    pair.engine.set_param("gemm_fused", fused)
    assert B.cerberus_bench_gemm(pair.engine.ctx, 203, 16 * pair.T) == fused         # the tile kernel takes it
    assert (B.cerberus_bench_gemm(pair.engine.ctx, 103, 16 * pair.T) >= 2.0) == (fused == 0)     # or the team kernel
    assert B.cerberus_bench_gemm(pair.engine.ctx, 103, 768) == 0.0
    taps, st = pair.taps(), pair.engine.new_state()
    osts = []
    for b in range(16):
        ost = orc.prefill(pair.cfg, pair.W, synth.make_token_ids(3 + 19 * b, pair.cfg["vocab"], seed=60 + b).numpy(), capacity=pair.kv_capacity)
        ost["flag"] = 1 if b in one_token else 0
        H.round_oracle_kv(ost, B.CERBERUS_BF16)
        H.upload_sequence(st, b, ost, B.CERBERUS_BF16)
        osts.append(ost)
    outs = [pair.oracle_step(ost) for ost in osts]
    pair.engine.verify_step(st, 16)
    torch.cuda.synchronize()
    assert int(st.status[0]) == 0
    for b, (ost, out) in enumerate(zip(osts, outs)):
        rep = H.compare_step(pair.cfg, out, st, taps, b, pair.T, B.CERBERUS_BF16, ost, tol=H.TOL_BF16)
        assert not rep.failures, f"seq {b}: " + "; ".join(rep.failures)
    pair.engine.close()


@pytest.mark.parametrize("lens", [(8100, 8000), (130, 8190), (0, 7)])
def test_attention_work_list_stays_within_the_partials(lens):
    """16 heads and two sequences of up to 8190 committed rows (64 chunks each): the partials have room for the 64 + 2 ranges of the
    default workgroup target, and a larger target (one range per chunk: 128) is cut back to that.  Every target against
    the plain kernel, which has no list; the bar is that of the tiny shapes."""
    print(f"committed rows {lens}", flush=True)
    pair = H.Pair("tiny", B.CERBERUS_BF16, "rand65s3k4", seed=7, max_batch=2, kv_capacity=8320, d_model=1024, n_heads=16, head_dim=64)
    taps, out = pair.taps(), {}
    for mfma, target in ((0, 1024), (1, 1024), (1, 65536), (1, 1)):
        pair.engine.set_param("attn_mfma", mfma)
        pair.engine.set_param("attn_target_wgs", target)
        st = pair.engine.new_state()
        g = torch.Generator(device="cuda")
        g.manual_seed(2)
        for layer in st.kv:
            layer.normal_(0.0, 1.0, generator=g)
        st.kv_len.copy_(torch.tensor(lens, dtype=torch.int32))
        st.cand.copy_(synth.make_candidates(pair.cfg, 2, seed=4))
        pair.engine.verify_step(st, 2)
        torch.cuda.synchronize()
        assert int(st.status[0]) == 0
        out[mfma, target] = taps.h_last.clone()
    for key, got in out.items():
        assert float((got - out[0, 1024]).abs().max()) <= H.TOL_BF16_TINY.hidden, key
    pair.engine.close()
