"""Edges of single kernels, each against the CPU oracle through a whole step of a small shape.  `-m gpu`, MI355X."""
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


@pytest.mark.parametrize("n_prompt,L0", [(385, 0), (576, 1), (700, 130), (1152, 0), (1153, 3)])
@pytest.mark.parametrize("dtype,attn_mfma", [(B.CERBERUS_F32, 0), (B.CERBERUS_BF16, 1), (B.CERBERUS_BF16, 0)])
def test_long_prompts_run_several_pieces_per_pass(dtype, attn_mfma, n_prompt, L0):
    """A prompt of more than two pieces of 192 tokens goes through the layers in passes of up to six pieces: the cache
    rows, the pending token and the tapped rows (the last piece's, from slot 0) against the same prompt handed over piece
    by piece (each call a pass of its own); then the same with a cache that lacks room for the later pieces.  The pieces'
    operands are the same either way and only sums change order: fp32 5e-5; bf16 within the bars of a prompt of two
    passes (a different last bit flips the bf16 rounding of a cached row now and then)."""
    print(f"prompt of {n_prompt} after {L0} rows, dtype={dtype}, attn_mfma={attn_mfma}", flush=True)
    P = B.CERBERUS_MAX_TREE
    tol = H.TOL_F32 if dtype == B.CERBERUS_F32 else H.TOL_BF16
    tokens = synth.make_token_ids(n_prompt, 1024, seed=5).cuda()
    pair = H.Pair("tiny", dtype, "p63", seed=2, max_batch=2, kv_capacity=1280, topk=6)
    pair.engine.set_param("attn_mfma", attn_mfma)

    def run(start, pieces):
        taps, st = pair.taps(), pair.engine.new_state()
        g = torch.Generator(device="cuda")
        g.manual_seed(1)
        for layer in st.kv:
            layer.normal_(0.0, 1.0, generator=g)
        st.kv_len.copy_(torch.tensor([17, start], dtype=torch.int32))
        st.gate_flag[:] = 1
        for i in range(0, n_prompt, pieces or n_prompt):
            pair.engine.prefill(st, 2, 1, tokens[i:i + (pieces or n_prompt)])
        torch.cuda.synchronize()
        return st, taps

    for start in (L0, 1280 - n_prompt // 2):          # the second start leaves room for about half of the prompt
        got, gt = run(start, None)
        want, wt = run(start, P)
        fits = start + n_prompt <= 1280
        last_fits = int(want.kv_len[1]) >= n_prompt - (n_prompt - 1) // P * P + start and int(want.gate_flag[1]) == 0
        assert int(got.kv_len[1]) == int(want.kv_len[1]) and int(got.kv_len[0]) == 17
        assert (int(got.kv_len[1]) == start + n_prompt) == fits
        assert int(got.status[0]) == int(want.status[0]) == (0 if fits else B.CERBERUS_DEV_KV_OVERFLOW)
        n = int(want.kv_len[1])
        assert torch.equal(got.kv[:, :, 0], want.kv[:, :, 0]) and torch.equal(got.kv[:, :, 1, :, n:], want.kv[:, :, 1, :, n:])
        mm = H.kv_mismatch(got.kv[:, :, 1, :, :n].double().cpu().numpy(), want.kv[:, :, 1, :, :n].double().cpu().numpy(), tol)
        assert mm is None, mm
        if fits:
            k = min((n_prompt - 1) % P + 1, pair.T)
            base = pair.T                              # taps: T rows per sequence, sequence 1
            assert float((gt.logits[base:base + k] - wt.logits[base:base + k]).abs().max()) <= tol.logits
            assert float((gt.h_last[base:base + k] - wt.h_last[base:base + k]).abs().max()) <= tol.hidden
            assert abs(float(got.entropy[1]) - float(want.entropy[1])) <= tol.entropy
            assert int(got.gate_flag[1]) == int(want.gate_flag[1])
            top = wt.logits[base + k - 1].sort().values if k == (n_prompt - 1) % P + 1 else None
            if top is not None and float(top[-1] - top[-2]) > 2 * tol.logits:
                assert int(got.root_token[1]) == int(want.root_token[1])
        else:
            # (piece by piece over several calls the gate runs after every piece; in one call only after the prompt's last)
            assert last_fits or int(got.gate_flag[1]) == 1
    pair.engine.close()


@pytest.mark.parametrize("one_token", [(), (0, 2, 3, 5, 6, 7, 9, 10, 12, 13, 15)])
def test_down_projection_of_a_large_batch(one_token):
    """16 sequences of a 192-node tree at d = 1024: the down projection runs on the team kernel (two column blocks, ten
    teams), with all 3072 rows and with 971 of them.  One workgroup per (item, head) of sequences of many lengths in
    attention.  Every row of every sequence against the oracle; the bars are those of the 7B shape, whose sums are longer."""
    print(f"down projection, one-token sequences {one_token}", flush=True)
    pair = H.Pair("tiny", B.CERBERUS_BF16, "bfs4x192", seed=4, max_batch=16, kv_capacity=512, d_model=1024, n_heads=8, head_dim=128, d_ffn=1000)
    assert B.cerberus_bench_gemm(pair.engine.ctx, 103, 16 * pair.T) >= 2.0          # the team kernel takes it
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
