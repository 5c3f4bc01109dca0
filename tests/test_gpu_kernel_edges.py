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
