"""The tile GEMMs of launches of more than 64 rows against the split-K path of the same library, at the edges of their tiles.
`-m gpu`, MI355X.

Both paths multiply the same operands (weights, and activations as hi + lo planes), only sums run in another order, so the
comparison is at the tight bar of the small shapes: one layer amplifies nothing.  The small shapes against the oracle, with more
than 64 rows, are in the other GPU tests."""
import pytest
import torch

pytestmark = pytest.mark.gpu

from paper_2410_13344_amd import binding as B
from paper_2410_13344_amd import synth
from tests import harness as H

TOL = H.TOL_BF16_TINY


def _forward(pair, batch, lens, flags, fused):
    """One verify step from random caches; every float output and the rows the step wrote."""
    pair.engine.set_param("gemm_fused", fused)
    taps, st = pair.taps(), pair.engine.new_state()
    g = torch.Generator(device="cuda")
    g.manual_seed(7)
    for layer in st.kv:
        layer.normal_(0.0, 1.0, generator=g)
    st.kv_len.copy_(torch.tensor(lens, dtype=torch.int32))
    st.gate_flag.copy_(torch.tensor(flags, dtype=torch.int32))
    st.root_token.copy_(synth.make_token_ids(batch, pair.cfg["vocab"], seed=4))
    st.cand.copy_(synth.make_candidates(pair.cfg, batch, seed=4))
    taps.logits.zero_()
    taps.h_last.zero_()
    pair.engine.verify_step(st, batch)
    torch.cuda.synchronize()
    assert int(st.status.abs().sum()) == 0
    rows = [1 if f else pair.T for f in flags]
    kv = [st.kv[:, :, b, :, n:n + (1 if f else min(pair.T, int(st.accept_len[b])))] for b, (n, f) in enumerate(zip(lens, flags))]
    return taps.logits.clone(), taps.h_last.clone(), [k.clone() for k in kv], rows


# rows live / planned: 65 (gate/up alone) ... 1024; few live rows of a large bound; odd row tiles and row blocks of unequal size
@pytest.mark.parametrize("tree,flags", [
    ("rand65s1k6", [0]), ("p120", [0]), ("rand129s2k6", [0]), ("p63", [1, 1, 1]), ("p63", [0, 1, 0]), ("rand192s3k6", [0]),
    ("rand81s4k6", [0, 0, 0]), ("rand97s5k6", [0, 0, 1, 0]), ("rand17s6k6", [0] * 15 + [1]), ("p63", [0] * 16),
])
# what decides the split over workgroups: widths (pairs per workgroup, rounds), head size, padded K, an FFN width of odd slabs
@pytest.mark.parametrize("over", [
    dict(),                                                             # d 256, heads of 64, FFN 688: K of down is padded
    dict(d_model=512, n_heads=4, head_dim=128, d_ffn=9472, vocab=512),  # gate/up in rounds at many rows, K of down 37 units
], ids=["d256", "d512"])
def test_tile_gemms_match_the_split_path(tree, flags, over):
    print(f"tree {tree}, flags {flags}, {over}", flush=True)
    batch = len(flags)
    pair = H.Pair("tiny", B.CERBERUS_BF16, tree, seed=9, max_batch=batch, kv_capacity=512, topk=10, **over)
    lens = [(37 * b + 11) % 200 for b in range(batch)]
    got, want = _forward(pair, batch, lens, flags, 1), _forward(pair, batch, lens, flags, 0)
    for b, n in enumerate(got[3]):
        s = slice(b * pair.T, b * pair.T + n)
        assert float((got[0][s] - want[0][s]).abs().max()) <= TOL.logits, b
        assert float((got[1][s] - want[1][s]).abs().max()) <= TOL.hidden, b
        mm = H.kv_mismatch(got[2][b].double().cpu().numpy(), want[2][b].double().cpu().numpy(), TOL)
        assert mm is None, (b, mm)
    again = _forward(pair, batch, lens, flags, 1)                       # bit for bit the same a second time
    assert torch.equal(again[0], got[0]) and all(torch.equal(x, y) for x, y in zip(again[2], got[2]))
    pair.engine.close()


def test_a_wide_qkv_runs_in_rounds():
    """d 4096: QKV has 384 slab pairs, twelve per workgroup at 1024 rows, which do not fit one round."""
    flags = [0] * 16
    pair = H.Pair("tiny", B.CERBERUS_BF16, "p63", seed=9, max_batch=16, kv_capacity=256, topk=10, n_layers=1, d_model=4096, n_heads=32,
                  head_dim=128, d_ffn=512, vocab=512, n_resblocks=1, special_block=-1, n_cerb_heads=4)
    lens = [(37 * b + 11) % 150 for b in range(16)]
    got, want = _forward(pair, 16, lens, flags, 1), _forward(pair, 16, lens, flags, 0)
    assert float((got[0] - want[0]).abs().max()) <= TOL.logits and float((got[1] - want[1]).abs().max()) <= TOL.hidden
    for b in range(16):
        mm = H.kv_mismatch(got[2][b].double().cpu().numpy(), want[2][b].double().cpu().numpy(), TOL)
        assert mm is None, (b, mm)
    pair.engine.close()
