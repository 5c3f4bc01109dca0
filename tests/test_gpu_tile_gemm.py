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
    """One verify step from random caches, every tree accepting along a deepest branch: every float output, the cache rows of all
    nodes (those of the accepted path moved up, in either run alike), the tokens accepted.  No other cache row may change."""
    pair.engine.set_param("gemm_fused", fused)
    taps, st = pair.taps(forced_argmax=True), pair.engine.new_state()
    g = torch.Generator(device="cuda")
    g.manual_seed(7)
    for layer in st.kv:
        layer.normal_(0.0, 1.0, generator=g)
    start = st.kv.clone()
    cand = synth.make_candidates(pair.cfg, batch, seed=4)
    st.kv_len.copy_(torch.tensor(lens, dtype=torch.int32))
    st.gate_flag.copy_(torch.tensor(flags, dtype=torch.int32))
    st.root_token.copy_(synth.make_token_ids(batch, pair.cfg["vocab"], seed=4))
    st.cand.copy_(cand)
    depths = [0] * pair.T
    for node in range(1, pair.T):
        depths[node] = depths[pair.parent[node]] + 1
    path = [depths.index(max(depths))]                                  # from the root to the first deepest node
    while path[0]:
        path.insert(0, pair.parent[path[0]])
    forced = torch.full((batch, pair.T), -1, dtype=torch.int32)
    for b in range(batch):
        for depth, (node, child) in enumerate(zip(path, path[1:])):
            forced[b, node] = cand[b, depth, pair.rank[child]]
    taps.forced_node_argmax.copy_(forced.flatten())
    taps.logits.zero_()
    taps.h_last.zero_()
    pair.engine.verify_step(st, batch)
    torch.cuda.synchronize()
    assert int(st.status.abs().sum()) == 0
    rows = [1 if f else pair.T for f in flags]
    accepted = st.accept_len[:batch].tolist()
    assert accepted == [1 if f else len(path) for f in flags] and len(path) > 2
    kv = []
    for b, (n, r) in enumerate(zip(lens, rows)):
        assert torch.equal(st.kv[:, :, b, :, :n], start[:, :, b, :, :n]) and torch.equal(st.kv[:, :, b, :, n + r:], start[:, :, b, :, n + r:])
        kv.append(st.kv[:, :, b, :, n:n + r].clone())
    return taps.logits.clone(), taps.h_last.clone(), kv, rows


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


@pytest.mark.parametrize("nodes", [16, 17, 33, 63, 64])
def test_a_gate_up_too_wide_for_the_whole_k_kernel(nodes):
    """FFN of 13824 columns: more slabs than the whole-K kernel of up to 64 rows has room for, so from 17 rows on gate/up runs on the
    tile kernel, the other projections as in any small launch."""
    pair = H.Pair("tiny", B.CERBERUS_BF16, f"rand{nodes}s7k6", seed=9, max_batch=1, kv_capacity=256, topk=10, d_ffn=13824)
    assert pair.T == nodes
    assert [B.cerberus_bench_gemm(pair.engine.ctx, 200 + kind, nodes) for kind in range(4)] == [0.0, 0.0, float(nodes > 16), 0.0]
    got, want = _forward(pair, 1, [29], [0], 1), _forward(pair, 1, [29], [0], 0)
    assert float((got[0] - want[0]).abs().max()) <= TOL.logits and float((got[1] - want[1]).abs().max()) <= TOL.hidden
    mm = H.kv_mismatch(got[2][0].double().cpu().numpy(), want[2][0].double().cpu().numpy(), TOL)
    assert mm is None, mm
    pair.engine.close()


@pytest.mark.parametrize("model,tree,batch", [("7b", "p63", 11), ("7b", "rand100s1k6", 11), ("7b", "p63", 16), ("13b", "rand100s1k6", 6), ("13b", "p63", 16)])
def test_sums_of_the_down_projection_stay_short(model, tree, batch):
    """A projection of known result with all its products positive, K = 11008 and 13824: token rows of one constant, FFN
    activations of one constant (the gate's exponential underflows), random positive weights.  A sum rounds its running value with
    every product, so what a column is off by shows how many products it was summed over in one piece: n roundings of at most
    half a unit, each of a value no larger than the result, have a standard deviation below 2^-24 sqrt(n / 3).  The 54 sums of 8
    k-steps, or the sums of 32 with 64 roundings of a fifth of the result or less, the planes, the residual and the norm count
    for fewer than 55; sums of 3670 to 6912 columns in one piece have 230 to 432."""
    cfg = synth.make_config(model, n_layers=1, vocab=256, n_cerb_heads=4, n_resblocks=1, special_block=-1, topk=6)
    d, F, e = cfg["d_model"], cfg["d_ffn"], 1.2421875                    # (e: eight significant bits, exact in bf16)
    W = synth.make_weights(cfg, seed=0, dtype=torch.bfloat16, device="cuda")
    layer = W["layers"][0]
    for t in (W["embed"], W["final_norm"], layer["attn_norm"], layer["ffn_norm"]):
        t.fill_(1.0)
    W["embed"].mul_(e)
    for name in ("wqkv", "wo", "w_gate_up"):
        layer[name].zero_()                                              # attention adds nothing
    layer["w_gate_up"][:F, 0], layer["w_gate_up"][F:, 0] = 32.0, e / 32  # silu(32) = 32 to the last bit
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    layer["w_down"].copy_((torch.rand(d, F, device="cuda", generator=g) + 1.0) * 2.0 ** -9)
    layer["w_down"][0] = 0                                               # column 0 stays at e: what the others are measured by
    parent, rank = synth.make_tree(tree, cfg["n_cerb_heads"])
    engine = B.Engine(cfg, W, parent, rank, B.CERBERUS_BF16, batch, 256)
    taps = B.DeviceTaps(cfg, batch, len(parent))
    engine.set_taps(taps)
    st = engine.new_state()
    engine.verify_step(st, batch)
    torch.cuda.synchronize()
    assert int(st.status.abs().sum()) == 0
    h = taps.h_last.double()
    want = layer["w_down"][1:].double().sum(1)
    off = (h[:, 1:] / h[:, :1] - 1.0) / want[None]                       # one constant, but for the error of the sums
    off = off / off.median() - 1.0
    slabs = off[:, 15:].reshape(off.shape[0], -1, 16).square().mean((0, 2)).sqrt()
    print(f"{model}, {off.shape[0]} rows: largest error of a slab {float(slabs.max()):.2e}", flush=True)
    assert float(slabs.max()) <= 2.0 ** -24 * (55 / 3) ** 0.5
    engine.close()


@pytest.mark.parametrize("kind,columns,least", [(0, 768, 1), (1, 256, 4), (2, 688, 1), (3, 256, 4)])
def test_benchmark_hook_runs_the_rows_it_is_asked_for(kind, columns, least):
    """192 rows asked for after a step that had three: the launch still reads and writes all of them, as the bytes it reports say.
    Nearly every byte of a value changes where a buffer takes other results, so `least` bytes per output element of half
    of the rows are a lower bound, three rows' worth of up to eight planes far below it."""
    pair = H.Pair("tiny", B.CERBERUS_BF16, "p63", seed=9, max_batch=3, kv_capacity=256, topk=10)
    st = pair.engine.new_state()
    st.cand.copy_(synth.make_candidates(pair.cfg, 3, seed=4))
    assert B.cerberus_bench_gemm(pair.engine.ctx, 200 + kind, 192) == 1.0           # on the tile kernel
    pair.engine.verify_step(st, 3)
    pair.engine.ar_step(st, 3)
    torch.cuda.synchronize()
    before = pair.engine.workspace.clone()
    B.cerberus_bench_gemm(pair.engine.ctx, kind, 192)
    torch.cuda.synchronize()
    changed = int((pair.engine.workspace != before).sum())
    print(f"kind {kind}: {changed} bytes changed", flush=True)
    assert changed >= 96 * columns * least
    pair.engine.close()


def test_hook_names_the_team_kernel_only_where_a_step_runs_it():
    """gemm_fused 0 keeps the tile kernel out: gate/up of 192 rows is then the team kernel's, as its own plan says."""
    pair = H.Pair("tiny", B.CERBERUS_BF16, "p63", seed=9, max_batch=3, kv_capacity=256, topk=10)
    query = lambda kind: B.cerberus_bench_gemm(pair.engine.ctx, kind, 192)
    assert (query(102), query(202)) == (0.0, 1.0)
    pair.engine.set_param("gemm_fused", 0)
    assert query(102) > 2.0 and query(202) == 0.0
    pair.engine.close()
