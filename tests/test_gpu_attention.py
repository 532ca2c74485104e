"""GPU parity: radar_tree_attention (through the C ABI) against the CPU oracle.

Contract (bf16 inputs, fp32 accumulation, bf16 output; probabilities are rounded to bf16 before
the P.V contraction): max-abs error <= 2e-2 and relative error (L2 norm over the compared block)
<= 1e-2, the bounds of the baseline description.  The tests hold the kernels to tighter,
per-element bounds derived from the arithmetic: both sides round the output to bf16 (half an ulp
each, 2^-8 relative), and the device's bf16 probabilities add at most 2^-9 of the largest value
in the row's average, so |error| <= ABS_TIGHT + REL_TIGHT * |reference| for every element.
The log-sum-exp output is fp32 on both sides (fp32 score accumulation, hardware exp2 / log2):
1e-4 absolute."""
import numpy as np
import pytest
import torch

from paper_2512_14069_amd import synth
from gpu_util import bf16_dev, bf16_bits, dev, host

pytestmark = pytest.mark.gpu

MAX_ABS = 2e-2          # the contract
REL = 1e-2
ABS_TIGHT = 6e-3        # per element: |err| <= ABS_TIGHT + REL_TIGHT * |ref|
REL_TIGHT = 8e-3        # one bf16 ulp
LSE_TOL = 1e-4


def f64(bits):
    return synth.bf16_bits_to_f32(bits).astype(np.float64)


def check_close(got_bits, ref_bits, what=""):
    got, ref = f64(got_bits), f64(ref_bits)
    assert np.all(np.isfinite(got)), what
    err = np.abs(got - ref)
    rel = np.linalg.norm(got - ref) / max(np.linalg.norm(ref), 1e-30)
    assert err.max() <= MAX_ABS, f"{what}: max abs {err.max():.3e}"
    assert rel <= REL, f"{what}: rel {rel:.3e}"
    over = err - (ABS_TIGHT + REL_TIGHT * np.abs(ref))
    assert over.max() <= 0, f"{what}: element error {err.flat[over.argmax()]:.3e} at |ref| {abs(ref.flat[over.argmax()]):.3e}"
    return err.max(), rel


def run_gpu(b, x, keys_per_split=0, want_lse=False, scale=0.0):
    q, kc, vc = bf16_dev(x["q"]), bf16_dev(x["k_cache"]), bf16_dev(x["v_cache"])
    B, T, Hq, D = q.shape
    lse = torch.full((B, T, Hq), 7.0, dtype=torch.float32, device="cuda") if want_lse else None
    out = torch.full(q.shape, 3.0, dtype=torch.bfloat16, device="cuda")
    b.radar_tree_attention(q, kc, vc, dev(x["parents"]), dev(x["ctx_lens"]), dev(x["n_nodes"]),
                           out=out, lse_out=lse, keys_per_split=keys_per_split, softmax_scale=scale)
    torch.cuda.synchronize()
    return (bf16_bits(out), host(lse)) if want_lse else bf16_bits(out)


def shape(B, Hq, Hkv, D, T, ctx, nn, dep, k=4):
    return synth.AttnShape(B=B, Hq=Hq, Hkv=Hkv, D=D, T=T, ctx_lens=tuple(ctx), n_nodes=tuple(nn), depths=tuple(dep), k=k)


CASES = {
    "c1_smoke": shape(1, 4, 1, 64, 16, [256], [16], [4]),
    "gqa4_d128_ragged_tail": shape(2, 8, 2, 128, 40, [333, 70], [40, 17], [5, 3]),
    "mha_d64": shape(1, 3, 3, 64, 33, [129], [33], [6]),
    "group_of_3": shape(1, 6, 2, 128, 20, [200], [20], [4]),
    "group_of_8_two_query_blocks": shape(2, 16, 2, 128, 64, [190, 65], [64, 50], [8, 8], k=10),
    "group_of_6": shape(1, 6, 1, 64, 12, [100], [12], [3]),
    "empty_prefix": shape(2, 4, 2, 128, 30, [0, 0], [30, 1], [4, 1]),
    "root_only": shape(1, 4, 4, 64, 8, [77], [1], [1]),
    "one_slot": shape(1, 2, 1, 128, 1, [50], [1], [1]),
}


@pytest.mark.parametrize("kps", [0, 64, 128])
@pytest.mark.parametrize("name", list(CASES))
def test_small_cases_match_oracle(oracle, name, kps):
    from paper_2512_14069_amd import binding as b
    a = CASES[name]
    x = synth.attention_inputs(a, seed=synth.seed_for(1, len(name)), shuffle=True)
    ref, ref_lse = oracle.tree_attention(x["q"], x["k_cache"], x["v_cache"], x["parents"], x["ctx_lens"],
                                         x["n_nodes"], want_lse=True)
    got, lse = run_gpu(b, x, keys_per_split=kps, want_lse=True)
    for bb in range(a.B):
        n = a.n_nodes[bb]
        check_close(got[bb, :n], ref[bb, :n], f"{name} b={bb}")
        assert np.max(np.abs(lse[bb, :n] - ref_lse[bb, :n])) < LSE_TOL
        assert np.all(got[bb, n:] == 0) and np.all(lse[bb, n:] == 0)     # unused rows are zeroed


LONG_CASES = {
    "d128_ragged": shape(2, 8, 2, 128, 40, [1100, 530], [40, 17], [5, 3]),
    "d64_two_query_blocks": shape(1, 8, 2, 64, 64, [700], [64], [8], k=10),
    "one_tile_and_root_only": shape(2, 4, 2, 128, 30, [0, 600], [30, 1], [4, 1]),
    "group_of_3_tail_of_33": shape(1, 6, 2, 128, 20, [1037], [20], [4]),
    # two blocks of units per range of cache rows (16 units), which sit a multiple of 8 apart in the grid
    "group_of_8_two_unit_blocks": shape(2, 16, 2, 128, 64, [1500, 700], [64, 50], [8, 8], k=10),
    # a cache that ends exactly at a tile (and range) boundary, and one row over it
    "aligned_end_and_one_row_over": shape(2, 4, 1, 128, 40, [984, 985], [40, 40], [5, 5]),
}


@pytest.mark.parametrize("kps", [512, 1024, 2048])
@pytest.mark.parametrize("name", list(LONG_CASES))
def test_long_ranges_match_oracle(oracle, name, kps):
    """Ranges of nine tiles or more run the long-range kernels (tiles loaded straight into LDS and taken
    in pairs at D = 128, two-ahead register staging at D = 64), eight tiles are the longest that the
    short-range one gets.  Ranges that end after one, two or several tiles, an odd and an even number of
    tiles, tree rows that straddle a tile or a range boundary, a single range (no merge), wavefronts without a unit."""
    from paper_2512_14069_amd import binding as b
    a = LONG_CASES[name]
    x = synth.attention_inputs(a, seed=synth.seed_for(1, 7 * len(name) + kps // 512), shuffle=True)
    ref, ref_lse = oracle.tree_attention(x["q"], x["k_cache"], x["v_cache"], x["parents"], x["ctx_lens"],
                                         x["n_nodes"], want_lse=True)
    got, lse = run_gpu(b, x, keys_per_split=kps, want_lse=True)
    for bb in range(a.B):
        n = a.n_nodes[bb]
        check_close(got[bb, :n], ref[bb, :n], f"{name} b={bb} kps={kps}")
        assert np.max(np.abs(lse[bb, :n] - ref_lse[bb, :n])) < LSE_TOL
        assert np.all(got[bb, n:] == 0) and np.all(lse[bb, n:] == 0)


def _ragged(seed, B, hi, T):
    rng = np.random.default_rng(seed)
    nodes = [int(v) for v in rng.integers(1, T + 1, B)]
    ctx = [int(v) for v in rng.integers(0, hi + 1, B)]
    ctx[B // 2] = hi
    return ctx, nodes, [min(8, max(1, n - 1)) for n in nodes]


DEALT_CASES = {                                   # name: B, Hq, Hkv, T, longest prefix, equal lengths
    "group_of_4": (32, 32, 8, 60, 700, False),                # trees on both sides of one block of 32 rows
    "one_head_per_kv_head": (64, 4, 4, 20, 1500, False),      # one unit
    "group_of_8_two_unit_blocks": (16, 64, 8, 64, 900, False),    # small trees: the unit blocks share a piece
    "group_of_12_three_unit_blocks": (21, 48, 4, 40, 520, False),
    "many_pieces_per_head": (2, 4, 2, 33, 36000, False),      # more partials than one batch of the merge
    "equal_lengths": (5, 16, 8, 40, 4200, True),              # whole pieces, six per head
    "one_sequence": (1, 8, 8, 60, 17000, True),
}


def scratch_bytes(b, B, Hq, Hkv, D, T, S):
    return b.radar_tree_attention_workspace_bytes(b.attn_desc(torch.empty((B, T, Hq, D), device="meta"), torch.empty((B, Hkv, S, D), device="meta")))


def dealt_bytes(B, Hq, Hkv, D, T):
    """What the workspace of a call whose rows are dealt out holds: a partial per unit for every share and every KV head, and
    the table for the merge."""
    blocks = -(-(Hq // Hkv) * (1 if T <= 32 else 2) // 8)
    entries = (256 // blocks + B * Hkv) * blocks * 8
    return 256 + sum(-(-n // 256) * 256 for n in (entries * 32 * (D // 2) * 4, entries * 96 * 4, B * Hkv * 8))


@pytest.mark.parametrize("name", list(DEALT_CASES))
def test_rows_dealt_out_on_the_device(oracle, name):
    """Long ranges that the caller does not fix are cut into shares on the device: pieces that begin and end
    anywhere, several pieces per workgroup, heads cut into many, idle workgroups, and trees that fill half of
    the workgroups, whose keys are then shared."""
    from paper_2512_14069_amd import binding as b
    B, Hq, Hkv, T, hi, equal = DEALT_CASES[name]
    ctx, nodes, depth = ([hi] * B, [T] * B, [8] * B) if equal else _ragged(len(name), B, hi, T)
    a = shape(B, Hq, Hkv, 128, T, ctx, nodes, depth, k=10)
    assert scratch_bytes(b, B, Hq, Hkv, 128, T, a.S) == dealt_bytes(B, Hq, Hkv, 128, T)
    x = synth.attention_inputs(a, seed=synth.seed_for(1, 11 * len(name)), shuffle=True)
    ref, ref_lse = oracle.tree_attention(x["q"], x["k_cache"], x["v_cache"], x["parents"], x["ctx_lens"],
                                         x["n_nodes"], want_lse=True)
    got, lse = run_gpu(b, x, want_lse=True)
    for bb in range(B):
        n = a.n_nodes[bb]
        check_close(got[bb, :n], ref[bb, :n], f"{name} b={bb}")
        assert np.max(np.abs(lse[bb, :n] - ref_lse[bb, :n])) < LSE_TOL
        assert np.all(got[bb, n:] == 0) and np.all(lse[bb, n:] == 0)


@pytest.mark.parametrize("D,S,kps", [(128, 300, 0), (128, 300, 64), (64, 1300, 1024), (128, 1300, 1024), (128, 41000, 0)])
def test_context_lengths_past_the_cache_are_cut_to_it(D, S, kps):
    """Lengths up to 2^31 - 1 (which wrap when the tree's rows are added): the rows that the caller described are
    attended to, by every path, and the tree has none.  One workspace, which holds another call's partials.
    Bound: as check_close, on both paths' arithmetic."""
    from paper_2512_14069_amd import binding as b
    g = torch.Generator().manual_seed(S + kps)
    q, kc, vc = (torch.randn(s, generator=g).to(torch.bfloat16) for s in ((3, 40, 4, D), (3, 2, S, D), (3, 2, S, D)))
    p = torch.einsum("btgd,bsd->btgs", q[:, :, :2].double(), kc[:, 0].double()).div(D ** 0.5).softmax(-1)
    want = torch.einsum("btgs,bsd->btgd", p, vc[:, 0].double())                 # the first KV head's two query heads
    par, nn = dev(np.tile(synth.chain_tree(40), (3, 1))), dev(np.array([40, 1, 33], np.int32))
    qd, kd, vd = q.cuda(), kc.cuda(), vc.cuda()
    ws = b.new_workspace(b.radar_tree_attention_workspace_bytes(b.attn_desc(qd, kd, keys_per_split=kps)))
    attend = lambda ctx: b.radar_tree_attention(qd, kd, vd, par, dev(np.array(ctx, np.int32)), nn, workspace=ws, keys_per_split=kps,
                                                out=torch.full(q.shape, 3.0, dtype=torch.bfloat16, device="cuda"))
    full = attend([S, S, S])
    attend([S - 40, 0, 7])
    past = attend([2 ** 31 - 1, 2 ** 31 - 2, S + 1])
    assert torch.equal(full, past)
    for i, n in enumerate((40, 1, 33)):
        assert torch.all(past[i, n:] == 0)
        err = (past[i, :n, :2].double().cpu() - want[i, :n]).abs()
        assert torch.all(err <= ABS_TIGHT + REL_TIGHT * want[i, :n].abs())


@pytest.mark.parametrize("D,ctx,nn,T", [
    (128, 0, 1, 1), (128, 0, 2, 64), (64, 0, 1, 33),                       # one row, two; a block of rows past the tree
    (128, 30, 1, 5), (128, 31, 1, 32), (64, 32, 1, 33),                     # 31, 32 and 33 rows: one wavefront or two
    (128, 223, 32, 32), (128, 200, 57, 60), (64, 255, 2, 2),                # 255, 257 and 257 rows: the second step's first
    (128, 320, 64, 64), (128, 352, 32, 32), (64, 768, 64, 64), (64, 799, 1, 33),   # the most rows that go in one launch
    (128, 321, 64, 64), (128, 353, 32, 32), (64, 769, 64, 64),              # one row more: ranges
    (128, 608, 32, 32), (64, 960, 64, 64),
])
def test_one_launch_over_whole_units(oracle, D, ctx, nn, T):
    """Short contexts take one launch in which eight wavefronts share a unit's rows; every count of rows around 32 (one
    wavefront's step) and 256 (the workgroup's), and the last ones that go this way.  The second sequence is shorter."""
    from paper_2512_14069_amd import binding as b
    nodes = [nn, (nn + 1) // 2]
    a = shape(2, 4, 2, D, T, [ctx, ctx // 3], nodes, [max(1, min(6, n - 1)) for n in nodes], k=64)
    x = synth.attention_inputs(a, seed=synth.seed_for(1, ctx * 64 + nn), shuffle=True)
    ref, ref_lse = oracle.tree_attention(x["q"], x["k_cache"], x["v_cache"], x["parents"], x["ctx_lens"],
                                         x["n_nodes"], want_lse=True)
    got, lse = run_gpu(b, x, want_lse=True)
    for bb in range(2):
        n = nodes[bb]
        check_close(got[bb, :n], ref[bb, :n], f"b={bb}")
        assert np.max(np.abs(lse[bb, :n] - ref_lse[bb, :n])) < LSE_TOL
        assert np.all(got[bb, n:] == 0) and np.all(lse[bb, n:] == 0)     # unused rows are zeroed


@pytest.mark.parametrize("B,Hq,Hkv,T,rows", [
    (1, 32, 8, 64, 513), (1, 32, 8, 60, 900),                               # 64 units: the third step's first row, and the line
    (2, 32, 8, 64, 769), (1, 64, 8, 64, 1400), (3, 32, 8, 60, 1280),        # 128 and 192 units
    (4, 32, 8, 40, 1600), (2, 64, 8, 60, 1569), (8, 16, 4, 33, 1025),       # 256 units: seven steps, full and begun
    (1, 32, 16, 64, 700), (3, 32, 8, 20, 800), (4, 48, 4, 32, 1100), (4, 64, 8, 17, 1057),
])
def test_one_launch_of_many_units_and_steps(oracle, B, Hq, Hkv, T, rows):
    """The longest calls that go in one launch at D = 128: 64 to 256 units, three to seven steps per wavefront, each of which
    lands where the one before it has been read.  The other sequences are shorter."""
    from paper_2512_14069_amd import binding as b
    nodes = [T] + [(T + 1) // 2] * (B - 1)
    ctx = [rows - T] + [(rows - T) * (i + 1) // (B + 1) for i in range(1, B)]
    a = shape(B, Hq, Hkv, 128, T, ctx, nodes, [max(1, min(6, n - 1)) for n in nodes], k=64)
    assert a.S == rows and scratch_bytes(b, B, Hq, Hkv, 128, T, rows) == 256          # no partials
    x = synth.attention_inputs(a, seed=synth.seed_for(1, rows + Hq), shuffle=True)
    ref, ref_lse = oracle.tree_attention(x["q"], x["k_cache"], x["v_cache"], x["parents"], x["ctx_lens"],
                                         x["n_nodes"], want_lse=True)
    got, lse = run_gpu(b, x, want_lse=True)
    for bb in range(B):
        n = nodes[bb]
        check_close(got[bb, :n], ref[bb, :n], f"b={bb}")
        assert np.max(np.abs(lse[bb, :n] - ref_lse[bb, :n])) < LSE_TOL
        assert np.all(got[bb, n:] == 0) and np.all(lse[bb, n:] == 0)     # unused rows are zeroed


@pytest.mark.parametrize("B,Hq,Hkv,D,T,rows", [
    (15, 8, 1, 64, 60, 1000), (16, 8, 1, 64, 16, 900), (17, 4, 1, 64, 60, 900),   # fifteen KV heads, sixteen, seventeen
    (11, 14, 7, 128, 17, 370), (9, 12, 3, 64, 33, 700), (8, 12, 3, 128, 60, 300), (25, 10, 5, 128, 5, 240),
    (64, 4, 1, 64, 60, 260), (32, 8, 1, 128, 20, 260),                      # as many units as an XCD holds
    (9, 28, 4, 128, 32, 900), (17, 14, 2, 64, 40, 900),                     # more than that on one of them: taken in order
])
def test_one_launch_of_kv_heads_by_eights(oracle, B, Hq, Hkv, D, T, rows):
    """One launch over many rows of a batch whose KV heads are no multiple of eight: its workgroups go through the heads of all
    sequences eight at a time, and find sequence and head from their number."""
    from paper_2512_14069_amd import binding as b
    nodes = [max(1, T - i % 3) for i in range(B)]
    ctx = [(rows - T) * (B - i) // B for i in range(B)]
    a = shape(B, Hq, Hkv, D, T, ctx, nodes, [max(1, min(6, n - 1)) for n in nodes], k=64)
    assert a.S == rows and scratch_bytes(b, B, Hq, Hkv, D, T, rows) == 256            # no partials
    x = synth.attention_inputs(a, seed=synth.seed_for(1, rows + Hq), shuffle=True)
    ref, ref_lse = oracle.tree_attention(x["q"], x["k_cache"], x["v_cache"], x["parents"], x["ctx_lens"],
                                         x["n_nodes"], want_lse=True)
    got, lse = run_gpu(b, x, want_lse=True)
    for bb in range(B):
        n = nodes[bb]
        check_close(got[bb, :n], ref[bb, :n], f"b={bb}")
        assert np.max(np.abs(lse[bb, :n] - ref_lse[bb, :n])) < LSE_TOL
        assert np.all(got[bb, n:] == 0) and np.all(lse[bb, n:] == 0)     # unused rows are zeroed


@pytest.mark.parametrize("D,ctx,nn,kps", [(128, 30, 3, 0), (128, 224, 33, 0), (128, 256, 1, 0), (64, 256, 16, 0), (64, 700, 60, 0), (128, 256, 32, 0),
                                          (128, 224, 33, 64), (64, 256, 16, 64), (128, 1000, 40, 64), (128, 2000, 17, 64),
                                          (128, 1000, 33, 576), (128, 1000, 33, 1088), (64, 1000, 33, 576), (128, 36000, 33, 0)])
def test_infinite_values_in_the_last_row(oracle, D, ctx, nn, kps):
    """The last node's V row holds +Inf and -Inf in two columns: its own output is the infinity there, whatever the count of rows
    leaves of a tile (rows past the end count for nothing, also as copies of the last one), and every other column is as without them.
    (The other nodes' products 0 * Inf in the two columns are not defined.)"""
    from paper_2512_14069_amd import binding as b
    a = shape(1, 4, 2, D, max(nn, 2), [ctx], [nn], [max(1, min(6, nn - 1))], k=64)
    x = synth.attention_inputs(a, seed=synth.seed_for(1, ctx + nn), shuffle=True)
    ref = oracle.tree_attention(x["q"], x["k_cache"], x["v_cache"], x["parents"], x["ctx_lens"], x["n_nodes"])
    x["v_cache"][0, :, ctx + nn - 1, 5], x["v_cache"][0, :, ctx + nn - 1, D - 3] = 0x7f80, 0xff80
    x["v_cache"][0, :, ctx + nn:] = 0x7fc0
    got = run_gpu(b, x, keys_per_split=kps)
    finite = [d for d in range(D) if d not in (5, D - 3)]
    check_close(got[0, :nn, :, finite], ref[0, :nn, :, finite], "columns without an infinity")
    assert np.all(f64(got[0, nn - 1, :, 5]) == np.inf) and np.all(f64(got[0, nn - 1, :, D - 3]) == -np.inf)


@pytest.mark.parametrize("parts", [2, 4, 5, 8, 9, 12, 13, 16, 17, 18, 19, 24, 25, 33, 36, 37])
def test_merge_takes_any_number_of_partials(oracle, parts):
    """The merge asks for up to 18 partials at a time, in steps of four, and for as few rounds as that allows: numbers of
    ranges at the edges of both, the second sequence with about a third of them."""
    from paper_2512_14069_amd import binding as b
    D, nn = (128, 64)[parts & 1], (20, 37)[parts >> 1 & 1]
    a = shape(2, 4, 2, D, 40, [parts * 64 - nn, parts * 64 // 3], [nn, 9], [5, 3])
    x = synth.attention_inputs(a, seed=synth.seed_for(1, parts), shuffle=True)
    ref, ref_lse = oracle.tree_attention(x["q"], x["k_cache"], x["v_cache"], x["parents"], x["ctx_lens"],
                                         x["n_nodes"], want_lse=True)
    got, lse = run_gpu(b, x, keys_per_split=64, want_lse=True)
    for bb in range(2):
        n = a.n_nodes[bb]
        check_close(got[bb, :n], ref[bb, :n], f"b={bb}")
        assert np.max(np.abs(lse[bb, :n] - ref_lse[bb, :n])) < LSE_TOL
        assert np.all(got[bb, n:] == 0) and np.all(lse[bb, n:] == 0)     # unused rows are zeroed


@pytest.mark.parametrize("D,T,kps", [(128, 16, 128), (128, 60, 128), (64, 33, 128), (128, 32, 64), (64, 60, 192), (128, 60, 192)])
def test_short_sequences_after_a_call_that_filled_every_range(oracle, D, T, kps):
    """A range of two tiles asks for both at once, before the lengths are there; sequences end in their first range, at a tile's
    edge, one row past it, within the second tile and in the last range.  What lies past the end is NaN in the cache, and the workspace holds
    NaN partials of a call over all of it.  The outputs and the log-sum-exp: as the other tests."""
    from paper_2512_14069_amd import binding as b
    nn = [T, 1, (T + 1) // 2, T, 2, T]
    rows = [kps - 1, 64, kps + 65, kps + 64 + T, 2 * kps, 9 * kps - 3]
    a = shape(6, 4, 2, D, T, [max(r - n, 0) for r, n in zip(rows, nn)], nn, [max(1, min(6, n - 1)) for n in nn], k=64)
    x = synth.attention_inputs(a, seed=synth.seed_for(1, D + T + kps), shuffle=True)
    ref, ref_lse = oracle.tree_attention(x["q"], x["k_cache"], x["v_cache"], x["parents"], x["ctx_lens"], x["n_nodes"], want_lse=True)
    for i, n in enumerate(nn):
        x["k_cache"][i, :, x["ctx_lens"][i] + n:] = x["v_cache"][i, :, x["ctx_lens"][i] + n:] = 0x7fc0
    q, kc, vc = bf16_dev(x["q"]), bf16_dev(x["k_cache"]), bf16_dev(x["v_cache"])
    lse = torch.full((6, T, 4), 7.0, dtype=torch.float32, device="cuda")
    ws = b.new_workspace(b.radar_tree_attention_workspace_bytes(b.attn_desc(q, kc, keys_per_split=kps)))
    attend = lambda k, v, ctx: b.radar_tree_attention(q, k, v, dev(x["parents"]), dev(ctx), dev(x["n_nodes"]), workspace=ws, keys_per_split=kps,
                                                      lse_out=lse, out=torch.full(q.shape, 3.0, dtype=torch.bfloat16, device="cuda"))
    attend(kc, torch.full_like(vc, float("nan")), np.full(6, a.S - T, np.int32))
    got, lse = bf16_bits(attend(kc, vc, x["ctx_lens"])), host(lse)
    for i, n in enumerate(nn):
        check_close(got[i, :n], ref[i, :n], f"b={i}")
        assert np.max(np.abs(lse[i, :n] - ref_lse[i, :n])) < LSE_TOL
        assert np.all(got[i, n:] == 0) and np.all(lse[i, n:] == 0)


def test_chain_and_star_trees_depth_63(oracle):
    from paper_2512_14069_amd import binding as b
    a = shape(2, 4, 1, 128, 64, [100, 31], [64, 64], [8, 8], k=10)
    x = synth.attention_inputs(a, seed=4)
    x["parents"][0] = synth.chain_tree(64)
    x["parents"][1] = synth.star_tree(64)
    ref = oracle.tree_attention(x["q"], x["k_cache"], x["v_cache"], x["parents"], x["ctx_lens"], x["n_nodes"])
    for kps in (0, 64):
        got = run_gpu(b, x, keys_per_split=kps)
        check_close(got, ref, f"kps={kps}")


def test_non_ancestors_and_padding_rows_do_not_leak(oracle):
    """Changing K/V of cache rows past the tree, of a leaf's non-ancestors, or parents past
    n_nodes leaves the affected outputs bit-identical on the device."""
    from paper_2512_14069_amd import binding as b
    a = shape(1, 8, 2, 128, 24, [150], [20], [4])
    x = synth.attention_inputs(a, seed=12)
    base = run_gpu(b, x)
    rng = np.random.default_rng(0)
    y = {k: v.copy() for k, v in x.items()}
    L, n = 150, 20
    y["k_cache"][0, :, L + n:] = synth.normal_bf16(rng, y["k_cache"][0, :, L + n:].shape)
    y["v_cache"][0, :, L + n:] = 0x7fc0                     # NaNs past the end must not leak
    y["parents"][0, n:] = 0
    victim = n - 1                                            # last node: ancestor of nobody else
    y["k_cache"][0, :, L + victim] = synth.normal_bf16(rng, (2, 128))
    y["v_cache"][0, :, L + victim] = synth.normal_bf16(rng, (2, 128))
    got = run_gpu(b, y)
    assert np.array_equal(got[0, :victim], base[0, :victim])
    assert not np.array_equal(got[0, victim], base[0, victim])


def test_strided_views_and_scale(oracle):
    """q taken from a fused [B,T,3*Hq,D] projection buffer and caches with a padded row pitch."""
    from paper_2512_14069_amd import binding as b
    a = shape(1, 8, 2, 128, 20, [90], [20], [4])
    x = synth.attention_inputs(a, seed=3)
    ref = oracle.tree_attention(x["q"], x["k_cache"], x["v_cache"], x["parents"], x["ctx_lens"], x["n_nodes"],
                                scale=0.05)
    fused = torch.zeros((1, 20, 24, 128), dtype=torch.bfloat16, device="cuda")
    fused[:, :, 8:16] = bf16_dev(x["q"])
    q = fused[:, :, 8:16]
    S = x["k_cache"].shape[2]
    kbuf = torch.zeros((1, 2, S + 9, 128), dtype=torch.bfloat16, device="cuda")
    vbuf = torch.zeros((1, 2, S + 9, 128), dtype=torch.bfloat16, device="cuda")
    kbuf[:, :, :S] = bf16_dev(x["k_cache"]); vbuf[:, :, :S] = bf16_dev(x["v_cache"])
    out = b.radar_tree_attention(q, kbuf[:, :, :S], vbuf[:, :, :S], dev(x["parents"]), dev(x["ctx_lens"]),
                                 dev(x["n_nodes"]), softmax_scale=0.05)
    torch.cuda.synchronize()
    check_close(bf16_bits(out), ref, "strided")


def test_long_range_strided_cache(oracle):
    """Long ranges over caches with a padded row pitch and a padded head pitch (the row-to-LDS loads
    compute their own addresses from the strides)."""
    from paper_2512_14069_amd import binding as b
    a = shape(2, 8, 2, 128, 33, [1200, 640], [33, 9], [6, 3])
    x = synth.attention_inputs(a, seed=11, shuffle=True)
    ref, ref_lse = oracle.tree_attention(x["q"], x["k_cache"], x["v_cache"], x["parents"], x["ctx_lens"], x["n_nodes"],
                                         want_lse=True)
    S = x["k_cache"].shape[2]
    kbuf = torch.full((2, 2, S + 5, 136), 9.0, dtype=torch.bfloat16, device="cuda")
    vbuf = torch.full((2, 2, S + 5, 136), -9.0, dtype=torch.bfloat16, device="cuda")
    kbuf[:, :, :S, :128] = bf16_dev(x["k_cache"]); vbuf[:, :, :S, :128] = bf16_dev(x["v_cache"])
    for kps in (512, 1024):
        lse = torch.zeros((2, 33, 8), dtype=torch.float32, device="cuda")
        out = b.radar_tree_attention(bf16_dev(x["q"]), kbuf[:, :, :S, :128], vbuf[:, :, :S, :128], dev(x["parents"]),
                                     dev(x["ctx_lens"]), dev(x["n_nodes"]), lse_out=lse, keys_per_split=kps)
        torch.cuda.synchronize()
        got = bf16_bits(out)
        for bb in range(a.B):
            n = a.n_nodes[bb]
            check_close(got[bb, :n], ref[bb, :n], f"strided long b={bb} kps={kps}")
            assert np.max(np.abs(host(lse)[bb, :n] - ref_lse[bb, :n])) < LSE_TOL


def whole_config_check(oracle, b, a, seed):
    """Full-size launch in the default plan; every output element and every log-sum-exp compared."""
    x = synth.attention_inputs(a, seed=seed)
    got, lse = run_gpu(b, x, want_lse=True)
    ref, ref_lse = oracle.tree_attention(x["q"], x["k_cache"], x["v_cache"], x["parents"], x["ctx_lens"], x["n_nodes"],
                                         want_lse=True)
    worst = (0.0, 0.0)
    for bb in range(a.B):
        n = a.n_nodes[bb]
        e = check_close(got[bb, :n], ref[bb, :n], f"b={bb}")
        worst = (max(worst[0], e[0]), max(worst[1], e[1]))
        assert np.max(np.abs(lse[bb, :n] - ref_lse[bb, :n])) < LSE_TOL
        assert np.all(got[bb, n:] == 0) and np.all(lse[bb, n:] == 0)
    return worst


def test_config2_full(oracle):
    """Llama-3.1-8B-shaped verify layer, every output compared."""
    from paper_2512_14069_amd import binding as b
    a = synth.config(2).attn
    x = synth.attention_inputs(a, seed=synth.seed_for(2))
    ref, ref_lse = oracle.tree_attention(x["q"], x["k_cache"], x["v_cache"], x["parents"], x["ctx_lens"], x["n_nodes"],
                                         want_lse=True)
    got, lse = run_gpu(b, x, want_lse=True)
    check_close(got, ref, "config 2")
    assert np.max(np.abs(lse - ref_lse)) < LSE_TOL
    again = run_gpu(b, x)
    assert np.array_equal(got, again)            # bit-reproducible
    for kps in (64, 256, 512, 1024, 4096):
        check_close(run_gpu(b, x, keys_per_split=kps), ref, f"config 2 kps {kps}")


def test_config4_ragged_whole(oracle):
    """Ragged dynamic-depth batch, 16 sequences: every output compared."""
    from paper_2512_14069_amd import binding as b
    whole_config_check(oracle, b, synth.config(4).attn, synth.seed_for(4))


def test_config5_whole(oracle):
    """70B-class verify layer (4 x 16384 context, 64 / 8 heads): every output compared."""
    from paper_2512_14069_amd import binding as b
    whole_config_check(oracle, b, synth.config(5).attn, synth.seed_for(5))


def test_bad_descriptors_are_rejected():
    from paper_2512_14069_amd import binding as b
    q = torch.zeros((1, 8, 4, 96), dtype=torch.bfloat16, device="cuda")
    kv = torch.zeros((1, 2, 64, 96), dtype=torch.bfloat16, device="cuda")
    par = torch.zeros((1, 8), dtype=torch.int32, device="cuda")
    ctx = torch.zeros(1, dtype=torch.int32, device="cuda")
    with pytest.raises(b.RadarError) as e:
        b.radar_tree_attention(q, kv, kv, par, ctx, workspace=b.new_workspace(1 << 20))
    assert e.value.status == -2                                   # head dim 96 is not compiled
    q = torch.zeros((1, 8, 4, 128), dtype=torch.bfloat16, device="cuda")
    kv = torch.zeros((1, 3, 64, 128), dtype=torch.bfloat16, device="cuda")
    with pytest.raises(b.RadarError) as e:
        b.radar_tree_attention(q, kv, kv, par, ctx, workspace=b.new_workspace(1 << 20))
    assert e.value.status == -1                                   # 4 query heads over 3 KV heads


@pytest.mark.parametrize("B,Hq,Hkv,D,T,rows,one", [
    (9, 8, 8, 128, 20, 1850, True), (9, 8, 8, 128, 20, 1851, False),        # 72 KV heads
    (12, 16, 8, 128, 17, 1850, True), (8, 16, 8, 128, 20, 1300, False),     # 96, 64
    (24, 8, 8, 128, 5, 1850, True), (25, 8, 8, 128, 5, 1301, False), (32, 8, 8, 128, 5, 1700, False),      # 192, 200, 256
    (5, 48, 8, 128, 28, 1400, True), (4, 64, 8, 128, 28, 1101, False),      # 40 in groups of six and 32 in groups of eight
    (12, 8, 4, 64, 33, 2660, True), (12, 8, 4, 64, 33, 2661, False),        # 48
    (8, 16, 8, 64, 9, 12000, True), (8, 16, 8, 64, 9, 12001, False),        # 64
    (20, 12, 3, 64, 20, 9001, True), (8, 16, 4, 64, 60, 1900, True),        # 60, taken by eights; 32 with 256 units
    (8, 8, 8, 64, 3, 7001, True), (9, 8, 8, 64, 3, 7001, False),            # 64 with as few units; 72, whose ranges are seven
    (12, 32, 8, 64, 20, 2660, True), (20, 16, 4, 64, 20, 1601, False),      # more units than CUs: 96 and 80
    (16, 16, 8, 64, 60, 8000, True), (64, 4, 4, 64, 3, 12001, True),        # 128; 256, at any length
])
def test_long_single_launches_of_many_kv_heads(oracle, B, Hq, Hkv, D, T, rows, one):
    """Where there are many KV heads one launch goes on to far longer contexts; both sides of each line.  Against the oracle for
    the longest sequence, the shortest and one in between."""
    from paper_2512_14069_amd import binding as b
    nodes = [max(1, T - i % 3) for i in range(B)]
    ctx = [(rows - T) * (B - i) // B for i in range(B)]
    a = shape(B, Hq, Hkv, D, T, ctx, nodes, [max(1, min(6, n - 1)) for n in nodes], k=64)
    assert a.S == rows and (scratch_bytes(b, B, Hq, Hkv, D, T, rows) == 256) == one
    x = synth.attention_inputs(a, seed=synth.seed_for(1, rows + Hq))
    got, lse = run_gpu(b, x, want_lse=True)
    for bb in (0, B // 2, B - 1):
        n = nodes[bb]
        ref, ref_lse = oracle.tree_attention(*(np.ascontiguousarray(x[name][bb:bb + 1]) for name in ("q", "k_cache", "v_cache", "parents", "ctx_lens", "n_nodes")),
                                             want_lse=True)
        check_close(got[bb, :n], ref[0, :n], f"b={bb}")
        assert np.max(np.abs(lse[bb, :n] - ref_lse[0, :n])) < LSE_TOL
        assert np.all(got[bb, n:] == 0) and np.all(lse[bb, n:] == 0)     # unused rows are zeroed
