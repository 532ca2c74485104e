"""GPU parity: radar_verify_accept (through the C ABI) against the CPU oracle.
Accepted lengths, paths and bonus tokens must be bit-exact, for EVERY sequence.  In sampling
mode the inputs are made tie-free first: a sequence in which the oracle reports a decision
within MARGIN of its threshold gets fresh seeded uniforms (the margins themselves are pinned
in tests/test_oracle_margins.py).  Over a 128K vocabulary one token carries about 1e-5 of the
mass, so the inverse-CDF draw always lands within that distance of a boundary and the device
has to resolve far finer than that.  It sums exponentials in fp64 (fp32 only inside expf),
which leaves about 1e-8; MARGIN sits an order of magnitude above."""
import numpy as np
import pytest
import torch

from paper_2512_14069_amd import synth
from gpu_util import dev, host, tie_free_uniforms

pytestmark = pytest.mark.gpu

MARGIN = 2e-7


def run_gpu(b, x, mode, temperature=1.0, D_max=None, ws=None, use_n_nodes=True):
    out = b.radar_verify_accept(dev(x["target_logits"]), dev(x["draft_tokens"]), dev(x["parents"]),
                                dev(x["n_nodes"]) if use_n_nodes else None,
                                dev(x["uniforms"]) if mode == 1 else None,
                                mode=mode, temperature=temperature, D_max=D_max, workspace=ws)
    torch.cuda.synchronize()
    return [host(t) for t in out]


def compare(oracle, b, x, mode, temperature=1.0):
    if mode == 1:
        def clear(u):
            m = oracle.accept_margins(x["target_logits"], x["draft_tokens"], x["parents"], x["n_nodes"], u, temperature)
            return (m[:, 0] > MARGIN) & (m[:, 1] > MARGIN)
        x = dict(x, uniforms=tie_free_uniforms(clear, x["uniforms"], np.random.default_rng(int(x["uniforms"].size))))
    ref = oracle.verify_accept(x["target_logits"], x["draft_tokens"], x["parents"], x["n_nodes"],
                               x["uniforms"] if mode == 1 else None, mode=mode, temperature=temperature)
    got = run_gpu(b, x, mode, temperature)
    for name, g, r in zip(("accept_len", "accept_path", "bonus_token"), got, ref):
        assert np.array_equal(g, r), (name, np.nonzero((g != r).reshape(len(r), -1).any(axis=1))[0][:8])
    return ref, got


def counters_are_clean(ws, B, T):
    """The arrival counters at the head of the workspace, 64 bytes apart: one per row, two per sequence."""
    return int(ws[:64 * (B * T + 2 * B)].view(torch.int32).abs().max().item()) == 0


def small_shape(B, T, nn, dep, k=4):
    return synth.AttnShape(B=B, Hq=1, Hkv=1, D=8, T=T, ctx_lens=(0,) * B, n_nodes=nn, depths=dep, k=k)


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("V", [4096, 5000, 128256])
def test_single_sequence(oracle, mode, V):
    from paper_2512_14069_amd import binding as b
    a = small_shape(1, 16, (16,), (4,))
    x = synth.accept_inputs(a, V, seed=synth.seed_for(1, V % 97 + mode), plant=0.8)
    if mode == 1:   # correlate tokens with the target so that some are accepted
        x["target_logits"] = (x["target_logits"] * 0.5).astype(np.float32)
    ref, _ = compare(oracle, b, x, mode)
    if mode == 0:
        assert ref[0][0] >= 1          # planting gives a non-trivial path


@pytest.mark.parametrize("mode", [0, 1])
def test_config2_shape(oracle, mode):
    from paper_2512_14069_amd import binding as b
    c = synth.config(2)
    x = synth.accept_inputs(c.attn, c.vocab, seed=synth.seed_for(2, mode), plant=0.75)
    compare(oracle, b, x, mode)


def test_config4_ragged_full_size(oracle):
    """Configuration 4 at full size: 16 sequences with trees of 2..60 nodes, V = 128256, greedy."""
    from paper_2512_14069_amd import binding as b
    c = synth.config(4)
    x = synth.accept_inputs(c.attn, c.vocab, seed=synth.seed_for(4, 3), plant=0.75)
    ref, _ = compare(oracle, b, x, 0)
    assert ref[0].max() >= 2 and ref[0].min() <= 1       # accepted lengths are spread


@pytest.mark.parametrize("mode", [0, 1])
def test_config5_full_size(oracle, mode):
    """Configuration 5 at full size: four sequences of 60 rows, V = 128256, greedy and sampled."""
    from paper_2512_14069_amd import binding as b
    c = synth.config(5)
    x = synth.accept_inputs(c.attn, c.vocab, seed=synth.seed_for(5, mode), plant=0.75)
    compare(oracle, b, x, mode)


@pytest.mark.parametrize("mode,temperature", [(0, 1.0), (1, 1.0), (1, 0.6)])
def test_ragged_batch(oracle, mode, temperature):
    from paper_2512_14069_amd import binding as b
    B = 6
    rng = np.random.default_rng(17)
    dep = tuple(int(d) for d in rng.integers(1, 6, B))
    nn = tuple(int(rng.integers(d + 1, min(30, 1 + 4 + 16 * (d - 1)) + 1)) for d in dep)
    nn = (1,) + nn[1:]                    # a sequence that is only its root
    dep = (1,) + dep[1:]
    a = small_shape(B, 30, nn, dep)
    x = synth.accept_inputs(a, 20011, seed=99 + mode, plant=0.7, shuffle=True)
    compare(oracle, b, x, mode, temperature)


def test_sampling_many_uniform_vectors_small_tree(oracle):
    """Many sequences share one small tree and logits; only the uniforms differ, so every
    branch of the walk (accept first / later sibling, reject all, leaf) is exercised."""
    from paper_2512_14069_amd import binding as b
    B, T, V = 256, 9, 1000
    rng = np.random.default_rng(3)
    parents, tokens, depths = synth.make_tree(rng, T, 3, 3, V)
    logits = synth.normal_logits(rng, (T, V), 2.0)
    for c in range(1, T):                   # give the draft tokens real mass
        logits[parents[c], tokens[c]] = 8.0
    x = dict(target_logits=np.broadcast_to(logits, (B, T, V)).copy(),
             draft_tokens=np.broadcast_to(tokens, (B, T)).copy(),
             parents=np.broadcast_to(parents, (B, T)).copy(),
             n_nodes=np.full(B, T, np.int32), uniforms=rng.random((B, T + 1), dtype=np.float32))
    ref, got = compare(oracle, b, x, 1)
    assert len(set(ref[0].tolist())) >= 3       # several different accepted lengths occurred


def test_greedy_extremes_and_dmax(oracle):
    from paper_2512_14069_amd import binding as b
    V, n = 128256, 60
    rng = np.random.default_rng(8)
    parents = synth.chain_tree(n)
    tokens = rng.integers(0, V, n).astype(np.int32)
    logits = synth.gumbel_logits(rng, (n, V))
    for i in range(n - 1):
        logits[i, tokens[i + 1]] = 70.0
    x = dict(target_logits=logits[None], draft_tokens=tokens[None], parents=parents[None],
             n_nodes=np.array([n], np.int32), uniforms=None)
    ref, got = compare(oracle, b, x, 0)
    assert got[0][0] == n - 1                   # chain fully accepted: depth 59
    # walk capped by D_max
    got = run_gpu(b, x, 0, D_max=5)
    assert got[0][0] == 5 and list(got[1][0]) == [0, 1, 2, 3, 4, 5]
    # n_nodes = NULL means every slot is a node
    got = run_gpu(b, x, 0, use_n_nodes=False)
    assert got[0][0] == n - 1


def test_workspace_reuse_and_determinism(oracle):
    from paper_2512_14069_amd import binding as b
    c = synth.config(2)
    x = synth.accept_inputs(c.attn, c.vocab, seed=5)
    ws = b.new_workspace(b.radar_verify_accept_workspace_bytes(b.accept_desc(1, 60, c.vocab, 59, 1, 1.0)))
    first = run_gpu(b, x, 1, ws=ws)
    for mode in (0, 1, 1):
        again = run_gpu(b, x, mode, ws=ws)
        if mode == 1:
            assert all(np.array_equal(p, q) for p, q in zip(first, again))
    assert counters_are_clean(ws, 1, 60)


def test_wide_levels_and_duplicate_sibling_tokens(oracle):
    """Star-shaped trees (up to 63 children of the root, tried all at once on the device) whose
    sibling tokens repeat: the earliest sibling with a token wins, later copies are skipped, and
    the residual draw removes every tried token.  Uniforms differ per sequence."""
    from paper_2512_14069_amd import binding as b
    B, T, V = 192, 64, 3000
    rng = np.random.default_rng(11)
    parents = synth.star_tree(T)
    parents[40:] = rng.integers(1, 8, size=T - 40)          # a second, narrower level under nodes 1..7
    tokens = rng.integers(0, V, size=T).astype(np.int32)
    tokens[5] = tokens[2]; tokens[17] = tokens[2]; tokens[30] = tokens[9]     # repeated sibling tokens
    logits = synth.normal_logits(rng, (T, V), 1.5)
    for c in range(1, T):
        logits[parents[c], tokens[c]] = 3.0 + 0.02 * c       # every draft token carries visible mass
    x = dict(target_logits=np.broadcast_to(logits, (B, T, V)).copy(),
             draft_tokens=np.broadcast_to(tokens, (B, T)).copy(),
             parents=np.broadcast_to(parents, (B, T)).copy(),
             n_nodes=np.full(B, T, np.int32), uniforms=rng.random((B, T + 1), dtype=np.float32))
    ref, got = compare(oracle, b, x, 1)
    assert len(set(ref[0].tolist())) >= 2 and (ref[0] == 0).any() and (ref[0] > 0).any()
    compare(oracle, b, x, 0)


@pytest.mark.parametrize("mode", [0, 1])
def test_large_vocabulary_many_blocks(oracle, mode):
    """More than 128 blocks of 1024 logits per row: the merge and the residual scan loop."""
    from paper_2512_14069_amd import binding as b
    V = 300001
    a = small_shape(2, 12, (12, 7), (3, 2), k=3)
    x = synth.accept_inputs(a, V, seed=77)
    compare(oracle, b, x, mode)


def log_mass(rows):
    """Logarithm of each row's sum of exponentials."""
    m = rows.max(axis=-1).astype(np.float64)
    return m + np.log(np.exp(rows - m[..., None]).sum(axis=-1))


@pytest.mark.parametrize("V", [65536, 65537, 131072, 131073, 196609])
def test_edges_of_the_groups_of_blocks(oracle, V):
    """64, 65, 128, 129 and 193 blocks of 1024 logits per row: the merging wavefront takes their sums and maxima 64 at a time.  The last block
    decides: its last logit weighs as much as the rest of the row, so does a child's token.  The child (a third of the row, half without the last
    block) is rejected at 0.4 in the first sequence; the bonus token of the others is drawn from the last block."""
    from paper_2512_14069_amd import binding as b
    a = small_shape(3, 9, (9, 1, 4), (3, 0, 2), k=3)
    x = synth.accept_inputs(a, V, seed=79, plant=0.0)
    tl, tok, par, u = (x[n] for n in ("target_logits", "draft_tokens", "parents", "uniforms"))
    rest = log_mass(tl)
    tl[:, :, -1] = rest
    first = [[c for c in range(1, x["n_nodes"][s]) if par[s, c] == 0][:1] for s in range(3)]
    for s, kids in enumerate(first):
        for c in kids:
            tl[s, 0, tok[s, c]] = rest[s, 0]
    u[0, :-1] = 0.4
    u[2, :-1] = 0.999
    u[1:, -1] = 0.8
    ref, _ = compare(oracle, b, x, 1)
    masked = tl.copy()
    masked[:, :, (V - 1) // 1024 * 1024:] = -100.0
    without = oracle.verify_accept(masked, tok, par, x["n_nodes"], u, mode=1, temperature=1.0)
    assert ref[0][0] == 0 and without[0][0] > 0                             # what the row's sum says
    assert (ref[2][1:] == V - 1).all() and (without[2][1:] != V - 1).all()  # where the draw lands


def test_draws_behind_the_first_128_blocks(oracle):
    """Bonus tokens in blocks 128 ... 191, 192 ... 255 and from 256 on: the draw goes over the masses 128 blocks at a time.  Three sequences each of
    a root alone, of a root whose three children are rejected (one token in each of these groups, a tenth of the row each) and of a root with
    an accepted child.  The logits are ordinary ones, a token has about 3e-6 of the row: a mass that is lost or counted twice moves the draw."""
    from paper_2512_14069_amd import binding as b
    V, B, T = 300001, 9, 4
    groups = ((128, 192), (192, 256), (256, (V - 1) // 1024 + 1))
    rng = np.random.default_rng(synth.seed_for(30, 41))
    tl = synth.normal_logits(rng, (B, T, V), 1.5)
    par = np.tile(np.array([-1, 0, 0, 0], np.int32), (B, 1))
    tok = np.zeros((B, T), np.int32)
    nn = np.array([1, 1, 1, 4, 4, 4, 2, 2, 2], np.int32)
    u = np.zeros((B, T + 1), np.float32)
    for s in range(B):
        lo, hi = groups[s % 3]
        tok[s, 1:] = [g[0] * 1024 + 5000 + 700 * s for g in groups]
        if s >= 3:
            tl[s, 0, tok[s, 1:nn[s]]] = log_mass(tl[s, 0]) - np.log(7.0)
        u[s, 1:nn[s]] = 0.99999 if s < 6 else 0.0
        # the place in the distribution of the row that is drawn from, without the rejected tokens
        e = np.exp(tl[s, 1 if s >= 6 else 0].astype(np.float64))
        if 3 <= s < 6:
            e[tok[s, 1:]] = 0.0
        cdf = np.cumsum(e) / e.sum()
        at = int(rng.integers(lo * 1024, min(hi * 1024, V)))
        while e[at] < 4 * MARGIN * e.sum():                                 # wide enough that its middle is clear of its ends
            at -= 1
        u[s, -1] = (cdf[at - 1] + cdf[at]) / 2
    x = dict(target_logits=tl, draft_tokens=tok, parents=par, n_nodes=nn, uniforms=u)
    margins = oracle.accept_margins(tl, tok, par, nn, u, 1.0)
    assert (margins > MARGIN).all()                                         # these uniforms are the ones compared
    ref, _ = compare(oracle, b, x, 1)
    for s in range(B):
        assert groups[s % 3][0] <= ref[2][s] // 1024 < groups[s % 3][1]
    assert (ref[0][:6] == 0).all() and (ref[0][6:] == 1).all()


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("B,T,V,chain", [(3, 64, 40000, True), (6, 64, 34000, False), (12, 64, 65539, False),
                                          (13, 64, 61001, True)])       # the rows behind the roots wait for the walk
def test_walk_carried_from_row_to_row(oracle, mode, B, T, V, chain):
    """The walk that goes on with whichever row completes next: trees as deep as they get, launches with more workgroups
    than start at once (rows off the path are left unread), two blocks per wavefront with odd row lengths, and one
    workspace for several inputs in a row."""
    from paper_2512_14069_amd import binding as b
    ws = b.new_workspace(b.radar_verify_accept_workspace_bytes(b.accept_desc(B, T, V, T - 1, mode, 1.0)))
    for seed in (1, 2):
        x = synth.accept_inputs(small_shape(B, T, (T,) * (B - 1) + (1,), (8,) * B, k=10), V, seed=70 + seed, plant=0.0 if chain else 0.9)
        if chain:
            x["parents"][:] = synth.chain_tree(T)
            x["n_nodes"][:] = T
            nodes = np.arange(1, T)
            for s in range(B):                            # rows that prefer their own child, up to some depth
                last = T if s == 0 else 5 * s
                x["target_logits"][s, nodes[:last - 1] - 1, x["draft_tokens"][s, 1:last]] = synth.PLANT_LOGIT
        compare(oracle, b, x, mode)
        ref = run_gpu(b, x, mode)
        assert all(np.array_equal(p, q) for p, q in zip(ref, run_gpu(b, x, mode, ws=ws)))
        assert not chain or ref[0].max() == T - 1
    assert counters_are_clean(ws, B, T)


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("nodes", [(6,), (11, 12, 13, 24, 25), (7, 8, 9, 11, 12), (1, 64, 2, 40)])
def test_small_trees_in_a_large_launch(oracle, mode, nodes):
    """A launch that is large by T_max: trees too small to wait for the roots, trees on both sides of that line (8 nodes
    greedy, 12 sampled), and both in one batch."""
    from paper_2512_14069_amd import binding as b
    B, T, V = 16, 64, 125001 if nodes[0] in (7, 11) else 50001
    nn = tuple(nodes[i % len(nodes)] for i in range(B))
    x = synth.accept_inputs(small_shape(B, T, nn, tuple(max(1, min(5, n - 1)) for n in nn), k=10), V, seed=81 + nodes[0], plant=0.9, shuffle=True)
    ref, _ = compare(oracle, b, x, mode)
    assert mode == 1 or ref[0].max() >= 2


@pytest.mark.parametrize("V,B", [(1, 2), (2, 3), (3, 2), (5, 2), (1025, 3), (2050, 3), (4099, 3), (4100, 3), (20003, 40)])   # the last: two blocks per wavefront
@pytest.mark.parametrize("offset", [0, 2])
def test_row_ends_at_any_alignment(oracle, V, B, offset):
    """Rows whose decisive logits are the last ones, rows shorter than a load, logits that start off a multiple of 16 bytes; larger values that
    are not the rows' own before and behind them."""
    from paper_2512_14069_amd import binding as b
    rng = np.random.default_rng(synth.seed_for(30, 900 + V % 100 + offset))
    T, D = (20, 4) if V > 1000 else (3, 2)
    par = np.full((B, T), -1, np.int32)
    tok = np.zeros((B, T), np.int32)
    for s in range(B):
        for n in range(1, T):
            par[s, n] = n - 1 if n <= D else (n - 1) // 4
            tok[s, n] = max(0, V - 1 - n % 4)
    logits = rng.standard_normal((B, T, V), dtype=np.float32)
    logits[:, :, max(0, V - 4):] += 9.0
    held = torch.full((B * T * V + 16,), 100.0, device="cuda")
    held[4 + offset:4 + offset + B * T * V] = dev(logits).view(-1)
    x = held[4 + offset:4 + offset + B * T * V].view(B, T, V)
    nn = np.full(B, T, np.int32)

    def clear(u):
        m = oracle.accept_margins(logits, tok, par, nn, u, 1.0)
        return (m[:, 0] > MARGIN) & (m[:, 1] > MARGIN)
    u = tie_free_uniforms(clear, rng.random((B, T + 1), dtype=np.float32), rng)
    for mode in (0, 1):
        ref = oracle.verify_accept(logits, tok, par, nn, u if mode else None, mode=mode, temperature=1.0)
        got = b.radar_verify_accept(x, dev(tok), dev(par), dev(nn), dev(u) if mode else None, mode=mode, temperature=1.0)
        for g, r in zip(got, ref):
            assert np.array_equal(host(g), r), mode
