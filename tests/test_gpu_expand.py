"""GPU parity: radar_draft_expand / radar_draft_rerank (through the C ABI) against the
CPU oracle on the same seeded inputs.  Token ids, frontier choices, kept node sets,
parents and depths must be bit-exact; cumulative log-probabilities within 1e-5."""
import numpy as np
import pytest
import torch

from paper_2512_14069_amd import synth
from gpu_util import dev, host

pytestmark = pytest.mark.gpu

SCORE_TOL = 1e-5      # log-prob tolerance of the baseline description
GAP = 1e-4            # selections decided by less than this are not compared bit-exactly


def np_pool(cap):
    return dict(tokens=np.zeros(cap, np.int32), scores=np.zeros(cap, np.float32), parents=np.zeros(cap, np.int32))


def min_boundary_gap(scores_sorted, k):
    """Smallest gap between neighbours among the k+1 best scores."""
    top = scores_sorted[:k + 1].astype(np.float64)
    return np.min(-np.diff(top)) if len(top) > 1 else np.inf


def run_both_step(oracle, b, logits, ps, ppi, k, gpu_pool, cpu_pool, ws=None):
    count = gpu_pool.count
    r = oracle.draft_expand(logits, ps, ppi, k, cpu_pool, count)
    g = b.radar_draft_expand(dev(logits), dev(ps), dev(ppi), k, gpu_pool, workspace=ws)
    torch.cuda.synchronize()
    F = logits.shape[0]
    assert np.array_equal(host(g.cand_tokens).reshape(F, k), r["cand_tokens"])
    assert np.max(np.abs(host(g.cand_scores).reshape(F, k).astype(np.float64) - r["cand_scores"])) <= SCORE_TOL
    flat = np.sort(r["cand_scores"].reshape(-1))[::-1]
    if min_boundary_gap(flat, k) > GAP:
        assert np.array_equal(host(g.frontier_pool_idx), r["frontier_pool_idx"])
        assert np.array_equal(host(g.frontier_tokens), r["frontier_tokens"])
        assert np.max(np.abs(host(g.frontier_scores).astype(np.float64) - r["frontier_scores"])) <= SCORE_TOL
        assert np.allclose(host(g.frontier_conf), r["frontier_conf"], rtol=2e-5, atol=0)
    else:   # near-tie: the GPU's choice must still be a valid top-k of its own scores
        gs = host(g.cand_scores)
        assert np.min(gs[host(g.frontier_pool_idx) - count]) >= np.sort(gs)[::-1][k - 1]
    n = count + F * k
    assert np.array_equal(host(gpu_pool.tokens)[count:n], cpu_pool["tokens"][count:n])
    assert np.array_equal(host(gpu_pool.parents)[count:n], cpu_pool["parents"][count:n])
    assert np.max(np.abs(host(gpu_pool.scores)[count:n].astype(np.float64) - cpu_pool["scores"][count:n])) <= SCORE_TOL
    return r, g


@pytest.mark.parametrize("F,V,k", [
    (4, 4096, 4),          # config 1
    (1, 128256, 10),       # first draft call of the paper's schedule
    (10, 128256, 10),      # config 3 shape
    (3, 4097, 5),          # ragged tail, unaligned rows
    (2, 10, 10),           # k == V
    (7, 12290, 16),        # largest k, tail of two elements
    (64, 8192, 2),         # most rows
    (2, 300000, 10),       # more than 64 chunks per row: chunk lists and partials are merged in several blocks
    (40, 128256, 10),      # too many workgroups for 4 or 8 logits per lane: 16 per lane
    (5, 20000, 1),         # k = 1
])
def test_expand_step_matches_oracle(oracle, F, V, k):
    from paper_2512_14069_amd import binding as b
    rng = np.random.default_rng(synth.seed_for(3, F * 7 + k))
    logits = synth.expand_logits(rng, F, V, 3.0, normalised=(V % 2 == 0))
    ps = (-rng.random(F) * 4).astype(np.float32)
    ppi = rng.integers(-1, 5, F).astype(np.int32)
    gp, cp = b.DraftPool(5 + F * k + 3), np_pool(5 + F * k + 3)
    gp.count = 5
    gp.tokens.fill_(-7)
    cp["tokens"][:] = -7
    run_both_step(oracle, b, logits, ps, ppi, k, gp, cp)
    assert np.all(host(gp.tokens)[:5] == -7) and np.all(host(gp.tokens)[5 + F * k:] == -7)


def test_expand_exact_ties_and_special_values(oracle):
    """Equal logits are ordered by token id everywhere: duplicates inside a chunk, across
    chunks, across the top-k boundary; -inf entries and -0.0 / +0.0."""
    from paper_2512_14069_amd import binding as b
    V, k, F = 20000, 8, 4
    rng = np.random.default_rng(5)
    logits = synth.normal_logits(rng, (F, V), 1.0)
    logits[0, :] = 0.25                                   # constant row
    logits[1, [3, 4100, 8200, 12300, 16400, 19999, 7, 8]] = 9.0     # same value in several chunks
    logits[2, ::3] = -np.inf
    logits[2, [5, 4099]] = [0.0, -0.0]
    logits[2, logits[2] > 0] *= -1                        # zero is the maximum: +0.0 and -0.0 tie
    logits[3, :] = np.arange(V, dtype=np.float32) / 8     # many equal neighbours after rounding? no: strictly increasing
    ps = np.zeros(F, np.float32)
    ppi = np.full(F, -1, np.int32)
    gp, cp = b.DraftPool(F * k), np_pool(F * k)
    r = oracle.draft_expand(logits, ps, ppi, k, cp, 0)
    g = b.radar_draft_expand(dev(logits), dev(ps), dev(ppi), k, gp)
    torch.cuda.synchronize()
    assert np.array_equal(host(g.cand_tokens).reshape(F, k), r["cand_tokens"])
    assert np.array_equal(r["cand_tokens"][0], np.arange(k))
    assert np.max(np.abs(host(g.cand_scores).reshape(F, k) - r["cand_scores"])) <= SCORE_TOL


@pytest.mark.parametrize("V", [4096, 8191, 70000, 131071, 131072])       # 4, 8 and 16 logits per lane, the last with both kinds of loads; a last chunk of few logits
@pytest.mark.parametrize("k", [1, 9, 16])
def test_expand_candidate_counts_at_the_edges_of_the_lists(oracle, V, k):
    """A chunk's candidates go out as they are up to 16 and ranked beyond; up to 32 lanes per wavefront and 512
    candidates are looked at one by one.  Rows with that many logits above the rest, and one more or less, distinct
    (order decides) and equal (token id decides), scattered and side by side in one wavefront's columns."""
    from paper_2512_14069_amd import binding as b
    rng = np.random.default_rng(V + k)
    rows = []
    for n in (15, 16, 17, 31, 33, 129, 132, 512, 513, 1000):
        for equal in (False, True):
            x = synth.normal_logits(rng, (V,), 1.0)
            where = rng.permutation(min(V, 4096))[:n] if n % 2 else np.arange(n) % 256 + np.arange(n) // 256 * 1024
            x[where] = 9.0 if equal else 9.0 + rng.permutation(n).astype(np.float32) / 64
            rows.append(x)
    logits = np.stack(rows)
    F = len(rows)
    ps, ppi = np.zeros(F, np.float32), np.full(F, -1, np.int32)
    gp, cp = b.DraftPool(F * k), np_pool(F * k)
    run_both_step(oracle, b, logits, ps, ppi, k, gp, cp)


@pytest.mark.parametrize("F,k", [(8, 16), (9, 15), (16, 16), (17, 16), (2, 1), (12, 10)])    # 128, 135, 256, 272, 2 and 120 candidates
def test_expand_survivors_at_the_edges_of_the_rankings(oracle, F, k):
    """What passes a wavefront's threshold is ranked in four parts up to 16 keys, in two up to 32, one by one beyond: rows with that
    many logits above the rest over all chunks, equal or apart, and every second row like the one before it with the same parent score,
    so that the frontier's candidates are equal in pairs (their number decides)."""
    from paper_2512_14069_amd import binding as b
    V = 60000
    rng = np.random.default_rng(F * 100 + k)
    counts = (15, 16, 17, 31, 32, 33, 64, 65, 200)
    logits = np.empty((F, V), np.float32)
    for f in range(F):
        n = counts[(f // 2 + F) % len(counts)]
        if f % 2 == 0:
            logits[f] = synth.normal_logits(rng, (V,), 1.0)
            logits[f, rng.permutation(V)[:n]] = 9.0 if n % 2 else 9.0 + rng.permutation(n).astype(np.float32) / 64
        else:
            logits[f] = logits[f - 1]
    ps, ppi = -(np.arange(F) // 2).astype(np.float32) / 8, np.full(F, -1, np.int32)
    cp = np_pool(F * k)
    g = b.radar_draft_expand(dev(logits), dev(ps), dev(ppi), k, b.DraftPool(F * k))
    r = oracle.draft_expand(logits, ps, ppi, k, cp, 0)
    torch.cuda.synchronize()
    assert np.array_equal(host(g.cand_tokens).reshape(F, k), r["cand_tokens"])
    got = host(g.cand_scores)
    assert np.max(np.abs(got.reshape(F, k) - r["cand_scores"])) <= SCORE_TOL
    best = np.lexsort((np.arange(F * k), -got.astype(np.float64)))[:k]           # of the device's own scores: score, then number
    assert np.array_equal(host(g.frontier_pool_idx), best)


@pytest.mark.parametrize("V", [131071, 131073, 200001, 262143, 262144, 262145])
@pytest.mark.parametrize("F,k", [(1, 10), (4, 16), (8, 10), (10, 3)])
def test_expand_rows_of_many_chunks(oracle, V, F, k):
    """Rows of more than 131072 logits: 16 chunks of the most logits per lane where they take 16-byte loads, more chunks of fewer
    where they do not, or both if there are many rows."""
    from paper_2512_14069_amd import binding as b
    rng = np.random.default_rng(V + F)
    logits = np.stack([synth.normal_logits(rng, (V,), 3.0) for _ in range(F)])
    logits[:, -1] = logits.max(axis=1) - 0.25                    # the last chunk's few logits count
    ps, ppi = rng.standard_normal(F).astype(np.float32), np.full(F, -1, np.int32)
    run_both_step(oracle, b, logits, ps, ppi, k, b.DraftPool(F * k), np_pool(F * k))


@pytest.mark.parametrize("cfg,first_F", [(1, 1), (3, 1), (3, 10)])
def test_expand_chain_and_rerank_match_oracle(oracle, cfg, first_F):
    """The whole drafting phase of a cycle: the paper's schedule (first call on the root
    alone, then k rows per call) or the timed shape (k rows every call), each step checked
    on identical inputs, then rerank to the best N and every tree field compared."""
    from paper_2512_14069_amd import binding as b
    c = synth.config(cfg)
    rng = np.random.default_rng(synth.seed_for(cfg, first_F))
    k, V, steps, N = c.k, c.vocab, c.expand_steps, c.N
    cap = first_F * k + (steps - 1) * k * k
    gp, cp = b.DraftPool(cap), np_pool(cap)
    ws = b.new_workspace(b.radar_draft_expand_workspace_bytes(b.expand_desc(k, V, k, 0, cap)))
    ps = np.zeros(first_F, np.float32) if first_F == 1 else (-rng.random(first_F)).astype(np.float32)
    ppi = np.full(first_F, -1, np.int32)
    for s in range(steps):
        logits = synth.expand_logits(rng, len(ps), V, c.logit_std, normalised=True)
        r, g = run_both_step(oracle, b, logits, ps, ppi, k, gp, cp, ws=ws)   # one workspace reused by all steps
        ps, ppi = r["frontier_scores"].copy(), r["frontier_pool_idx"].copy()
    assert gp.count == cap
    tree = oracle.draft_rerank(cp, cap, N, root_token=1234)
    # feed the GPU rerank the oracle's pool so that both order identical scores
    gp.tokens.copy_(dev(cp["tokens"])); gp.scores.copy_(dev(cp["scores"])); gp.parents.copy_(dev(cp["parents"]))
    t = b.radar_draft_rerank(gp, N, 1234)
    torch.cuda.synchronize()
    assert int(host(t.n_nodes)[0]) == tree["n_nodes"]
    for name in ("tokens", "parents", "depth", "pool_idx"):
        assert np.array_equal(host(getattr(t, name)), tree[name]), name
    assert np.array_equal(host(t.scores), tree["scores"])
    bad = b.radar_debug_validate_tree(t.parents.view(1, -1), t.n_nodes)
    assert int(host(bad)[0]) == 0


@pytest.mark.parametrize("count,N", [(0, 5), (3, 10), (64, 63), (810, 60), (4096, 60), (257, 1)])
def test_rerank_sizes_and_ties(oracle, count, N):
    from paper_2512_14069_amd import binding as b
    rng = np.random.default_rng(count + N)
    gp = b.DraftPool(max(count, 1))
    cp = np_pool(max(count, 1))
    # a forest whose scores never grow downwards, with exact score ties
    for i in range(count):
        par = -1 if i < 4 or rng.random() < 0.1 else int(rng.integers(0, i))
        drop = float(rng.integers(0, 4)) * 0.25            # many exact ties (including 0 drop)
        cp["parents"][i] = par
        cp["scores"][i] = (cp["scores"][par] if par >= 0 else 0.0) - drop
        cp["tokens"][i] = int(rng.integers(0, 1000))
    gp.tokens.copy_(dev(cp["tokens"])); gp.scores.copy_(dev(cp["scores"])); gp.parents.copy_(dev(cp["parents"]))
    gp.count = count
    tree = oracle.draft_rerank(cp, count, N, root_token=7)
    t = b.radar_draft_rerank(gp, N, 7)
    torch.cuda.synchronize()
    assert int(host(t.n_nodes)[0]) == tree["n_nodes"]
    for name in ("tokens", "parents", "depth", "pool_idx", "scores"):
        assert np.array_equal(host(getattr(t, name)), tree[name]), name


@pytest.mark.parametrize("count", [1, 127, 128, 129, 480, 481, 512, 1024, 1025, 4096])
@pytest.mark.parametrize("shape", ["equal", "two_lanes", "chain"])
def test_rerank_survivors_and_depths_at_their_edges(oracle, count, shape):
    """All scores equal (everything survives the threshold: up to 128 are ranked in one pass, up to 480 in slots that are cleared
    beforehand), the largest scores in one pair of lanes, and a chain as deep as the tree can be."""
    from paper_2512_14069_amd import binding as b
    rng = np.random.default_rng(count)
    gp, cp = b.DraftPool(count), np_pool(count)
    i = np.arange(count)
    cp["parents"][:] = i - 1 if shape == "chain" else -1 if shape == "two_lanes" else np.where(i < 10, -1, i // 7 - 1)
    cp["scores"][:] = 0.0 if shape == "equal" else -0.125 * i if shape == "chain" else np.where(i % 256 < 2, -0.5, -1.0 - 0.001 * i)
    cp["tokens"][:] = rng.integers(0, 1000, count)
    gp.tokens.copy_(dev(cp["tokens"])); gp.scores.copy_(dev(cp["scores"])); gp.parents.copy_(dev(cp["parents"]))
    gp.count = count
    for N in (1, 63):
        tree = oracle.draft_rerank(cp, count, N, root_token=7)
        t = b.radar_draft_rerank(gp, N, 7)
        torch.cuda.synchronize()
        assert int(host(t.n_nodes)[0]) == tree["n_nodes"]
        for name in ("tokens", "parents", "depth", "pool_idx", "scores"):
            assert np.array_equal(host(getattr(t, name)), tree[name]), (name, N)


def test_expand_counts_on_one_counter_or_by_rows(oracle):
    """Up to 96 workgroups count on one counter, more of them by rows: both sides of that line in turn on one
    workspace, each call starting from what the one before it left."""
    from paper_2512_14069_amd import binding as b
    rng = np.random.default_rng(96)
    k, V = 8, 32000                                                # eight chunks per row
    ws = b.new_workspace(b.radar_draft_expand_workspace_bytes(b.expand_desc(13, V, k, 0, 4096)))
    for F in (12, 13, 1, 13, 12, 11):
        logits = synth.expand_logits(rng, F, V, 2.0)
        gp, cp = b.DraftPool(F * k), np_pool(F * k)
        run_both_step(oracle, b, logits, (-rng.random(F)).astype(np.float32), np.full(F, -1, np.int32), k, gp, cp, ws=ws)
        assert int(ws[:4096].view(torch.int32).abs().sum().item()) == 0   # counters left clean


def test_expand_is_deterministic_and_workspace_reusable(oracle):
    from paper_2512_14069_amd import binding as b
    rng = np.random.default_rng(1)
    logits = dev(synth.expand_logits(rng, 10, 128256, 3.0))
    ps, ppi = dev(np.zeros(10, np.float32)), dev(np.full(10, -1, np.int32))
    ws = b.new_workspace(b.radar_draft_expand_workspace_bytes(b.expand_desc(10, 128256, 10, 0, 100)))
    outs = []
    for _ in range(3):
        gp = b.DraftPool(100)
        g = b.radar_draft_expand(logits, ps, ppi, 10, gp, workspace=ws)
        torch.cuda.synchronize()
        outs.append((host(g.cand_tokens).copy(), host(g.cand_scores).copy(), host(g.frontier_pool_idx).copy()))
    for o in outs[1:]:
        assert all(np.array_equal(x, y) for x, y in zip(o, outs[0]))
    assert int(ws[:16384].view(torch.int32).abs().sum().item()) == 0    # counters left clean


@pytest.mark.parametrize("V", [1, 2, 3, 5, 1026, 4095, 16387, 65534, 130001])   # rows shorter than a load, every remainder of four, each plan
@pytest.mark.parametrize("offset", [0, 1])                                     # floats between the logits' start and a multiple of 16 bytes
def test_expand_row_ends_at_any_alignment(oracle, V, offset):
    """The best logits of each row are its last ones, which a 16-byte load reaches only from before where it belongs, and its
    first; rows of any alignment, and a row that is preceded and followed by larger values that are not its own."""
    from paper_2512_14069_amd import binding as b
    rng = np.random.default_rng(synth.seed_for(3, 700 + V % 1000 + offset))
    F, k = 5, min(V, 7)
    logits = synth.expand_logits(rng, F, V, 1.0)
    for f in range(F):
        for i, j in enumerate(range(max(0, V - 4), V)):
            logits[f, j] = 8.0 + f + ((i * 3 + f) % 4) * 0.5
        logits[f, 0] = 7.0 if V > 4 else logits[f, 0]
    held = torch.full((F * V + 16,), 100.0, device="cuda")
    held[4 + offset:4 + offset + F * V] = dev(logits).view(-1)
    x = held[4 + offset:4 + offset + F * V].view(F, V)
    assert x.data_ptr() % 16 == 4 * offset
    ps, ppi = (-rng.random(F) * 4).astype(np.float32), np.full(F, -1, np.int32)
    cp = np_pool(F * k)
    r = oracle.draft_expand(logits, ps, ppi, k, cp, 0)
    g = b.radar_draft_expand(x, dev(ps), dev(ppi), k, b.DraftPool(F * k))
    assert np.array_equal(host(g.cand_tokens).reshape(F, k), r["cand_tokens"])
    assert np.max(np.abs(host(g.cand_scores).reshape(F, k).astype(np.float64) - r["cand_scores"])) <= SCORE_TOL


@pytest.mark.parametrize("F,k", [(16, 16), (17, 16), (32, 16), (33, 16), (64, 16), (64, 5), (52, 5), (64, 4)])    # 256 ... 1024 candidates, 256 to a wavefront
@pytest.mark.parametrize("best", ["anywhere", "last rows", "equal"])
def test_expand_frontier_of_many_candidates(oracle, F, k, best):
    """The frontier's entries come from all wavefronts' shares of the candidates, from the last one's alone, and from rows that are the
    same (the lowest candidate indices win)."""
    from paper_2512_14069_amd import binding as b
    rng = np.random.default_rng(synth.seed_for(3, 800 + F + k))
    V = 600
    logits = synth.expand_logits(rng, F, V, 2.0)
    ps = (-rng.random(F) * 3).astype(np.float32)
    if best == "last rows":
        ps -= np.where(np.arange(F) < F - 2, np.float32(20), np.float32(0))
    elif best == "equal":
        logits[:] = logits[0]
        ps[:] = -1.0
    cp = np_pool(F * k)
    r = oracle.draft_expand(logits, ps, np.full(F, -1, np.int32), k, cp, 0)
    g = b.radar_draft_expand(dev(logits), dev(ps), dev(np.full(F, -1, np.int32)), k, b.DraftPool(F * k))
    assert np.array_equal(host(g.cand_tokens).reshape(F, k), r["cand_tokens"])
    flat = np.sort(r["cand_scores"].reshape(-1))[::-1]
    if best == "equal" or min_boundary_gap(flat, k) > GAP:
        assert np.array_equal(host(g.frontier_pool_idx), r["frontier_pool_idx"])
        assert np.array_equal(host(g.frontier_tokens), r["frontier_tokens"])
    gs = host(g.cand_scores)
    assert np.array_equal(np.sort(gs)[::-1][:k], np.sort(gs[host(g.frontier_pool_idx)])[::-1])


@pytest.mark.parametrize("B,F,V,k", [(1, 3, 8192, 6), (1, 10, 131072, 10), (1, 20, 8192, 5), (1, 64, 4096, 16), (1, 2, 524288, 16), (1, 10, 128257, 10), (40, 10, 32768, 10)])   # the last in two launches
def test_rows_with_fewer_numbers_than_candidates(B, F, V, k):
    """Rows with no logit that is a number, with fewer than k, with k and one more; rows of numbers among them.  Which tokens such a row
    gives is not specified, but they are k different ones of the vocabulary, a NaN's with a NaN score, they are in the pool too, and the frontier is
    k different candidates: nothing of an earlier call is left in any output, and a repeated call gives the same bits."""
    from paper_2512_14069_amd import binding as b
    rng = np.random.default_rng(synth.seed_for(3, 950 + F))
    logits = rng.standard_normal((B, F, V), dtype=np.float32)
    kept = [None if f % 3 == 2 else (0, 1, k - 1, k, k + 1)[(f - f // 3) % 5] for f in range(F)]
    for f, n in enumerate(kept):
        if n is not None:
            at = np.sort(rng.permutation(V)[:n])
            row = np.full(V, np.nan, np.float32)
            row[at] = logits[0, f, at]
            logits[:, f] = row
    x, ps, ppi = dev(logits), dev(np.zeros((B, F), np.float32)), dev(np.full((B, F), -1, np.int32))
    runs = []
    for left in (123, 77):                                         # what an earlier call may have left
        pool, out = b.DraftPool(F * k, B=B), b.ExpandOut(F, k, "cuda", B=B)
        for t in list(vars(out).values()) + [pool.tokens, pool.scores, pool.parents]:
            t.fill_(left)
        b.radar_draft_expand_batch(x, ps, ppi, k, pool, out=out)
        torch.cuda.synchronize()
        runs.append({n: host(t).copy() for n, t in list(vars(out).items()) + [("pool_" + n, getattr(pool, n)) for n in ("tokens", "scores", "parents")]})
    for n in runs[0]:
        assert np.array_equal(runs[0][n], runs[1][n], equal_nan=True), n
    r = runs[0]
    tok, sc = r["cand_tokens"].reshape(B, F, k), r["cand_scores"].reshape(B, F, k)
    for f, n in enumerate(kept):
        if n is None:
            assert np.all(np.isfinite(sc[:, f])) and np.all(tok[:, f] >= 0)
            continue
        for t, v in zip(tok[:, f], sc[:, f]):
            assert np.all((t >= 0) & (t < V)) and len(set(t)) == k, (f, n)
            assert np.all(np.isnan(v[np.isnan(logits[0, f, t])]))
    assert np.array_equal(r["pool_tokens"].reshape(B, -1), tok.reshape(B, -1))
    assert np.array_equal(r["pool_scores"].reshape(B, -1), sc.reshape(B, -1), equal_nan=True)
    assert np.all(r["pool_parents"] == -1)
    for s in range(B):
        at = r["frontier_pool_idx"].reshape(B, k)[s]
        assert len(set(at)) == k and at.min() >= 0 and at.max() < F * k
        assert np.array_equal(r["frontier_tokens"].reshape(B, k)[s], tok[s].reshape(-1)[at])
        assert np.array_equal(r["frontier_scores"].reshape(B, k)[s], sc[s].reshape(-1)[at], equal_nan=True)
