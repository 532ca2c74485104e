"""GPU tests of the calls around the three steps: pre-marshalled calls and per-kernel timing."""
import numpy as np
import pytest
import torch

from paper_2512_14069_amd import synth
from gpu_util import bf16_dev, dev, host

pytestmark = pytest.mark.gpu


def test_prepared_calls_replay_the_same_work(oracle):
    from paper_2512_14069_amd import binding as b
    a = synth.config(1).attn
    x = synth.attention_inputs(a, seed=5)
    q, kc, vc = bf16_dev(x["q"]), bf16_dev(x["k_cache"]), bf16_dev(x["v_cache"])
    par, ctx, nn = dev(x["parents"]), dev(x["ctx_lens"]), dev(x["n_nodes"])
    direct = b.radar_tree_attention(q, kc, vc, par, ctx, nn)
    call = b.radar_tree_attention(q, kc, vc, par, ctx, nn, prepared=True)
    assert isinstance(call, b.BoundCall)
    call.out.fill_(7.0)
    out = call()
    torch.cuda.synchronize()
    assert torch.equal(out, direct)
    q.mul_(0.5)                                  # same pointers, new contents: a replay sees them
    again = b.radar_tree_attention(q, kc, vc, par, ctx, nn)
    assert torch.equal(call(), again)


def test_profile_reports_each_kernel(oracle):
    from paper_2512_14069_amd import binding as b
    rng = np.random.default_rng(2)
    F, V, k = 3, 5000, 4
    logits = dev(synth.normal_logits(rng, (F, V), 2.0))
    ps = torch.zeros(F, device="cuda")
    ppi = torch.full((F,), -1, dtype=torch.int32, device="cuda")
    pool = b.DraftPool(4 * F * k)
    b.radar_profile_begin(16)
    for _ in range(3):
        b.radar_draft_expand(logits, ps, ppi, k, pool)
    b.radar_draft_rerank(pool, 5, 1)
    torch.cuda.synchronize()
    t = b.radar_profile_end()
    assert t["expand"]["calls"] == 3 and t["rerank"]["calls"] == 1
    assert "zero_fill" in t                      # the workspaces made on the way were cleared by a kernel
    for v in t.values():
        assert 0.0 < v["min_us"] <= v["mean_us"] <= v["max_us"] < 1e5
    # nothing is recorded outside begin/end, and an empty session is fine
    b.radar_draft_rerank(pool, 5, 1)
    b.radar_profile_begin(4)
    assert b.radar_profile_end() == {}
    with pytest.raises(b.RadarError):
        b.radar_profile_begin(0)


def test_one_workspace_serves_several_entry_points_between_inits(oracle):
    """A workspace may go from one entry point (or descriptor) to another once it has been passed
    through radar_workspace_init again: the results equal those obtained with fresh workspaces."""
    from paper_2512_14069_amd import binding as b
    rng = np.random.default_rng(11)
    ws = b.new_workspace(64 << 20)

    # sampled verify-accept, two sequences
    a = synth.AttnShape(B=2, Hq=1, Hkv=1, D=8, T=20, ctx_lens=(0, 0), n_nodes=(20, 9), depths=(4, 3), k=4)
    x = synth.accept_inputs(a, 9000, seed=synth.seed_for(1, 41), plant=0.7)
    args = (dev(x["target_logits"]), dev(x["draft_tokens"]), dev(x["parents"]), dev(x["n_nodes"]), dev(x["uniforms"]))
    fresh = [host(t) for t in b.radar_verify_accept(*args, mode=1)]
    got = [host(t) for t in b.radar_verify_accept(*args, mode=1, workspace=ws)]
    assert all(np.array_equal(u, v) for u, v in zip(fresh, got))

    # expansion on the same memory
    b.radar_workspace_init(ws)
    F, V, k = 5, 12345, 6
    logits = dev(synth.normal_logits(rng, (F, V), 2.0))
    ps = torch.zeros(F, device="cuda")
    ppi = torch.full((F,), -1, dtype=torch.int32, device="cuda")
    p1, p2 = b.DraftPool(F * k), b.DraftPool(F * k)
    e1 = b.radar_draft_expand(logits, ps, ppi, k, p1)
    e2 = b.radar_draft_expand(logits, ps, ppi, k, p2, workspace=ws)
    torch.cuda.synchronize()
    for name in ("cand_tokens", "cand_scores", "frontier_pool_idx", "frontier_tokens", "frontier_scores", "frontier_conf"):
        assert torch.equal(getattr(e1, name), getattr(e2, name)), name

    # attention with several key ranges, then accept again with another shape
    b.radar_workspace_init(ws)
    s = synth.AttnShape(B=2, Hq=8, Hkv=2, D=128, T=24, ctx_lens=(300, 90), n_nodes=(24, 11), depths=(4, 3), k=4)
    y = synth.attention_inputs(s, seed=synth.seed_for(1, 43))
    q, kc, vc = bf16_dev(y["q"]), bf16_dev(y["k_cache"]), bf16_dev(y["v_cache"])
    targs = (q, kc, vc, dev(y["parents"]), dev(y["ctx_lens"]), dev(y["n_nodes"]))
    o1 = b.radar_tree_attention(*targs, keys_per_split=64)
    o2 = b.radar_tree_attention(*targs, keys_per_split=64, workspace=ws)
    assert torch.equal(o1, o2)

    b.radar_workspace_init(ws)
    a2 = synth.AttnShape(B=3, Hq=1, Hkv=1, D=8, T=33, ctx_lens=(0,) * 3, n_nodes=(33, 2, 17), depths=(6, 1, 4), k=4)
    x2 = synth.accept_inputs(a2, 20000, seed=synth.seed_for(1, 47), plant=0.7)
    args2 = (dev(x2["target_logits"]), dev(x2["draft_tokens"]), dev(x2["parents"]), dev(x2["n_nodes"]), dev(x2["uniforms"]))
    fresh2 = [host(t) for t in b.radar_verify_accept(*args2, mode=1)]
    got2 = [host(t) for t in b.radar_verify_accept(*args2, mode=1, workspace=ws)]
    assert all(np.array_equal(u, v) for u, v in zip(fresh2, got2))


def test_verify_step_replays_from_a_graph(oracle):
    """Tree attention (the library's plan on a short cache, and long ranges of a longer one) and sampled
    verify-accept captured once in a HIP graph and replayed with new inputs, with the program's own eager
    work and synchronisations between the replays; every replay is compared with the eager calls on the
    same inputs bit for bit, and the first with the oracle."""
    from paper_2512_14069_amd import binding as b
    from gpu_util import bf16_bits
    from test_gpu_attention import check_close
    V = 5000
    short = synth.AttnShape(B=2, Hq=8, Hkv=2, D=128, T=40, ctx_lens=(333, 70), n_nodes=(40, 17), depths=(5, 3), k=4)
    long_ = synth.AttnShape(B=2, Hq=8, Hkv=2, D=128, T=40, ctx_lens=(1100, 530), n_nodes=(40, 17), depths=(5, 3), k=4)

    def device_inputs(seed):
        xs, xl = synth.attention_inputs(short, seed=seed), synth.attention_inputs(long_, seed=seed + 1, shuffle=True)
        xa = synth.accept_inputs(short, V, seed=seed + 2, plant=0.7)
        return xs, xl, xa

    xs, xl, xa = device_inputs(100)
    bufs = dict(
        qs=bf16_dev(xs["q"]), ks=bf16_dev(xs["k_cache"]), vs=bf16_dev(xs["v_cache"]), ps=dev(xs["parents"]),
        cs=dev(xs["ctx_lens"]), ns=dev(xs["n_nodes"]),
        ql=bf16_dev(xl["q"]), kl=bf16_dev(xl["k_cache"]), vl=bf16_dev(xl["v_cache"]), pl=dev(xl["parents"]),
        cl=dev(xl["ctx_lens"]), nl=dev(xl["n_nodes"]),
        lg=dev(xa["target_logits"]), tk=dev(xa["draft_tokens"]), pa=dev(xa["parents"]), na=dev(xa["n_nodes"]),
        un=dev(xa["uniforms"]))

    def load(xs, xl, xa):
        for name, arr, bits in (("qs", xs["q"], True), ("ks", xs["k_cache"], True), ("vs", xs["v_cache"], True),
                                ("ql", xl["q"], True), ("kl", xl["k_cache"], True), ("vl", xl["v_cache"], True)):
            bufs[name].copy_(bf16_dev(arr))
        for name, arr in (("ps", xs["parents"]), ("pl", xl["parents"]), ("lg", xa["target_logits"]), ("tk", xa["draft_tokens"]),
                          ("pa", xa["parents"]), ("un", xa["uniforms"])):
            bufs[name].copy_(dev(arr))

    class Step:
        """One verify step with its own outputs and workspaces; run() enqueues it on the current stream."""
        def __init__(self):
            ds = b.attn_desc(bufs["qs"], bufs["ks"])
            dl = b.attn_desc(bufs["ql"], bufs["kl"], keys_per_split=512)
            self.ws = (b.new_workspace(b.radar_tree_attention_workspace_bytes(ds)),
                       b.new_workspace(b.radar_tree_attention_workspace_bytes(dl)),
                       b.new_workspace(b.radar_verify_accept_workspace_bytes(b.accept_desc(2, 40, V, 39, 1, 1.0))))
            self.out = (torch.empty_like(bufs["qs"]), torch.empty_like(bufs["ql"]),
                        (torch.empty(2, dtype=torch.int32, device="cuda"), torch.empty((2, 40), dtype=torch.int32, device="cuda"),
                         torch.empty(2, dtype=torch.int32, device="cuda")))

        def run(self):
            b.radar_tree_attention(bufs["qs"], bufs["ks"], bufs["vs"], bufs["ps"], bufs["cs"], bufs["ns"], out=self.out[0],
                                   workspace=self.ws[0])
            b.radar_tree_attention(bufs["ql"], bufs["kl"], bufs["vl"], bufs["pl"], bufs["cl"], bufs["nl"], out=self.out[1],
                                   keys_per_split=512, workspace=self.ws[1])
            b.radar_verify_accept(bufs["lg"], bufs["tk"], bufs["pa"], bufs["na"], bufs["un"], mode=1, out=self.out[2],
                                  workspace=self.ws[2])

    captured, eager = Step(), Step()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):                          # warm-up outside the capture (one-time launch set-up)
        captured.run()
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        captured.run()
    for i in range(4):
        xs, xl, xa = device_inputs(200 + 10 * i)
        load(xs, xl, xa)
        g.replay()
        torch.cuda.synchronize()
        got = captured.out
        eager.run()                                        # eager work between the replays
        torch.cuda.synchronize()
        ref = eager.out
        assert torch.equal(got[0], ref[0]) and torch.equal(got[1], ref[1]), i
        assert all(torch.equal(u, v) for u, v in zip(got[2], ref[2])), i
        if i == 0:
            for x, a, o in ((xs, short, got[0]), (xl, long_, got[1])):
                want = oracle.tree_attention(x["q"], x["k_cache"], x["v_cache"], x["parents"], x["ctx_lens"], x["n_nodes"])
                for bb in range(a.B):
                    n = a.n_nodes[bb]
                    check_close(bf16_bits(o)[bb, :n], want[bb, :n], f"graph replay b={bb}")


@pytest.mark.parametrize("B,T,V", [(1, 1, 17), (2, 9, 1000), (3, 64, 4099)])
def test_direct_calls_match_prepared_calls(B, T, V):
    """The native marshaller and the ctypes path make the same calls; arguments the first does not take reach the second's checks."""
    from paper_2512_14069_amd import binding as b
    rng = np.random.default_rng(B * 100 + T)
    logits, uni = dev(synth.normal_logits(rng, (B, T, V), 2.0)), dev(rng.random((B, T + 1), dtype=np.float32))
    par = dev(np.tile(synth.chain_tree(T), (B, 1)))
    tok = dev(rng.integers(0, V, size=(B, T)).astype(np.int32))
    ws = b.new_workspace(b.radar_verify_accept_workspace_bytes(b.accept_desc(B, T, V, T - 1, b.RADAR_ACCEPT_SAMPLE, 1.0)))
    qws = b.new_workspace(b.radar_verify_accept_q_workspace_bytes(b.accept_q_desc(B, T, T, V, T - 1)))
    for name, args, kw in (("radar_verify_accept", (logits, tok, par, None, uni), dict(mode=b.RADAR_ACCEPT_SAMPLE, workspace=ws)),
                           ("radar_accept_length_distribution", (logits, tok, par), dict(workspace=ws)),
                           ("radar_verify_accept_q", (logits, logits, tok, par, None, uni), dict(workspace=qws))):
        f = getattr(b, name)
        b.radar_workspace_init(kw["workspace"])
        direct, prepared = f(*args, **kw), f(*args, prepared=True, **kw)()
        for x, y in zip(direct if isinstance(direct, tuple) else (direct,), prepared if isinstance(prepared, tuple) else (prepared,)):
            assert x.dtype == y.dtype and x.shape == y.shape and torch.equal(x, y), name
        with pytest.raises(ValueError):
            f(args[0].double(), *args[1:], **kw)
        with pytest.raises(ValueError):
            f(args[0].transpose(0, 1).contiguous().transpose(0, 1)[:, :, ::2], *args[1:], **kw)


class _Both:
    """Runs a call natively (and sees that it did go there) and by ctypes; everything it returns or writes is equal."""

    def __init__(self, b, monkeypatch):
        self.b, self.taken = b, 0
        real, outer = b._native, self

        class Spy:
            def __getattr__(self, name):
                def call(*args):
                    got = getattr(real, name)(*args)
                    outer.taken += got is not None
                    return got
                return call
        monkeypatch.setattr(b, "_direct", lambda prepared: None if prepared or not self.native else Spy())

    def __call__(self, what, call):
        """call() -> tensors; made twice, on buffers of its own each time."""
        self.native, before = True, self.taken
        direct = call()
        assert self.taken == before + 1, f"{what}: the native half refused it"
        self.native = False
        other = call()
        torch.cuda.synchronize()
        assert len(direct) == len(other)
        for i, (x, y) in enumerate(zip(direct, other)):
            assert x.shape == y.shape and x.dtype == y.dtype and torch.equal(x, y), (what, i)


@pytest.mark.parametrize("D,S,kps", [(64, 150, 0), (128, 150, 64), (64, 1300, 1024), (128, 20000, 0)])
def test_native_attention_calls_match_ctypes(monkeypatch, D, S, kps):
    """Every form of an attention call that the native half reads by itself: log-sum-exp, scale, rows taken from a
    fused projection and caches with a row pitch, trees of the full size, outputs of the caller's."""
    from paper_2512_14069_amd import binding as b
    b.load()
    both = _Both(b, monkeypatch)
    g = torch.Generator(device="cuda").manual_seed(S)
    B, T, Hq, Hkv = 2, 33, 4, 2
    fused = torch.randn((B, T, 3 * Hq, D), generator=g, device="cuda").to(torch.bfloat16)
    kbuf, vbuf = (torch.randn((B, Hkv, S + T + 3, D + 8), generator=g, device="cuda").to(torch.bfloat16) for _ in range(2))
    par = dev(np.stack([synth.chain_tree(T), synth.star_tree(T)]).astype(np.int32))
    ctx, nn = dev(np.array([S, S // 3], np.int32)), dev(np.array([T, 9], np.int32))
    q, k, v = fused[:, :, Hq:2 * Hq], kbuf[:, :, :S + T, :D], vbuf[:, :, :S + T, :D]
    for dense in (False, True):
        if dense:
            q, k, v = q.contiguous(), k.contiguous(), v.contiguous()
        ws = b.new_workspace(b.radar_tree_attention_workspace_bytes(b.attn_desc(q, k, kps)))
        for nodes in (nn, None):
            for scale in (0.0, 0.04):
                for given in (False, True):
                    def call():
                        lse = torch.full((B, T, Hq), 5.0, device="cuda")
                        out = torch.full((B, T, Hq, D), 5.0, dtype=torch.bfloat16, device="cuda") if given else None
                        return b.radar_tree_attention(q, k, v, par, ctx, nodes, out=out, lse_out=lse, workspace=ws, keys_per_split=kps,
                                                      softmax_scale=scale), lse
                    both((dense, nodes is None, scale, given), call)


@pytest.mark.parametrize("V,k", [(1000, 4), (32000, 10)])
def test_native_drafting_calls_match_ctypes(monkeypatch, V, k):
    """Expansion alone, with the prediction model, with a cycle's state and for a batch, with and without a hidden state and
    a uniform; the reranks over what they left; the model's step by itself."""
    from paper_2512_14069_amd import binding as b
    b.load()
    both = _Both(b, monkeypatch)
    rng = np.random.default_rng(V + k)
    F, B, N, cap = 3, 2, 7, 4 * 3 * k
    pp = b.policy_params({n: dev(v) for n, v in synth.policy_params(rng, k).items()})
    H = synth.POLICY_H
    f32 = lambda *shape: dev(rng.standard_normal(shape).astype(np.float32))    # noqa: E731
    logits, ps, pi = f32(B, F, V), -f32(B, F).abs(), torch.full((B, F), -1, dtype=torch.int32, device="cuda")
    h, c, uni = f32(B, H), f32(B, H), dev(rng.random(B, dtype=np.float32))
    desc = b.expand_desc(F, V, k, 0, cap)
    ws = b.new_workspace(b.radar_draft_expand_batch_workspace_bytes(desc, B))
    fields = lambda o: [getattr(o, n).clone() for n in (getattr(o, "__slots__", None) or vars(o)) if isinstance(getattr(o, n), torch.Tensor)]   # noqa: E731
    states = ((None, None, None), (h, c, None), (h, c, uni), (None, None, uni))

    def draft(fn, batch, state=False, params=None, hcu=(None, None, None)):
        def call():
            b.radar_workspace_init(ws)
            pool = b.DraftPool(cap, B=B if batch else None)
            for t in (pool.tokens, pool.scores, pool.parents):
                t.zero_()
            out = b.ExpandOut(F, k, "cuda", B=B if batch else None)
            pout = b.PolicyOut(B if batch else 1, H, "cuda") if params else None
            st = (torch.zeros((B, 4), dtype=torch.int32, device="cuda") if batch else b.new_cycle_state()) if state else None
            lg, s, i = (logits, ps, pi) if batch else (logits[0], ps[0], pi[0])
            own = [None if t is None else t if batch else t[:1] for t in hcu]
            kw = dict(out=out, workspace=ws)
            if params:
                kw.update(params=params, h=own[0], c=own[1], uniform=own[2], policy_out=pout)
            if batch:
                fn(lg, s, i, k, pool, states=st, pool_count_max=0 if state else None, **kw)
            elif state:
                fn(lg, s, i, k, pool, 0, st, **kw)
            else:
                fn(lg, s, i, k, pool, **kw)
            return fields(out) + fields(pool) + (fields(pout) if params else []) + ([st] if state else [])
        return call

    both("expand", draft(b.radar_draft_expand, False))
    both("cycle", draft(b.radar_draft_expand_cycle, False, state=True))
    both("batch", draft(b.radar_draft_expand_batch, True))
    both("batch, states", draft(b.radar_draft_expand_batch, True, state=True))
    for hcu in states:
        given = tuple(t is not None for t in hcu)
        both(("policy", given), draft(b.radar_draft_expand_policy, False, params=pp, hcu=hcu))
        both(("cycle, policy", given), draft(b.radar_draft_expand_cycle, False, state=True, params=pp, hcu=hcu))
        both(("batch, policy", given), draft(b.radar_draft_expand_batch, True, params=pp, hcu=hcu))
        both(("batch, states, policy", given), draft(b.radar_draft_expand_batch, True, state=True, params=pp, hcu=hcu))
        both(("step", given), lambda: fields(b.radar_policy_step(ps[:, :1].exp().repeat(1, k).contiguous(), pp, hcu[0], hcu[1], hcu[2])))

    pool1, poolB = b.DraftPool(cap), b.DraftPool(cap, B=B)
    b.radar_draft_expand(logits[0], ps[0], pi[0], k, pool1)
    b.radar_draft_expand_batch(logits, ps, pi, k, poolB)
    st1, stB = (torch.tensor([0, F * k, 1, 0] * n, dtype=torch.int32, device="cuda") for n in (1, B))
    roots = dev(np.arange(B, dtype=np.int32))
    both("rerank", lambda: fields(b.radar_draft_rerank(pool1, N, 5)))
    both("rerank, state", lambda: fields(b.radar_draft_rerank_cycle(pool1, st1, cap, N, 5)))
    both("rerank, batch", lambda: fields(b.radar_draft_rerank_batch(poolB, N, roots)))
    both("rerank, batch, states", lambda: fields(b.radar_draft_rerank_batch(poolB, N, roots, states=stB.view(B, 4), pool_count_max=cap)))


@pytest.mark.parametrize("B,T,V", [(1, 1, 17), (3, 24, 5000)])
def test_native_verification_calls_match_ctypes(monkeypatch, B, T, V):
    """Greedy and sampled walks, the length distribution and the walk with draft distributions, with whole and ragged
    trees, outputs of the caller's and fresh ones, a row map and none, depths and temperatures."""
    from paper_2512_14069_amd import binding as b
    b.load()
    both = _Both(b, monkeypatch)
    rng = np.random.default_rng(B + T + V)
    x, y = (dev(synth.normal_logits(rng, (B, T, V), 2.0)) for _ in range(2))
    uni, par = dev(rng.random((B, T + 1), dtype=np.float32)), dev(np.tile(synth.chain_tree(T), (B, 1)).astype(np.int32))
    tok, nn = dev(rng.integers(0, V, size=(B, T)).astype(np.int32)), dev(rng.integers(1, T + 1, size=B).astype(np.int32))
    rows = dev(rng.integers(0, T, size=(B, T)).astype(np.int32))
    for D_max in {T - 1, T // 2}:
        ws = b.new_workspace(b.radar_verify_accept_workspace_bytes(b.accept_desc(B, T, V, D_max, b.RADAR_ACCEPT_SAMPLE, 1.0)))
        wsq = b.new_workspace(b.radar_verify_accept_q_workspace_bytes(b.accept_q_desc(B, T, T, V, D_max)))
        for given in (False, True):
            def fresh():
                return tuple(torch.full(s, 9, dtype=torch.int32, device="cuda") for s in ((B,), (B, D_max + 1), (B,))) if given else None
            for nodes in (nn, None):
                for temp in (1.0, 0.7):
                    kw = dict(D_max=D_max, temperature=temp, workspace=ws)
                    what = (D_max, given, nodes is None, temp)
                    both(("greedy",) + what, lambda: b.radar_verify_accept(x, tok, par, nodes, mode=b.RADAR_ACCEPT_GREEDY, out=fresh(), **kw))
                    both(("sample",) + what, lambda: b.radar_verify_accept(x, tok, par, nodes, uni, mode=b.RADAR_ACCEPT_SAMPLE, out=fresh(), **kw))
                    dist = torch.full((B, D_max + 1), 9.0, dtype=torch.float64, device="cuda") if given else None
                    both(("length",) + what, lambda: (b.radar_accept_length_distribution(x, tok, par, nodes, out=dist, **kw).clone(),))
                    for qr in (rows, None):
                        for limit in (0, -1):
                            both(("q", qr is None, limit) + what, lambda: b.radar_verify_accept_q(
                                x, y, tok, par, nodes, uni, qr, draft_temperature=1.2, out=fresh(), walk_spin_limit=limit, **dict(kw, workspace=wsq)))
