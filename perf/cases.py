"""The work a program has this library do, as measurable cases.

Four kinds, each through the binding's public calls:

  attention  one layer of tree-verify attention over a batch of sequences
  draft      the drafting of one cycle: one expansion per draft call, then the rerank
  verify     the acceptance walk over a batch of verified trees (greedy, sampled, with draft
             distributions) or the accepted length's distribution
  cycle      drafting with the stop decided on the device, rerank, one attention layer, acceptance

`prepared` says how the calls are made: a serving loop over fixed buffers marshals its calls once and
replays them; a program whose tensors change from step to step calls the functions themselves, with
its workspaces kept.  Lengths, tree sizes and the draft calls at which sequences stop come from
`shape_seed`, so a case's work is known without its inputs; values come from prepare()'s seed.
"""
import math
import random

import numpy as np
import torch

from paper_2512_14069_amd import binding as rb, synth

V_LLAMA = 128256
BRANCH = 10                                     # children per expanded node in verified trees
SHORT = 0.999999                                # a uniform that makes the prediction model stop; 0 continues


def listed():
    return [
        # the smallest layer the repository configures (head dimension 64, one KV head): bound by the call itself
        dict(name="attention_smoke", kind="attention", B=1, Hq=4, Hkv=1, D=64, T=16, nodes_lo=16, ctx_lo=256, ctx_hi=256,
             depth=4, lse=True, prepared=False, shape_seed=1),
        # one layer of an 8B-class target verifying a 60-node tree: the call made 32 times per cycle
        dict(name="attention_8b", kind="attention", B=1, Hq=32, Hkv=8, D=128, T=60, nodes_lo=60, ctx_lo=2048, ctx_hi=2048,
             depth=8, lse=False, prepared=True, shape_seed=2),
        # a served batch: 16 conversations of different lengths whose drafting stopped at different depths
        dict(name="attention_ragged16", kind="attention", B=16, Hq=32, Hkv=8, D=128, T=60, nodes_lo=2, ctx_lo=512, ctx_hi=8192,
             depth=8, lse=False, prepared=True, shape_seed=4),
        # long contexts on a 70B-class target, the largest layer configured
        dict(name="attention_70b", kind="attention", B=4, Hq=64, Hkv=8, D=128, T=60, nodes_lo=60, ctx_lo=16384, ctx_hi=16384,
             depth=8, lse=False, prepared=True, shape_seed=5),
        # the drafting of one sequence driven by the host: eight draft calls, then the rerank
        dict(name="draft_8b", kind="draft", B=1, calls=8, first=10, k=10, V=V_LLAMA, N=60, policy=False, prepared=False, shape_seed=3),
        # a served batch with the prediction model in every draft call; sequences stop at different calls
        dict(name="draft_policy16", kind="draft", B=16, calls=8, first=1, k=10, V=V_LLAMA, N=60, policy=True, prepared=True, shape_seed=6),
        # a large batch, bound by reading the logits
        dict(name="draft_batch64", kind="draft", B=64, calls=2, first=10, k=10, V=V_LLAMA, N=60, policy=False, prepared=True, shape_seed=7),
        # rejection sampling over one verified tree
        dict(name="accept_8b_sampled", kind="verify", mode="sample", B=1, T=61, nodes_lo=61, depth=8, V=V_LLAMA, temperature=1.0,
             prepared=False, shape_seed=3),
        # greedy acceptance for a served batch of ragged trees
        dict(name="accept_ragged16_greedy", kind="verify", mode="greedy", B=16, T=60, nodes_lo=2, depth=8, V=V_LLAMA,
             temperature=1.0, prepared=True, shape_seed=4),
        # trees whose tokens were drawn from the draft model's distributions
        dict(name="accept_q_8b", kind="verify", mode="q", B=1, T=61, nodes_lo=61, depth=8, V=V_LLAMA, temperature=1.0,
             prepared=False, shape_seed=8),
        # a whole cycle at the smallest configuration, called step by step
        dict(name="cycle_smoke", kind="cycle", B=1, calls=4, first=1, k=4, V=4096, N=15, Hq=4, Hkv=1, D=64, ctx_lo=256, ctx_hi=256,
             mode="greedy", prepared=False, shape_seed=1),
        # a whole cycle of one sequence at the 8B shape with nothing decided on the host
        dict(name="cycle_8b", kind="cycle", B=1, calls=8, first=1, k=10, V=V_LLAMA, N=60, Hq=32, Hkv=8, D=128, ctx_lo=2048,
             ctx_hi=2048, mode="sample", prepared=True, shape_seed=2),
    ]


# ------------------------------------------------------------------ drawn cases

def _log(rng, lo, hi):
    return max(lo, min(hi, round(math.exp(rng.uniform(math.log(lo), math.log(hi))))))


def _heads(rng):
    return rng.choice([(4, 1, 64), (8, 4, 64), (8, 2, 128), (16, 8, 128), (32, 8, 128), (32, 8, 128), (64, 8, 128), (8, 1, 128)])


def _tree(rng, most):
    depth = rng.randint(1, 8)
    T = _log(rng, depth + 1, min(most, 11 if depth == 1 else most))
    return T, depth


def _draw_attention(rng):
    while True:
        Hq, Hkv, D = _heads(rng)
        T, depth = _tree(rng, 64)
        hi = _log(rng, 16, 16384)
        B = _log(rng, 1, 16)
        lo = hi if rng.random() < 0.4 else max(1, hi // rng.randint(2, 16))
        c = dict(kind="attention", B=B, Hq=Hq, Hkv=Hkv, D=D, T=T, nodes_lo=depth + 1 if rng.random() < 0.5 else T, ctx_lo=lo, ctx_hi=hi,
                 depth=depth, lse=rng.random() < 0.3, prepared=rng.random() < 0.6, shape_seed=rng.randrange(1 << 20))
        if B * Hq * D * (hi + T) <= 4 * 64 * 128 * 16444 and B * Hkv * D * (hi + T) <= 16 * 8 * 128 * 8252:
            return c


def _draw_draft(rng):
    while True:
        B, k, calls = _log(rng, 1, 64), rng.randint(2, 16), rng.randint(1, 8)
        V = rng.choice([_log(rng, 4096, 131072), 32000, V_LLAMA])
        first = rng.choice([1, k])
        if calls * k * k <= rb.RADAR_POOL_MAX and calls * (12 + 4e-6 * B * k * V) < 450:
            return dict(kind="draft", B=B, calls=calls, first=first, k=k, V=V, N=rng.randint(8, 63), policy=rng.random() < 0.5,
                        prepared=rng.random() < 0.6, shape_seed=rng.randrange(1 << 20))


def _draw_verify(rng):
    while True:
        mode = rng.choice(["greedy", "sample", "sample", "q", "length"])
        T, depth = _tree(rng, 64)
        B = _log(rng, 1, 8 if mode == "q" else 16)
        V = rng.choice([_log(rng, 4096, 131072), 32000, V_LLAMA])
        if B * T * V <= 16 * 60 * V_LLAMA // (2 if mode == "q" else 1):
            return dict(kind="verify", mode=mode, B=B, T=T, nodes_lo=depth + 1 if rng.random() < 0.5 else T, depth=depth, V=V,
                        temperature=rng.choice([1.0, 1.0, 0.7]), prepared=rng.random() < 0.6, shape_seed=rng.randrange(1 << 20))


def _draw_cycle(rng):
    while True:
        Hq, Hkv, D = _heads(rng)
        B, k, calls, hi = _log(rng, 1, 4), rng.randint(4, 12), rng.randint(2, 8), _log(rng, 64, 4096)
        V = rng.choice([_log(rng, 4096, 131072), 32000, V_LLAMA])
        if calls * (16 + 4e-6 * B * k * V) < 250 and B * Hq * hi <= 64 * 4096:
            return dict(kind="cycle", B=B, calls=calls, first=1, k=k, V=V, N=rng.randint(8, 63), Hq=Hq, Hkv=Hkv, D=D,
                        ctx_lo=max(1, hi // 2), ctx_hi=hi, mode=rng.choice(["greedy", "sample"]), prepared=rng.random() < 0.6,
                        shape_seed=rng.randrange(1 << 20))


def draw(rng):
    return rng.choice([_draw_attention] * 3 + [_draw_draft] * 3 + [_draw_verify] * 3 + [_draw_cycle])(rng)


# ------------------------------------------------------------------ shapes of a case

def _lens(c, lo, hi, what):
    """One whole number per sequence, spread over [lo, hi]; the largest is hi."""
    r = random.Random(c["shape_seed"] * 8 + what)
    v = [r.randint(lo, hi) for _ in range(c["B"])]
    v[r.randrange(c["B"])] = hi
    return v


def _ctx(c):
    return _lens(c, c["ctx_lo"], c["ctx_hi"], 0)


def _nodes(c):
    return _lens(c, min(c["nodes_lo"], c["T"]), c["T"], 1)


def _stops(c):
    """The draft call after which each sequence stops (c["calls"]: it never does)."""
    if c["B"] == 1:
        return [c["calls"]]
    return _lens(c, 1, c["calls"], 2)


def _rows(c, s):
    return c["first"] if s == 0 else c["k"]


def _drafts(c):
    """Whether the case decides on the device when to stop."""
    return c["kind"] == "cycle" or c["policy"]


# ------------------------------------------------------------------ inputs

def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


def _i32(v):
    return torch.tensor(v, dtype=torch.int32, device="cuda")


def _trees(c, rng, V):
    """parents, tokens int32 [B,T] of the case's ragged batch of draft trees."""
    par, tok = np.full((c["B"], c["T"]), -1, np.int32), np.zeros((c["B"], c["T"]), np.int32)
    few = min(V, 4096)                          # siblings' tokens are distinct; drawn from few and spread over the vocabulary
    for b, n in enumerate(_nodes(c)):
        if n > 1:
            p, t, _ = synth.make_tree(rng, n, min(c["depth"], n - 1), BRANCH, few)
            par[b, :n], tok[b, :n] = p, t * (V // few)
    return par, tok


def _target_logits(gen, par, tok, V):
    """N(0,1) + Gumbel(0,1) rows in which the children's tokens carry a good part of the mass, as a draft model's
    best guesses do: the walk goes several nodes deep."""
    B, T = tok.shape
    x = torch.randn((B, T, V), generator=gen, device="cuda")
    for b in range(B):                          # one sequence at a time: no second copy of the batch
        x[b] -= torch.empty((T, V), device="cuda").exponential_(generator=gen).log_()
    b, n = np.nonzero(par >= 0)
    if len(b):
        lift = torch.randn(len(b), generator=gen, device="cuda") * 1.5 + (math.log(V) + 1.0)
        x.view(-1)[_dev((b.astype(np.int64) * T + par[b, n]) * V + tok[b, n])] = lift
    return x


def _prepare_attention(c, gen, rng, parents=None, n_nodes=None):
    B, T, Hq, Hkv, D = c["B"], c["T"], c["Hq"], c["Hkv"], c["D"]
    S = c["ctx_hi"] + T
    randn = lambda *shape: torch.randn(shape, generator=gen, device="cuda", dtype=torch.bfloat16)   # noqa: E731
    q, kc, vc = randn(B, T, Hq, D), randn(B, Hkv, S, D), randn(B, Hkv, S, D)
    desc = rb.attn_desc(q, kc)
    ws = rb.new_workspace(rb.radar_tree_attention_workspace_bytes(desc))
    if parents is None:
        parents, n_nodes = _dev(_trees(c, rng, 1 << 16)[0]), _i32(_nodes(c))
    ctx = _i32(_ctx(c))
    lse = torch.empty((B, T, Hq), dtype=torch.float32, device="cuda") if c.get("lse") else None
    out = torch.empty_like(q) if c["prepared"] else None

    def call(prepared=False):
        return rb.radar_tree_attention(q, kc, vc, parents, ctx, n_nodes, out=out, lse_out=lse, workspace=ws, prepared=prepared)
    return call, (lambda o: (o, lse))


def _verify_call(c, mode, logits, tokens, parents, n_nodes, uniforms, D_max, draft=None, q_rows=None):
    B, T, V = logits.shape
    temp = c.get("temperature", 1.0)
    m = rb.RADAR_ACCEPT_GREEDY if mode == "greedy" else rb.RADAR_ACCEPT_SAMPLE
    if mode == "q":
        ws = rb.new_workspace(rb.radar_verify_accept_q_workspace_bytes(rb.accept_q_desc(B, T, draft.shape[1], V, D_max, temp, temp)))
    else:
        ws = rb.new_workspace(rb.radar_verify_accept_workspace_bytes(rb.accept_desc(B, T, V, D_max, m, temp)))
    out = None
    if c["prepared"]:
        out = torch.empty((B, D_max + 1), dtype=torch.float64, device="cuda") if mode == "length" else (
            torch.empty(B, dtype=torch.int32, device="cuda"), torch.empty((B, D_max + 1), dtype=torch.int32, device="cuda"),
            torch.empty(B, dtype=torch.int32, device="cuda"))

    def call(prepared=False):
        if mode == "q":
            return rb.radar_verify_accept_q(logits, draft, tokens, parents, n_nodes, uniforms, q_rows, temperature=temp,
                                            draft_temperature=temp, D_max=D_max, out=out, workspace=ws, prepared=prepared)
        if mode == "length":
            return rb.radar_accept_length_distribution(logits, tokens, parents, n_nodes, temperature=temp, D_max=D_max, out=out,
                                                       workspace=ws, prepared=prepared)
        return rb.radar_verify_accept(logits, tokens, parents, n_nodes, uniforms if mode == "sample" else None, mode=m,
                                      temperature=temp, D_max=D_max, out=out, workspace=ws, prepared=prepared)
    return call


def _prepare_verify(c, gen, rng):
    B, T, V = c["B"], c["T"], c["V"]
    par, tok = _trees(c, rng, V)
    nn, uni = _i32(_nodes(c)), torch.rand((B, T + 1), generator=gen, device="cuda")
    draft = q_rows = None
    if c["mode"] == "q":                        # siblings are drawn from their parent's row of a draft that tracks the target loosely
        logits = torch.randn((B, T, V), generator=gen, device="cuda") * 2.0
        draft = logits + torch.randn((B, T, V), generator=gen, device="cuda")
        rows = np.maximum(par, 0)
        q_rows = _dev(rows)
        tok = tok.copy()
        for b in range(B):
            noise = torch.empty((T, V), device="cuda").exponential_(generator=gen).log_()
            drawn = (draft[b][_dev(rows[b].astype(np.int64))] / c["temperature"] - noise).argmax(dim=-1).to(torch.int32)
            tok[b, 1:] = drawn.cpu().numpy()[1:]
    else:
        logits = _target_logits(gen, par, tok, V)
    return _verify_call(c, c["mode"], logits, _dev(tok), _dev(par), nn, uni, c["depth"], draft, q_rows)


class _Draft:
    """The drafting of one cycle: its calls in order, over buffers that the program keeps."""

    def __init__(self, c, gen, rng):
        self.c = c
        B, k, V, calls = c["B"], c["k"], c["V"], c["calls"]
        self.batch, self.device_stop = B > 1, _drafts(c)
        lead = (B,) if self.batch else ()
        self.logits = [torch.log_softmax(torch.randn(lead + (_rows(c, s), V), generator=gen, device="cuda") * 3.0, dim=-1).contiguous()
                       for s in range(calls)]
        self.cap = sum(_rows(c, s) * k for s in range(calls))
        self.pool = rb.DraftPool(self.cap, B=B if self.batch else None)
        self.outs = [rb.ExpandOut(_rows(c, s), k, "cuda", B=B if self.batch else None) for s in range(calls)]
        self.tree = rb.TreeOut(c["N"], "cuda", B=B if self.batch else None)
        F = max(_rows(c, s) for s in range(calls))
        desc = rb.expand_desc(F, V, k, 0, self.cap)
        self.ws = rb.new_workspace(rb.radar_draft_expand_batch_workspace_bytes(desc, B) if self.batch else rb.radar_draft_expand_workspace_bytes(desc))
        self.ps = torch.zeros(lead + (c["first"],), dtype=torch.float32, device="cuda")
        self.pi = torch.full(lead + (c["first"],), -1, dtype=torch.int32, device="cuda")
        self.roots = torch.randint(0, V, (B,), generator=gen, device="cuda").to(torch.int32)
        self.params = self.state = self.pol = None
        for t in [x for o in self.outs for x in vars(o).values()]:
            t.zero_()                           # a skipped draft call leaves its outputs alone
        if self.device_stop:
            self.state = torch.zeros((B, 4), dtype=torch.int32, device="cuda") if self.batch else rb.new_cycle_state()
            self.params = rb.policy_params({n: _dev(v) for n, v in synth.policy_params(rng, k).items()})
            self.pol = rb.PolicyOut(B, synth.POLICY_H, "cuda")
            for n in rb.PolicyOut.__slots__:
                getattr(self.pol, n).zero_()
            uni = np.zeros((calls, B), np.float32)
            for b, s in enumerate(_stops(c)):
                if s < calls:
                    uni[s - 1, b] = SHORT
            self.uni = _dev(uni)

    def steps(self):
        """One function per call; each takes `prepared`."""
        c, k, got, ps, pi, most = self.c, self.c["k"], [], self.ps, self.pi, 0
        for s in range(c["calls"]):
            decide = self.device_stop and s + 1 < c["calls"]
            kw = dict(out=self.outs[s], workspace=self.ws)
            if self.device_stop:
                kw.update(params=self.params if decide else None, h=self.pol.h if decide and s else None,
                          c=self.pol.c if decide and s else None, uniform=self.uni[s] if decide else None,
                          policy_out=self.pol if decide else None)
            got.append(self._expand(self.logits[s], ps, pi, most, kw))
            most += _rows(c, s) * k
            ps, pi = self.outs[s].frontier_scores, self.outs[s].frontier_pool_idx
        got.append(self._rerank())
        return got

    def _expand(self, lg, ps, pi, most, kw):
        k, pool = self.c["k"], self.pool
        if self.batch:
            def call(prepared=False):
                pool.count = most
                return rb.radar_draft_expand_batch(lg, ps, pi, k, pool, states=self.state, pool_count_max=most if self.device_stop else None,
                                                   prepared=prepared, **kw)
        elif self.device_stop:
            def call(prepared=False):
                return rb.radar_draft_expand_cycle(lg, ps, pi, k, pool, most, self.state, prepared=prepared, **kw)
        else:
            def call(prepared=False):
                pool.count = most
                return rb.radar_draft_expand(lg, ps, pi, k, pool, prepared=prepared, **kw)
        return call

    def _rerank(self):
        c = self.c
        if self.batch:
            return lambda prepared=False: rb.radar_draft_rerank_batch(self.pool, c["N"], self.roots, states=self.state, pool_count_max=self.cap,
                                                                      out=self.tree, prepared=prepared)
        if self.device_stop:
            return lambda prepared=False: rb.radar_draft_rerank_cycle(self.pool, self.state, self.cap, c["N"], 1, out=self.tree, prepared=prepared)
        return lambda prepared=False: rb.radar_draft_rerank(self.pool, c["N"], 1, out=self.tree, prepared=prepared)

    def results(self, whole=True):
        """Everything the drafting wrote (a cycle leaves out the candidate arrays: the pool holds the same values)."""
        names = ("cand_tokens", "cand_scores") if whole else ()
        got = [[getattr(o, n) for n in names + ("frontier_pool_idx", "frontier_tokens", "frontier_scores", "frontier_conf")] for o in self.outs]
        t, p = self.tree, self.pool
        got += [p.tokens, p.scores, p.parents, t.tokens, t.parents, t.scores, t.depth, t.pool_idx, t.n_nodes]
        if self.device_stop:
            got += [self.state] + [getattr(self.pol, n) for n in rb.PolicyOut.__slots__]
        return got


class _Cycle:
    """Drafting, then one attention layer and the acceptance walk over the tree it produced."""

    def __init__(self, c, gen, rng):
        B, T, V = c["B"], c["N"] + 1, c["V"]
        self.draft = _Draft(c, gen, rng)
        tree = self.draft.tree
        tokens, parents = tree.tokens.view(B, T), tree.parents.view(B, T)
        self.attend, _ = _prepare_attention(dict(c, T=T), gen, rng, parents, tree.n_nodes)
        for f in self.draft.steps():                # the target's logits belong to the tree that this drafting yields
            f()
        logits = _target_logits(gen, parents.cpu().numpy(), tokens.cpu().numpy(), V)
        uni = torch.rand((B, T + 1), generator=gen, device="cuda")
        self.accept = _verify_call(c, c["mode"], logits, tokens, parents, tree.n_nodes, uni, c["calls"])

    def steps(self):
        return self.draft.steps() + [self.attend, self.accept]

    def results(self, attended, accepted):
        return [self.draft.results(whole=False), attended, accepted]


def prepare(case, seed):
    c = dict(case)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed) * 7919 + 13)
    rng = np.random.default_rng([int(seed), 17])
    collect = None
    if c["kind"] == "attention":
        call, collect = _prepare_attention(c, gen, rng)
        steps = [call]
    elif c["kind"] == "verify":
        steps = [_prepare_verify(c, gen, rng)]
    else:
        work = (_Draft if c["kind"] == "draft" else _Cycle)(c, gen, rng)
        steps = work.steps()
        collect = (lambda *o: work.results()) if c["kind"] == "draft" else (lambda *o: work.results(*o[-2:]))
    if c["prepared"]:
        steps = [f(prepared=True) for f in steps]
    return steps, collect


def run(state):
    steps, collect = state
    got = [f() for f in steps]
    return collect(*got) if collect else got[0]


# ------------------------------------------------------------------ what a pass cannot do without

def _attention_work(c, nodes):
    keys = [l + n for l, n in zip(_ctx(c), nodes)]
    kv = sum(keys) * c["Hkv"] * c["D"] * 2 * 2
    qo = (sum(nodes) + c["B"] * c["T"]) * c["Hq"] * c["D"] * 2
    return kv + qo, 4.0 * sum(k * n for k, n in zip(keys, nodes)) * c["Hq"] * c["D"]


def _draft_work(c):
    byt = flops = 0
    for stop in _stops(c) if _drafts(c) else [c["calls"]] * c["B"]:
        rows = sum(_rows(c, s) for s in range(stop))
        byt += rows * (c["V"] * 4 + c["k"] * 20) + stop * c["k"] * 16 + (c["N"] + 1) * 20
        flops += rows * c["V"] * 3.0
    return byt, flops


def _verify_work(c, nodes):
    rows = sum(nodes)
    if c["mode"] == "q":                        # every target row and the draft rows of nodes that have children: about half
        rows = sum(1.5 * n for n in nodes)
    return rows * c["V"] * 4, rows * c["V"] * (1.0 if c["mode"] == "greedy" else 3.0)


def work(case):
    c = dict(case)
    if c["kind"] == "attention":
        parts = [_attention_work(c, _nodes(c))]
    elif c["kind"] == "draft":
        parts = [_draft_work(c)]
    elif c["kind"] == "verify":
        parts = [_verify_work(c, _nodes(c))]
    else:
        pool = [sum(_rows(c, s) for s in range(stop)) * c["k"] for stop in _stops(c)]
        nodes = [1 + min(c["N"], p) for p in pool]
        parts = [_draft_work(c), _attention_work(dict(c, T=c["N"] + 1), nodes), _verify_work(c, nodes)]
    return {"bytes": sum(p[0] for p in parts), "flops": sum(p[1] for p in parts)}


def tolerance(case):
    kind = case["kind"]
    if kind in ("attention", "cycle"):
        return {"rel": 1e-2}                    # bf16 probabilities and outputs, fp32 sums
    if kind == "draft":
        return {"rel": 3e-5 if case["policy"] else 1e-5, "max": 4e-4}      # fp32 log-probabilities; confidences are their exponentials
    return {"rel": 1e-6, "max": 1e-5} if case["mode"] == "length" else "exact"
