"""GPU parity: radar_accept_length_distribution (through the C ABI) against the CPU oracle
(Sec. 4.3, Eq. 11-13).  Probabilities agree within DIST_TOL: the device takes fp32 exponentials
for the row sums (relative error of a row's log-sum-exp about 1e-8) and fp64 everywhere else."""
import numpy as np
import pytest
import torch

from paper_2512_14069_amd import synth
from gpu_util import dev, host

pytestmark = pytest.mark.gpu

DIST_TOL = 1e-6


def check(oracle, b, x, temperature=1.0, D_max=None):
    ref = oracle.accept_length_distribution(x["target_logits"], x["draft_tokens"], x["parents"], x["n_nodes"],
                                            temperature=temperature, D_max=D_max)
    got = b.radar_accept_length_distribution(dev(x["target_logits"]), dev(x["draft_tokens"]), dev(x["parents"]),
                                             dev(x["n_nodes"]), temperature=temperature, D_max=D_max)
    torch.cuda.synchronize()
    got = host(got)
    assert got.shape == ref.shape
    assert np.max(np.abs(got - ref)) <= DIST_TOL, np.max(np.abs(got - ref))
    assert np.max(np.abs(got.sum(axis=1) - 1.0)) <= DIST_TOL
    return ref, got


def small_shape(B, T, nn, dep, k=4):
    return synth.AttnShape(B=B, Hq=1, Hkv=1, D=8, T=T, ctx_lens=(0,) * B, n_nodes=nn, depths=dep, k=k)


def make_inputs(a, V, seed, std=1.5):
    """Seeded trees and target logits N(0, std) with every node's token lifted under its parent's
    row, so that deeper accepted lengths carry visible mass (nothing is planted as a sure path)."""
    rng = np.random.default_rng(seed)
    B, T = a.B, a.T
    x = dict(target_logits=synth.normal_logits(rng, (B, T, V), std),
             draft_tokens=np.zeros((B, T), np.int32), parents=np.full((B, T), -1, np.int32),
             n_nodes=np.array(a.n_nodes, np.int32))
    for b in range(B):
        n = a.n_nodes[b]
        par, tok, _ = synth.make_tree(rng, n, a.depths[b], a.k, V)
        x["parents"][b, :n], x["draft_tokens"][b, :n] = par, tok
    return lift(x)


def lift(x):
    for b in range(x["parents"].shape[0]):
        for c in range(1, int(x["n_nodes"][b])):
            x["target_logits"][b, x["parents"][b, c], x["draft_tokens"][b, c]] += np.float32(np.log(x["target_logits"].shape[2]))
    return x


@pytest.mark.parametrize("V,temperature", [(4096, 1.0), (5000, 0.7), (65537, 1.0), (128256, 1.0), (131073, 0.7)])
def test_ragged_batch_matches_oracle(oracle, V, temperature):
    from paper_2512_14069_amd import binding as b
    a = small_shape(5, 40, (40, 1, 17, 33, 2), (6, 0, 3, 8, 1), k=5)
    x = make_inputs(a, V, 91)
    ref, got = check(oracle, b, x, temperature)
    assert (ref[:, 2:] > 1e-4).any()                 # several lengths really occur


@pytest.mark.parametrize("V", [65537, 131073, 196609])
def test_last_block_of_a_group_counts(oracle, V):
    """65, 129 and 193 blocks of 1024 logits per row, of which the last holds one logit that weighs as much as a lifted token."""
    from paper_2512_14069_amd import binding as b
    x = make_inputs(small_shape(3, 12, (12, 1, 7), (3, 0, 2), k=4), V, 95)
    x["target_logits"][:, :, -1] += np.float32(np.log(V))
    ref, _ = check(oracle, b, x)
    masked = x["target_logits"].copy()
    masked[:, :, (V - 1) // 1024 * 1024:] = -100.0
    without = oracle.accept_length_distribution(masked, x["draft_tokens"], x["parents"], x["n_nodes"])
    assert (np.abs(ref - without).max(axis=1)[[0, 2]] > 1000 * DIST_TOL).all()


def test_config3_shape_star_and_chain(oracle):
    from paper_2512_14069_amd import binding as b
    a = small_shape(3, 61, (61, 61, 61), (8, 1, 60), k=10)
    rng = np.random.default_rng(92)
    par0, tok0, _ = synth.make_tree(rng, 61, 8, 10, 128256)
    x = dict(target_logits=synth.normal_logits(rng, (3, 61, 128256), 1.5),
             draft_tokens=np.stack([tok0, rng.permutation(128256)[:61].astype(np.int32),
                                    rng.permutation(128256)[:61].astype(np.int32)]),
             parents=np.stack([par0, synth.star_tree(61), synth.chain_tree(61)]).astype(np.int32),
             n_nodes=np.array([61, 61, 61], np.int32))
    x["draft_tokens"][1, 7] = x["draft_tokens"][1, 3]            # a repeated sibling token under the root
    lift(x)
    check(oracle, b, x)
    check(oracle, b, x, D_max=3)                                   # walk cut: deeper mass folds onto length 3
    check(oracle, b, x, D_max=0)


def test_same_kernel_still_walks_afterwards(oracle):
    """The distribution and the walk share workspace and kernel; alternate them on one workspace."""
    from paper_2512_14069_amd import binding as b
    a = small_shape(2, 12, (12, 9), (3, 3), k=3)
    x = make_inputs(a, 3000, 93)
    x["uniforms"] = np.random.default_rng(94).random((2, 13), dtype=np.float32)
    desc = b.accept_desc(2, 12, 3000, 11, b.RADAR_ACCEPT_SAMPLE, 1.0)
    ws = b.new_workspace(b.radar_verify_accept_workspace_bytes(desc))
    tl, tk, pa, nn, un = (dev(x[k]) for k in ("target_logits", "draft_tokens", "parents", "n_nodes", "uniforms"))
    ref_d = oracle.accept_length_distribution(x["target_logits"], x["draft_tokens"], x["parents"], x["n_nodes"])
    ref_w = oracle.verify_accept(x["target_logits"], x["draft_tokens"], x["parents"], x["n_nodes"], None, mode=0)
    for _ in range(3):
        d = b.radar_accept_length_distribution(tl, tk, pa, nn, workspace=ws)
        w = b.radar_verify_accept(tl, tk, pa, nn, None, mode=0, workspace=ws)
        torch.cuda.synchronize()
        assert np.max(np.abs(host(d) - ref_d)) <= DIST_TOL
        assert np.array_equal(host(w[0]), ref_w[0]) and np.array_equal(host(w[2]), ref_w[2])
    with pytest.raises(b.RadarError):
        b.radar_accept_length_distribution(tl, tk, pa, nn, temperature=0.0)
