"""The binding's native half without a GPU: arguments it cannot take, and the C++ exceptions that torch throws
while it reads them, come back as None (the caller then goes on with the path that raises the exact error).
Run in a child process: an exception that escaped would end it."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CHILD = r"""
import ctypes
import sys
import warnings

import torch
from torch._subclasses.fake_tensor import FakeTensorMode

from paper_2512_14069_amd import binding as b

warnings.simplefilter("ignore")
b.load()
n = b._native
assert not torch.cuda.is_available()
with FakeTensorMode():                      # tensors that say they are on a GPU; there is none to allocate on or take a stream from
    f = lambda *shape: torch.empty(shape, device="cuda")
    i = lambda *shape: torch.empty(shape, dtype=torch.int32, device="cuda")
    h = lambda *shape: torch.empty(shape, dtype=torch.bfloat16, device="cuda")
    d = lambda *shape: torch.empty(shape, dtype=torch.float64, device="cuda")
    q, kv, x, t, un = h(1, 2, 4, 64), h(1, 1, 8, 64), f(1, 2, 64), i(1, 2), f(1, 3)
    outs = (i(1), i(1, 2), i(1))
    expand = (f(3, 64), f(3), i(3), 2, 0, 64, i(6), f(6), i(2), i(2), f(2), f(2), i(64), f(64), i(64))
    pp = b.PolicyParams()
    pp.k, pp.H, pp.M = 2, 128, 128
    policy = (f(1, 128), f(1, 128), None, f(1, 128), f(1, 128), f(1, 2), f(1, 2), i(1))
    at = ctypes.addressof(pp)
    calls = {
        "tree_attention": (n.tree_attention, (q, kv, kv, t, i(1), None, h(1, 2, 4, 64), None, 0, 0.0)),
        "tree_attention, allocates": (n.tree_attention, (q, kv, kv, t, i(1), None, None, None, 0, 0.0)),
        "draft_expand": (n.draft_expand, (0,) + expand + (None, 0)),
        "draft_expand, policy": (n.draft_expand, (0,) + expand + (None, at) + policy),
        "draft_expand, cycle": (n.draft_expand, (0,) + expand + (i(4), 0)),
        "draft_rerank": (n.draft_rerank, (0, i(64), f(64), i(64), None, 9, 64, 5, 1, i(6), i(6), f(6), i(6), i(6), i(1))),
        "verify_accept": (n.verify_accept, (x, t, t, None, un, 1, 1.0, 1) + outs),
        "verify_accept, allocates": (n.verify_accept, (x, t, t, None, un, 1, 1.0, 1, None, None, None)),
        "verify_accept, deepest": (n.verify_accept, (x, t, t, None, un, 1, 1.0, 2**31 - 1, None, None, None)),
        "verify_accept_q": (n.verify_accept_q, (x, x, None, t, t, None, un, 1.0, 1.0, 1, 0) + outs),
        "verify_accept_q, allocates": (n.verify_accept_q, (x, x, None, t, t, None, un, 1.0, 1.0, 1, 0, None, None, None)),
        "accept_length_distribution": (n.accept_length_distribution, (x, t, t, None, 1.0, 1, d(1, 2))),
        "accept_length_distribution, allocates": (n.accept_length_distribution, (x, t, t, None, 1.0, 1, None)),
        "policy_step": (n.policy_step, (f(1, 2), at) + policy),
    }
sparse = torch.sparse_coo_tensor(torch.zeros((1, 1), dtype=torch.long), torch.ones(1), (4,))
bare = ("draft_rerank", "policy_step")      # no workspace among their arguments
what = sys.argv[1]
for name, (fn, args) in calls.items():
    print(name, flush=True)
    if what == "exceptions":                # the stream, or an output's memory
        assert fn(*args, *(() if name in bare else (None,))) is None
    elif what == "workspace":               # a workspace without storage, alone and behind an argument that failed already
        if name not in bare:
            assert fn(*args, sparse) is None
            assert fn(*[a.cpu() if isinstance(a, torch.Tensor) and not j else a for j, a in enumerate(args)], sparse) is None
            assert fn(*args, "workspace") is None
    else:                                   # every argument left out, one after the other, and every tensor of another kind
        for k in range(len(args)):
            assert fn(*args[:k]) is None
            for other in (torch.zeros(1), "text", None if k < 2 else torch.zeros(2, dtype=torch.int8), 1 << 40):
                if isinstance(args[k], torch.Tensor) or not isinstance(other, int):
                    assert fn(*args[:k], other, *args[k + 1:], *(() if name in bare else (None,))) is None
print("done")
"""


@pytest.mark.parametrize("what", ["exceptions", "workspace", "arguments"])
def test_nothing_leaves_the_native_half_but_none(what):
    env = dict(os.environ, HIP_VISIBLE_DEVICES="-1", PYTHONPATH=ROOT)
    r = subprocess.run([sys.executable, "-W", "ignore", "-c", CHILD, what], cwd=ROOT, env=env, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.rstrip().endswith("done"), (r.returncode, r.stdout[-500:], r.stderr[-2000:])


def test_the_binding_raises_what_python_can_catch():
    """verify_accept with a workspace that has no storage: the caller gets a Python exception, not the process's end."""
    code = ("import torch\nfrom paper_2512_14069_amd import binding as b\n"
            "ws = torch.sparse_coo_tensor(torch.zeros((1, 1), dtype=torch.long), torch.ones(1), (4,))\n"
            "t = torch.zeros((1, 2), dtype=torch.int32)\n"
            "try:\n    b.radar_verify_accept(torch.zeros((1, 2, 64)), t, t, workspace=ws)\n"
            "except (RuntimeError, ValueError, NotImplementedError) as e:\n    print('caught', type(e).__name__)\n")
    env = dict(os.environ, HIP_VISIBLE_DEVICES="-1", PYTHONPATH=ROOT)
    r = subprocess.run([sys.executable, "-c", code], cwd=ROOT, env=env, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and "caught" in r.stdout, (r.returncode, r.stderr[-2000:])
