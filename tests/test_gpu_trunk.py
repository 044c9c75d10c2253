"""The one-launch convolution stack of the forward-only calls (Section 5.1).

Its workgroups walk samples n, n + 256, ...: sizes around one and two rounds of
256, and the smallest.  Sums are of exact products in fp32; the bound on Q is
four layers of at most 8 roundings of 2^-24 each relative to the sums' terms:
4 * 8 * 6e-8 = 2e-6 of the largest |Q| (measured 3e-7 to 6e-7)."""
from __future__ import annotations

import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle
import paper_1507_04296_amd as g
from paper_1507_04296_amd import datagen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("n", [1, 2, 255, 256, 257, 513])
def test_q_of_every_round(n, bf16):
    A = 7
    inp = datagen.actor_inputs(91 + n, n, A)
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(n)
    theta = inp.theta + np.float32(0.02) * rng.standard_normal(inp.theta.shape).astype(np.float32)
    t = torch.from_numpy(theta).to(dev)
    if bf16:
        t = t.bfloat16()
        theta = t.float().cpu().numpy()
    states = inp.states.copy()
    states[0, :2] = 0          # blank channels, as at an episode start
    states[-1] = 255           # the largest input
    ctx = g.Context((n + 1) // 2, A, dtype=g.dtype_of(t))
    q = g.q_forward(ctx, t, A, torch.from_numpy(states).to(dev))
    ctx.check()
    rows = sorted({r for r in (0, 1, 254, 255, 256, 300, 511, 512, n - 1) if r < n})
    ref = oracle.q_forward(oracle.Net(n_actions=A), theta, states[rows])
    got = q.cpu().numpy()
    assert np.isfinite(got).all()
    assert np.abs(got[rows] - ref).max() <= 2e-6 * np.abs(ref).max()
    if n <= g.NOALLOC_MAX_STATES:
        acts = torch.empty(n, dtype=torch.int32, device=dev)
        q2 = torch.empty_like(q)
        g.gorila_act_noalloc(g.Context(0, A), t, A, torch.from_numpy(states).to(dev), 0.0, 3, acts, q2)
        assert torch.equal(q, q2) and np.array_equal(acts.cpu().numpy(), got.argmax(1))
    ctx.close()
