"""The one-launch convolution stack (Section 5.1): forward-only calls, and the
target's rows of a learner step whose rounds of 256 are nearly full.

Its workgroups walk samples n, n + 256, ...: sizes around one and two rounds of
256, and the smallest.  Sums are of exact products in fp32; the bound on Q is
four layers of at most 8 roundings of 2^-24 each relative to the sums' terms:
4 * 8 * 6e-8 = 2e-6 of the largest |Q| (measured 3e-7 to 6e-7)."""
from __future__ import annotations

import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle
import parity
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
    q, stages = parity.stages_of(ctx, lambda: g.q_forward(ctx, t, A, torch.from_numpy(states).to(dev)))
    assert "conv_fwd" in stages and "conv1_fwd" not in stages
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


# the rows where the choice changes with 256 units, and bf16's first round
@pytest.mark.parametrize("G,b,bf16,one", [
    (1, 230, False, False), (1, 231, False, True), (7, 33, False, True), (1, 460, False, False),
    (1, 461, False, True), (1, 614, False, False), (1, 615, False, True), (2, 128, True, False),
    (4, 115, True, False), (4, 116, True, True)])
def test_target_rows(G, b, bf16, one):
    """Against the fp64 oracle, at the bars of every learner test."""
    print(f"[gpu-case] target rows G={G} b={b} bf16={bf16}", flush=True)
    A = 18
    inp = datagen.grouped_inputs(7700 + G * b, G, b, A)
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    inp.s2[0, :3] = 0          # blank channels, as at an episode start
    rep = g.Replay.stacked(t(inp.s), t(inp.s2), t(inp.a), t(inp.r), t(inp.term))
    idx = np.arange(G * b, dtype=np.int64)
    th64 = [datagen.bf16_bits_to_f64(x) for x in inp.theta_bf16]
    tg64 = datagen.bf16_bits_to_f64(inp.target_bf16)
    ctx = g.Context(b, A, groups=G, dtype=g.GORILA_BF16 if bf16 else g.GORILA_F32)
    if bf16:
        th, tg = t(inp.theta_bf16.view(np.int16)), t(inp.target_bf16.view(np.int16))
    else:
        th, tg = [t(x.astype(np.float32)) for x in th64], t(tg64.astype(np.float32))
    (grads, loss), stages = parity.stages_of(
        ctx, lambda: g.learner_step_grouped(ctx, th, tg, A, rep, t(idx), inp.gamma, 1.0))
    if torch.cuda.get_device_properties(0).multi_processor_count == 256:
        assert ("conv_fwd" in stages) == one
    ctx.check()
    ctx.close()
    got, got_l = grads.cpu().numpy().reshape(G, -1), loss.cpu().numpy()
    net = oracle.Net(n_actions=A)
    for i, x in enumerate(th64):
        rows = idx[i * b:(i + 1) * b]
        ref = oracle.learner_step(net, x, tg64, inp.s[rows], inp.s2[rows], inp.a[rows], inp.r[rows],
                                  inp.term[rows], inp.gamma, 1.0)
        parity.assert_grads_close(got[i], ref["grads"], A,
                                  parity.GRAD_TOL_BF16 if bf16 else parity.GRAD_TOL)
        assert abs(got_l[i] - ref["loss"]) <= parity.LOSS_TOL * abs(ref["loss"])


# One infinite weight of conv2, conv3 and the FC layer (fp32 tiles, plane tiles):
# Q is infinite where the reference's is, NaN or finite where that is.  The
# reference adds in fp64 and takes a ReLU's NaN as zero, as the kernels do.
@pytest.mark.parametrize("n", [3, 257])
@pytest.mark.parametrize("layer", ["conv2", "conv3", "fc1"])
def test_infinite_weight(layer, n):
    A = 5
    inp = datagen.actor_inputs(17 + n, n, A)
    theta = inp.theta.copy()
    at = {"conv2": 8224 + 3 * 512 + 37, "conv3": 41056 + 5 * 576 + 100, "fc1": 77984 + 9 * 3136 + 1300}[layer]
    theta[at] = np.inf
    states = inp.states[:n]
    F = torch.nn.functional
    p = torch.from_numpy(theta.astype(np.float64))
    cut = lambda o, *s: p[o:o + int(np.prod(s))].view(*s)
    relu = lambda x: torch.nan_to_num(x, nan=0.0, posinf=np.inf, neginf=-np.inf).clamp_min(0.0)
    x = torch.from_numpy(states).double() / 255.0
    conv = lambda x, o, c, ci, k, s: relu(
        (F.unfold(x, k, stride=s).transpose(1, 2) @ cut(o, c, ci * k * k).T).transpose(1, 2)
        + cut(o + c * ci * k * k, c)[None, :, None])
    h1 = conv(x, 0, 32, 4, 8, 4).view(n, 32, 20, 20)
    h2 = conv(h1, 8224, 64, 32, 4, 2).view(n, 64, 9, 9)
    h3 = conv(h2, 41056, 64, 64, 3, 1).reshape(n, 3136)
    h4 = relu(h3 @ cut(77984, 512, 3136).T + cut(1683616, 512))
    ref = (h4 @ cut(1684128, A, 512).T + cut(1684128 + A * 512, A)).numpy()
    ctx = g.Context((n + 1) // 2, A)
    got = g.q_forward(ctx, torch.from_numpy(theta).cuda(), A, torch.from_numpy(states).cuda()).cpu().numpy()
    ctx.check()
    ctx.close()
    assert np.array_equal(np.isfinite(got), np.isfinite(ref))
    assert np.array_equal(np.isnan(got), np.isnan(ref))
    fin = np.isfinite(ref)
    assert np.array_equal(got[np.isinf(ref)], ref[np.isinf(ref)])
    if fin.any():
        assert np.abs(got[fin] - ref[fin]).max() <= 2e-6 * np.abs(ref[fin]).max()
    if layer == "fc1":
        assert np.isinf(ref).any()
