"""The FC-512 layer on bf16 planes, where its launches change and tiles end:
forward-only calls from 193 states (tiles of 128 rows), fp32 gradients from 321
rows a learner (128 x 128 tiles, chunks of 32 rows), bf16 gradients of more than
128 rows in all (64-row tiles; the weight gradient first from 257 rows a
learner), against the fp64 oracle, and twice for the same bits.  Q: four layers
of at most 8 roundings of 2^-24 each, 2e-6 of the largest |Q|; gradients: the
bars of every learner test (tests/parity.py), 1e-3 relative L2 a tensor, 2e-2
for bf16 operands."""
import numpy as np
import pytest

import oracle
import parity
from paper_1507_04296_amd import datagen

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _t(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("n", [192, 193, 256, 385])
def test_forward_rows(n):
    import paper_1507_04296_amd as g
    print(f"[gpu-case] fc1 forward n={n}", flush=True)
    A = 18
    inp = datagen.actor_inputs(7500 + n, n, A)
    ctx = g.Context((n + 1) // 2, A)
    theta, states = _t(inp.theta), _t(inp.states)
    q = g.q_forward(ctx, theta, A, states)
    assert torch.equal(q, g.q_forward(ctx, theta, A, states))
    ctx.check()
    ctx.close()
    rows = [0, 63, 64, 127, 128, 191, n - 1]
    ref = oracle.q_forward(oracle.Net(n_actions=A), inp.theta, inp.states[rows])
    assert np.abs(q.cpu().numpy()[rows] - ref).max() <= 2e-6 * np.abs(ref).max()


@pytest.mark.parametrize("G,b,bf16", [(1, 320, False), (1, 321, False), (1, 385, False),
                                      (2, 353, False), (2, 256, True), (2, 257, True),
                                      (9, 15, True), (3, 65, True)])
def test_gradient_rows(G, b, bf16):
    import paper_1507_04296_amd as g
    print(f"[gpu-case] fc1 backward G={G} b={b} bf16={bf16}", flush=True)
    A = 5
    inp = datagen.grouped_inputs(7600 + G * b, G, b, A)
    rep = g.Replay.stacked(_t(inp.s), _t(inp.s2), _t(inp.a), _t(inp.r), _t(inp.term))
    idx = np.arange(G * b, dtype=np.int64)
    th64 = [datagen.bf16_bits_to_f64(t) for t in inp.theta_bf16]
    tg64 = datagen.bf16_bits_to_f64(inp.target_bf16)
    if bf16:
        ctx = g.Context(b, A, groups=G, dtype=g.GORILA_BF16)
        th, tg = _t(inp.theta_bf16.view(np.int16)), _t(inp.target_bf16.view(np.int16))
    else:  # the same values, held in fp32
        ctx = g.Context(b, A, groups=G)
        th, tg = [_t(t.astype(np.float32)) for t in th64], _t(tg64.astype(np.float32))
    run = lambda: g.learner_step_grouped(ctx, th, tg, A, rep, _t(idx), inp.gamma, 1.0)
    grads, loss = run()
    again, loss2 = run()
    assert torch.equal(grads, again) and torch.equal(loss, loss2)
    ctx.check()
    ctx.close()
    got, got_l = grads.cpu().numpy().reshape(G, -1), loss.cpu().numpy()
    net = oracle.Net(n_actions=A)
    tol = parity.GRAD_TOL_BF16 if bf16 else parity.GRAD_TOL
    for i, th in enumerate(th64):
        rows = idx[i * b:(i + 1) * b]
        ref = oracle.learner_step(net, th, tg64, inp.s[rows], inp.s2[rows], inp.a[rows],
                                  inp.r[rows], inp.term[rows], inp.gamma, 1.0)
        parity.assert_grads_close(got[i], ref["grads"], A, tol)
        assert abs(got_l[i] - ref["loss"]) <= parity.LOSS_TOL * abs(ref["loss"])


def _kernels(call):
    """Names of the kernels that `call` launches."""
    from torch.profiler import ProfilerActivity, profile
    call()
    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CUDA]) as p:
        call()
        torch.cuda.synchronize()
    names = " ".join(e.name for e in p.events())
    if "gorila" not in names:
        pytest.skip("the profiler names no kernels here")
    return names


@pytest.mark.parametrize("n,planes", [(192, False), (193, True)])
def test_forward_tiles(n, planes):
    """The rows above are on the side of the line that they are meant for."""
    import paper_1507_04296_amd as g
    print(f"[gpu-case] fc1 forward tiles n={n}", flush=True)
    A = 18
    inp = datagen.actor_inputs(7500 + n, n, A)
    ctx = g.Context((n + 1) // 2, A)
    theta, states = _t(inp.theta), _t(inp.states)
    names = _kernels(lambda: g.q_forward(ctx, theta, A, states))
    assert ("PgFwdJob" in names) == planes and ("Fc1FwdJob" in names) != planes
    ctx.close()


@pytest.mark.parametrize("G,b,bf16,planes", [(1, 320, False, False), (1, 321, False, True),
                                             (2, 64, True, False), (9, 15, True, True)])
def test_gradient_tiles(G, b, bf16, planes):
    import paper_1507_04296_amd as g
    print(f"[gpu-case] fc1 backward tiles G={G} b={b} bf16={bf16}", flush=True)
    A = 5
    inp = datagen.grouped_inputs(7600 + G * b, G, b, A)
    rep = g.Replay.stacked(_t(inp.s), _t(inp.s2), _t(inp.a), _t(inp.r), _t(inp.term))
    idx = _t(np.arange(G * b, dtype=np.int64))
    th, tg = _t(inp.theta_bf16.view(np.int16)), _t(inp.target_bf16.view(np.int16))
    if not bf16:
        th = [_t(datagen.bf16_bits_to_f64(x).astype(np.float32)) for x in inp.theta_bf16]
        tg = _t(datagen.bf16_bits_to_f64(inp.target_bf16).astype(np.float32))
    ctx = g.Context(b, A, groups=G, dtype=g.GORILA_BF16 if bf16 else g.GORILA_F32)
    names = _kernels(lambda: g.learner_step_grouped(ctx, th, tg, A, rep, idx, inp.gamma, 1.0))
    assert ("PgWgradJob" in names) == planes and ("Fc1WgradJob" in names) != planes
    ctx.check()
    ctx.close()
