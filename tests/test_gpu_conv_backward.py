"""The convolutions' backward launches at the edges of their row counts: dz3 in
four, two or one partial plane (up to 64, 128 and more learner rows), one or
two samples a workgroup (256, and 512 with bf16 operands, run at once), sample
ranges of unequal length, against the fp64 oracle; and twice for the same bits.
Bars as everywhere (tests/parity.py): 1e-3 relative L2 a tensor, 2e-2 for bf16
operands."""
import numpy as np
import pytest

import parity
from paper_1507_04296_amd import datagen

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _t(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _check(g, oracle_mod, ctx, call, thetas64, target64, inp, idx, b, A, tol, shared):
    (grads, loss), stages = parity.stages_of(ctx, call)
    assert {"conv_dgrad", "conv_wgrad"} <= stages
    if torch.cuda.get_device_properties(0).multi_processor_count == 256:
        assert ("conv1_wgrad" not in stages) == shared
    g2, l2 = call()
    assert torch.equal(grads, g2) and torch.equal(loss, l2)
    got, got_l = grads.cpu().numpy().reshape(len(thetas64), -1), loss.cpu().numpy()
    net = oracle_mod.Net(n_actions=A)
    for i, th in enumerate(thetas64):
        rows = idx[i * b:(i + 1) * b]
        ref = oracle_mod.learner_step(net, th, target64, inp.s[rows], inp.s2[rows], inp.a[rows],
                                      inp.r[rows], inp.term[rows], inp.gamma, 1.0)
        parity.assert_grads_close(got[i], ref["grads"], A, tol)
        assert abs(got_l[i] - ref["loss"]) <= parity.LOSS_TOL * abs(ref["loss"])


@pytest.fixture(scope="module")
def oracle_mod():
    import oracle
    return oracle


# also around the rows where conv1's weight gradient shares the others' launch:
# one, two, three and four units of it a wave (32, 64, 96, 128), none (144), and
# the sizes beyond where the others' ranges have room for it again
@pytest.mark.parametrize("B,shared", [(1, True), (2, True), (7, True), (32, True), (40, True),
                                      (64, True), (65, True), (96, True), (128, True), (129, True),
                                      (144, False), (150, True), (176, True), (200, False),
                                      (230, True), (257, False), (513, False)])
def test_fp32_rows(oracle_mod, B, shared):
    import paper_1507_04296_amd as g
    print(f"[gpu-case] conv backward fp32 B={B}", flush=True)
    A = 5
    inp = datagen.learner_inputs(7300 + B, B, A)
    ctx = g.Context(B, A)
    rep = g.Replay.stacked(_t(inp.s), _t(inp.s2), _t(inp.a), _t(inp.r), _t(inp.term))
    th, tg, idx = _t(inp.theta), _t(inp.theta_target), _t(inp.idx)
    _check(g, oracle_mod, ctx, lambda: g.learner_step(ctx, th, tg, A, rep, idx, inp.gamma, 1.0),
           [inp.theta.astype(np.float64)], inp.theta_target.astype(np.float64), inp, inp.idx, B, A,
           parity.GRAD_TOL, shared)
    ctx.check()
    ctx.close()


@pytest.mark.parametrize("G,b", [(2, 32), (2, 64), (3, 43), (16, 33)])
def test_bf16_rows(oracle_mod, G, b):
    import paper_1507_04296_amd as g
    print(f"[gpu-case] conv backward bf16 G={G} b={b}", flush=True)
    A = 5
    inp = datagen.grouped_inputs(7400 + G * b, G, b, A)
    ctx = g.Context(b, A, groups=G, dtype=g.GORILA_BF16)
    rep = g.Replay.stacked(_t(inp.s), _t(inp.s2), _t(inp.a), _t(inp.r), _t(inp.term))
    th, tg = _t(inp.theta_bf16.view(np.int16)), _t(inp.target_bf16.view(np.int16))
    idx = np.arange(G * b, dtype=np.int64)
    _check(g, oracle_mod, ctx,
           lambda: g.learner_step_grouped(ctx, th, tg, A, rep, _t(idx), inp.gamma, 1.0),
           [datagen.bf16_bits_to_f64(t) for t in inp.theta_bf16],
           datagen.bf16_bits_to_f64(inp.target_bf16), inp, idx, b, A, parity.GRAD_TOL_BF16, False)
    ctx.check()
    ctx.close()


@pytest.mark.parametrize("G,b,shared", [(2, 15, True), (2, 16, True), (2, 17, True), (4, 1, True),
                                        (2, 85, True), (4, 42, True), (2, 70, False), (4, 33, False)])
def test_fp32_groups(oracle_mod, G, b, shared):
    """Several fp32 learners: conv1's weight gradient beside the others (and not)."""
    import paper_1507_04296_amd as g
    print(f"[gpu-case] conv backward fp32 G={G} b={b}", flush=True)
    A = 5
    inp = datagen.grouped_inputs(7500 + G * b, G, b, A)
    ctx = g.Context(b, A, groups=G)
    rep = g.Replay.stacked(_t(inp.s), _t(inp.s2), _t(inp.a), _t(inp.r), _t(inp.term))
    th64 = [datagen.bf16_bits_to_f64(t) for t in inp.theta_bf16]
    tg64 = datagen.bf16_bits_to_f64(inp.target_bf16)
    th, tg = [_t(x.astype(np.float32)) for x in th64], _t(tg64.astype(np.float32))
    idx = np.arange(G * b, dtype=np.int64)
    _check(g, oracle_mod, ctx,
           lambda: g.learner_step_grouped(ctx, th, tg, A, rep, _t(idx), inp.gamma, 1.0),
           th64, tg64, inp, idx, b, A, parity.GRAD_TOL, shared)
    ctx.check()
    ctx.close()


# One infinite activation channel (conv1's first bias), gradient (a weight of the
# head) or weight (of conv2, conv3: beside the border, and at pixels where its tap
# is outside) through every backward launch: 4, 2 and 1 planes of dz3, the FC
# layer's fp32 and plane tiles.  Every weight, bias and byte is positive, so no
# infinity meets a zero or another sign and the fp64 oracle's gradient is infinite
# or finite, never NaN; padding and borders have to leave it so.  (Rows a multiple
# of 32: the FC weight gradient's chunks.  Infinite values of W1 are not compared:
# conv1's padding pixels read real gradients.)
@pytest.mark.parametrize("what,B,bf16", [("activation", 32, False), ("activation", 96, False),
                                         ("activation", 160, False), ("activation", 352, False),
                                         ("gradient", 32, False), ("gradient", 96, False),
                                         ("gradient", 160, False), ("gradient", 352, False),
                                         ("gradient", 32, True), ("gradient", 160, True),
                                         ("weight2", 32, False), ("weight2", 160, False),
                                         ("weight3", 32, False), ("weight3", 160, False)])
def test_infinite_operand(oracle_mod, what, B, bf16):
    import paper_1507_04296_amd as g
    print(f"[gpu-case] conv backward infinite {what} B={B} bf16={bf16}", flush=True)
    A = 1
    inp = datagen.learner_inputs(7600 + B, B, A)
    bf = lambda x: torch.from_numpy(x).bfloat16()
    sl = datagen.tensor_slices(A)
    theta = np.abs(bf(inp.theta).float().numpy()) + np.float32(2.0**-10)
    theta = bf(theta).float().numpy()
    target = bf(inp.theta_target).float().numpy()
    theta[{"activation": sl["b1"].start, "gradient": sl["W5"].start,
           "weight2": sl["W2"].start + ((3 * 32 + 2) * 4 + 1) * 4 + 2,
           "weight3": sl["W3"].start + ((5 * 64 + 7) * 3 + 2) * 3}[what]] = np.inf
    inp.s[...] = np.maximum(inp.s, 1)
    rep = g.Replay.stacked(_t(inp.s), _t(inp.s2), _t(inp.a), _t(inp.r), _t(inp.term))
    ctx = g.Context(B, A, dtype=g.GORILA_BF16 if bf16 else g.GORILA_F32)
    th, tg = (_t(x) if not bf16 else bf(x).cuda() for x in (theta, target))
    grads, loss = g.learner_step_grouped(ctx, [th], tg, A, rep, _t(inp.idx), inp.gamma, 1.0)
    ctx.check()
    ctx.close()
    got = grads.cpu().numpy().reshape(-1)
    ref = oracle_mod.learner_step(oracle_mod.Net(n_actions=A), theta.astype(np.float64),
                                  target.astype(np.float64), inp.s[inp.idx], inp.s2[inp.idx], inp.a[inp.idx],
                                  inp.r[inp.idx], inp.term[inp.idx], inp.gamma, 1.0)
    assert np.isinf(loss.cpu().numpy()).all() and np.isinf(ref["loss"])
    for name in parity.TENSORS:
        x, y = got[sl[name]].astype(np.float64), ref["grads"][sl[name]]
        assert not np.isnan(y).any(), name
        inf = np.isinf(y)
        if name == "W1":
            x, y, inf = x[~inf], y[~inf], inf[~inf]
        assert np.array_equal(x[inf], y[inf]) and np.isfinite(x[~inf]).all(), (name, int(np.isnan(x).sum()))
        if not inf.all():
            tol = parity.GRAD_TOL_BF16 if bf16 else parity.GRAD_TOL
            assert np.linalg.norm(x[~inf] - y[~inf]) <= tol * np.linalg.norm(y[~inf]), name
