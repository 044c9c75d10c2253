"""Performance cases of the Gorila learner, actor and parameter-server calls.

The cases are the work that a Gorila bundle hands to this library, through its
public calls: actors choosing actions and storing frames, learners drawing a
minibatch from replay and computing the DQN gradient, and the parameter server
applying gradients and handing parameters out again.

    listed()            the cases that are always measured
    draw(rng)           one more case of the same ranges
    prepare(case, seed) what the program holds before the call, on the GPU
    run(state)          one pass through the public calls; returns the outputs
    work(case)          bytes and operations that one pass cannot do without
    tolerance(case)     largest difference two correct implementations show
    exact(case, seed)   the outputs in 64 bits, in plain torch
"""
from __future__ import annotations

import math

import numpy as np
import torch
import torch.nn.functional as F

import paper_1507_04296_amd as g

GAMMA, CLIP = 0.99, 1.0
FRAME = 84 * 84
# (shape, fan_in) of the flat parameter vector's tensors, in order (A = actions)
HIDDEN = (((32, 4, 8, 8), 256), ((32,), 0), ((64, 32, 4, 4), 512), ((64,), 0),
          ((64, 64, 3, 3), 576), ((64,), 0), ((512, 3136), 3136), ((512,), 0))
FWD_MAC = 400 * 32 * 256 + 81 * 64 * 512 + 49 * 64 * 576 + 512 * 3136  # and 512 * A
BWD_MAC = 2 * (81 * 64 * 512 + 49 * 64 * 576 + 512 * 3136) + 400 * 32 * 256  # and 2 * 512


def listed():
    return [
        # One actor of the paper's topology (one environment per actor) asking
        # for its next action: all latency.  The no-allocation call is the one
        # made for such loops.
        dict(name="act_1", kind="act_noalloc", n=1, A=18, eps=0.1),
        # All environments of one GPU stepping together.
        dict(name="act_1024", kind="act", n=1024, A=18, eps=0.05),
        # Q values of a ragged set of states on a bf16 replica (evaluation of
        # a pulled copy; a game with few actions).
        dict(name="q_333_bf16", kind="q", n=333, A=4, bf16=True),
        # The paper's learner step: DQN's minibatch of 32, full action set.
        dict(name="learn_32", kind="learn", B=32, A=18, ring=False),
        # Sixteen such minibatches as one: the library's benchmark.
        dict(name="learn_512", kind="learn", B=512, A=6, ring=False),
        # A minibatch drawn from the paper's replay of a million frames.
        dict(name="learn_ring_256", kind="learn", B=256, A=18, ring=True, capacity=1_000_000),
        # A large, ragged minibatch (gradient accumulated in one call).
        dict(name="learn_2001", kind="learn", B=2001, A=6, ring=False),
        # Sixteen learners with stale bf16 replicas bundled on one GPU.
        dict(name="grouped_16x64_bf16", kind="grouped", G=16, b=64, A=18, bf16=True),
        # A few learners with fp32 replicas and a ragged minibatch.
        dict(name="grouped_4x33", kind="grouped", G=4, b=33, A=18, bf16=False),
        # A sampled minibatch materialised as stacks (for another consumer).
        dict(name="gather_256", kind="gather", n=256, A=18, capacity=1_000_000),
        # One parameter-server turn for sixteen learners: loss filter, AdaGrad
        # apply of their gradients, and the pull into their bf16 replicas.
        dict(name="server_16", kind="server", G=16, A=18),
        # One step of 1024 actors stored into their replay rings.
        dict(name="insert_1024", kind="insert", rings=1024, m=1, capacity=32),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, round(math.exp(rng.uniform(math.log(lo), math.log(hi))))))


def draw(rng):
    """Sizes over the whole range (uniform in the logarithm), odd ones among them."""
    A = rng.choice([3, 4, 6, 9, 14, 18])
    kind = rng.choice(["act_noalloc", "act", "q", "learn", "learn", "learn", "ring", "grouped",
                       "grouped", "gather", "server", "insert"])
    if kind == "act_noalloc":
        return dict(kind=kind, n=_log_int(rng, 1, 256), A=A, eps=rng.choice([0.05, 0.1, 1.0]))
    if kind == "act":
        return dict(kind=kind, n=_log_int(rng, 2, 2048), A=A, eps=rng.choice([0.05, 0.1]))
    if kind == "q":
        return dict(kind=kind, n=_log_int(rng, 1, 2048), A=A, bf16=rng.random() < 0.5)
    if kind == "learn":
        return dict(kind=kind, B=_log_int(rng, 8, 2001), A=A, ring=False)
    if kind == "ring":
        return dict(kind="learn", B=_log_int(rng, 16, 1024), A=A, ring=True,
                    capacity=_log_int(rng, 5_000, 1_000_000))
    if kind == "grouped":
        G = rng.randint(2, 16)
        return dict(kind=kind, G=G, b=_log_int(rng, 8, 1024 // G), A=A, bf16=rng.random() < 0.6)
    if kind == "gather":
        return dict(kind=kind, n=_log_int(rng, 16, 2048), A=A,
                    capacity=_log_int(rng, 5_000, 1_000_000))
    if kind == "server":
        return dict(kind=kind, G=rng.randint(1, 32), A=A)
    return dict(kind=kind, rings=_log_int(rng, 1, 2048), m=rng.randint(1, 4), capacity=16)


# ---- inputs (from the seed alone) ----

def _gen(seed, salt=0):
    return torch.Generator(device="cuda").manual_seed(1507 + 1000003 * int(seed) + salt)


def _shapes(A):
    return HIDDEN + (((A, 512), 512), ((A,), 0))


def _theta(gen, A):
    """He-normal weights and small biases, as a network under training holds them."""
    parts = []
    for shape, fan_in in _shapes(A):
        n = math.prod(shape)
        x = torch.randn(n, generator=gen, device="cuda")
        parts.append(x * (math.sqrt(2.0 / fan_in) if fan_in else 0.01))
    return torch.cat(parts)


def _noise(gen, theta, sigma):
    return theta + sigma * torch.randn(theta.shape, generator=gen, device="cuda")


def _bytes(gen, *shape):
    return torch.randint(0, 256, shape, generator=gen, device="cuda", dtype=torch.uint8)


def _sprites(gen, n):
    """Dark frames with three bright 8x8 sprites moving over the four frames."""
    out = torch.randint(0, 25, (n, 4, 84, 84), generator=gen, device="cuda", dtype=torch.uint8)
    ax = torch.arange(84, device="cuda")
    for _ in range(3):
        bright = torch.randint(160, 256, (n, 1, 1, 1), generator=gen, device="cuda").to(torch.uint8)
        p0 = torch.randint(0, 77, (n, 1, 2), generator=gen, device="cuda")
        vel = torch.randint(-4, 5, (n, 1, 2), generator=gen, device="cuda")
        p = (p0 + vel * torch.arange(4, device="cuda")[None, :, None]).clamp(0, 76)  # [n, 4, 2]
        y, x = p[..., 0, None], p[..., 1, None]
        iy, ix = (ax >= y) & (ax < y + 8), (ax >= x) & (ax < x + 8)
        out = torch.where(iy[..., :, None] & ix[..., None, :], torch.maximum(out, bright), out)
    return out


def _rewards(gen, *shape):
    u = torch.rand(shape, generator=gen, device="cuda")
    return (u > 0.95).float() - (u < 0.05).float()


def _ring(gen, capacity, A):
    """A full ring: random frames, episodes of 2000 frames on average."""
    return dict(frames=_bytes(gen, capacity, 84, 84),
                ep=(torch.rand(capacity, generator=gen, device="cuda") < 1 / 2000).to(torch.uint8),
                action=torch.randint(0, A, (capacity,), generator=gen, device="cuda",
                                     dtype=torch.int32),
                reward=_rewards(gen, capacity),
                head=int(torch.randint(0, capacity, (1,), generator=gen, device="cuda")))


def _replay(gen, rows, A, ring, capacity=0):
    """Replay tensors and a minibatch of `rows` indices."""
    if ring:
        d = _ring(gen, capacity, A)
        d["idx"] = torch.randint(0, capacity - 1, (rows,), generator=gen, device="cuda")
        return d
    return dict(s=_bytes(gen, rows, 4, 84, 84), s2=_bytes(gen, rows, 4, 84, 84),
                action=torch.randint(0, A, (rows,), generator=gen, device="cuda", dtype=torch.int32),
                reward=_rewards(gen, rows),
                term=(torch.rand(rows, generator=gen, device="cuda") < 0.01).to(torch.uint8),
                idx=torch.randperm(rows, generator=gen, device="cuda"))


def _inputs(case, seed):
    kind, gen = case["kind"], _gen(seed)
    if kind in ("act", "act_noalloc", "q"):
        theta = _theta(gen, case["A"])
        return dict(theta=theta.bfloat16() if case.get("bf16") else theta,
                    states=_sprites(gen, case["n"]))
    if kind == "learn":
        theta = _theta(gen, case["A"])
        d = _replay(gen, case["B"], case["A"], case["ring"], case.get("capacity", 0))
        return dict(theta=theta, target=_noise(gen, theta, 0.01), **d)
    if kind == "grouped":  # replicas a few updates apart, one shared target
        base = _theta(gen, case["A"])
        thetas = torch.stack([_noise(gen, base, 0.005) for _ in range(case["G"])])
        target = _noise(gen, base, 0.01)
        if case["bf16"]:
            thetas, target = thetas.bfloat16(), target.bfloat16()
        else:  # rows of a flat fp32 set have to start on 16 bytes
            thetas = [t.clone() for t in thetas]
        d = _replay(gen, case["G"] * case["b"], case["A"], False)
        return dict(theta=thetas, target=target, **d)
    if kind == "gather":
        return _replay(gen, case["n"], case["A"], True, case["capacity"])
    if kind == "server":
        G, theta = case["G"], _theta(gen, case["A"])
        return dict(theta=theta, accum=torch.rand(theta.shape, generator=gen, device="cuda") * 1e-4,
                    grads=1e-3 * torch.randn((G, theta.numel()), generator=gen, device="cuda"),
                    loss=torch.rand(G, generator=gen, device="cuda") * 0.1,
                    stats=torch.tensor([[100.0, 0.05, 0.01]] * G, dtype=torch.float64, device="cuda"))
    R, m = case["rings"], case["m"]
    return dict(frames=_bytes(gen, m, R, 84, 84),
                ep=(torch.rand((m, R), generator=gen, device="cuda") < 1 / 2000).to(torch.uint8),
                action=torch.randint(0, 18, (m, R), generator=gen, device="cuda", dtype=torch.int32),
                reward=_rewards(gen, m, R))


def _empty(*shape, dtype=torch.float32):
    return torch.empty(shape, dtype=dtype, device="cuda")


def prepare(case, seed):
    kind, d = case["kind"], _inputs(case, seed)
    st = dict(case=case, seed=seed, **d)
    if kind in ("act", "act_noalloc", "q"):
        n, A = case["n"], case["A"]
        if kind == "act_noalloc":
            st["ctx"] = g.Context(0, A)
        else:
            st["ctx"] = g.Context((n + 1) // 2, A, dtype=g.dtype_of(d["theta"]))
        st["actions"], st["q"] = _empty(n, dtype=torch.int32), _empty(n, A)
    elif kind in ("learn", "grouped"):
        if kind == "learn":
            A, G, b = case["A"], 1, case["B"]
        else:
            A, G, b = case["A"], case["G"], case["b"]
        st["ctx"] = g.Context(b, A, groups=G, dtype=g.dtype_of(d["target"]))
        if kind == "learn" and case["ring"]:
            st["replay"] = g.Replay.ring(d["frames"], d["ep"], d["action"], d["reward"], d["head"])
        else:
            st["replay"] = g.Replay.stacked(d["s"], d["s2"], d["action"], d["reward"], d["term"])
        P = g.param_count(A)
        st["grads"] = _empty(P) if kind == "learn" else _empty(G, P)
        st["loss"] = _empty(G)
    elif kind == "gather":
        n = case["n"]
        st["ctx"] = g.Context(1, case["A"])
        st["replay"] = g.Replay.ring(d["frames"], d["ep"], d["action"], d["reward"], d["head"])
        st["out"] = dict(s=_empty(n, 4, 84, 84, dtype=torch.uint8),
                         s2=_empty(n, 4, 84, 84, dtype=torch.uint8),
                         frame_map=_empty(n, 2, 4, dtype=torch.int64),
                         a=_empty(n, dtype=torch.int32), r=_empty(n),
                         term=_empty(n, dtype=torch.uint8))
    elif kind == "server":
        G, P = case["G"], d["theta"].numel()
        st["ctx"] = g.Context(0, case["A"])
        st["version"] = torch.zeros(1, dtype=torch.int64, device="cuda")
        st["grad_version"] = torch.zeros(G, dtype=torch.int64, device="cuda")
        st["replicas"] = _empty(min(G, 16), P, dtype=torch.int16)  # bf16 bit patterns
        st["held"] = torch.zeros(min(G, 16), dtype=torch.int64, device="cuda")
        st["keep"], st["applied"] = (_empty(G, dtype=torch.uint8) for _ in range(2))
    else:
        st["ctx"] = g.Context(0, 18)
        st["rings"] = g.RingSet(case["rings"], case["capacity"])
    return st


def run(st):
    case, kind, ctx = st["case"], st["case"]["kind"], st["ctx"]
    if kind == "act":
        g.gorila_act(ctx, st["theta"], case["A"], st["states"], case["eps"], st["seed"],
                     st["actions"], st["q"])
        return dict(actions=st["actions"], q=st["q"])
    if kind == "act_noalloc":
        g.gorila_act_noalloc(ctx, st["theta"], case["A"], st["states"], case["eps"], st["seed"],
                             st["actions"], st["q"])
        return dict(actions=st["actions"], q=st["q"])
    if kind == "q":
        g.gorila_q_forward(ctx, st["theta"], case["A"], st["states"], st["q"])
        return dict(q=st["q"])
    if kind == "learn":
        g.gorila_learner_step(ctx, st["theta"], st["target"], case["A"], st["replay"], st["idx"],
                              GAMMA, CLIP, st["grads"], st["loss"])
        return dict(grads=st["grads"], loss=st["loss"])
    if kind == "grouped":
        g.gorila_learner_step_grouped(ctx, st["theta"], st["target"], case["A"], st["replay"],
                                      st["idx"], case["b"], GAMMA, CLIP, st["grads"], st["loss"])
        return dict(grads=st["grads"], loss=st["loss"])
    if kind == "gather":
        o = st["out"]
        g.gorila_gather(ctx, st["replay"], st["idx"], o["s"], o["s2"], o["frame_map"], o["a"],
                        o["r"], o["term"])
        return o
    if kind == "server":
        # the filter reports, the server applies what the learners sent; no
        # gradient is stale (every learner pulls at the end of its turn)
        g.gorila_loss_filter(ctx, st["stats"], st["loss"], 0.01, 5.0, 10, st["keep"])
        g.gorila_ps_apply(ctx, st["theta"], st["accum"], st["grads"], st["grad_version"],
                          st["version"], 1 << 40, 0.01, 1e-6, st["applied"], keep=st["keep"])
        g.gorila_params_sync(ctx, st["theta"], st["replicas"], st["held"], st["version"], 0)
        return dict(theta=st["theta"], accum=st["accum"], replicas=st["replicas"],
                    stats=st["stats"], keep=st["keep"], applied=st["applied"],
                    version=st["version"], held=st["held"])
    rs = st["rings"]
    g.gorila_replay_insert(ctx, rs, st["frames"], st["ep"], st["action"], st["reward"])
    return dict(frames=rs.frames, ep=rs.ep_start, action=rs.action, reward=rs.reward)


def work(case):
    kind = case["kind"]
    P = sum(math.prod(s) for s, _ in _shapes(case["A"])) if "A" in case else 0
    if kind in ("act", "act_noalloc", "q"):
        n, A = case["n"], case["A"]
        return dict(bytes=n * 4 * FRAME + P * (2 if case.get("bf16") else 4) + n * (A + 1) * 4,
                    flops=2 * n * (FWD_MAC + 512 * A))
    if kind in ("learn", "grouped"):
        G, rows = (1, case["B"]) if kind == "learn" else (case["G"], case["G"] * case["b"])
        frames = 5 if case.get("ring") else 8
        return dict(bytes=rows * frames * FRAME + (G + 1) * P * (2 if case.get("bf16") else 4)
                    + G * P * 4,
                    flops=2 * rows * (2 * (FWD_MAC + 512 * case["A"]) + BWD_MAC + 2 * 512))
    if kind == "gather":
        return dict(bytes=case["n"] * 13 * FRAME, flops=0)
    if kind == "server":
        G = case["G"]
        return dict(bytes=P * (4 * G + 16 + 2 * min(G, 16)), flops=6 * G * P)
    return dict(bytes=case["rings"] * case["m"] * 2 * FRAME, flops=0)


def tolerance(case):
    kind = case["kind"]
    if kind in ("gather", "insert"):
        return "exact"
    # About four times the largest error against exact() over the ranges.
    if kind == "server":  # measured 1e-7; replicas round the last bit of theta+ either way
        return {"rel": 5e-7, "differ": 1e-3}
    if kind in ("act", "act_noalloc", "q"):  # measured 7e-7; near ties between actions
        return {"rel": 3e-6, "differ": 2e-3}
    # Measured 3e-7 (fp32) without, and up to 2.6e-4 with hidden units whose
    # sum rounds to the other side of zero: such a unit takes its sample's
    # gradient with it, so the error is a few units' shares and not the
    # rounding of the sums.  bf16 replicas: 2e-3.
    return {"rel": 1e-2} if case.get("bf16") else {"rel": 1e-3}


# ---- the outputs in 64 bits ----

def _split(theta, A):
    out, o = [], 0
    for shape, _ in _shapes(A):
        n = math.prod(shape)
        out.append(theta[o:o + n].view(shape))
        o += n
    return out


def _conv(x, w, b, k, stride):
    n, h = x.shape[0], (x.shape[2] - k) // stride + 1
    cols = F.unfold(x, k, stride=stride)  # [n, C k k, h h]
    y = cols.transpose(1, 2).reshape(n * h * h, -1) @ w.reshape(w.shape[0], -1).t() + b
    return F.relu(y).view(n, h * h, -1).transpose(1, 2).reshape(n, -1, h, h)


def _q64(p, states):
    x = states.double() / 255.0
    x = _conv(x, p[0], p[1], 8, 4)
    x = _conv(x, p[2], p[3], 4, 2)
    x = _conv(x, p[4], p[5], 3, 1)
    x = F.relu(x.reshape(x.shape[0], -1) @ p[6].t() + p[7])
    return x @ p[8].t() + p[9]


CHUNK = 128


def _step64(theta, target, A, s, s2, a, r, term):
    th = theta.double().requires_grad_(True)
    p, pt = _split(th, A), _split(target.double(), A)
    B, total = s.shape[0], 0.0
    for i in range(0, B, CHUNK):
        sl = slice(i, i + CHUNK)
        with torch.no_grad():
            y = r[sl].double() + GAMMA * (term[sl] == 0) * _q64(pt, s2[sl]).max(1).values
        q = _q64(p, s[sl]).gather(1, a[sl].long()[:, None])[:, 0]
        part = F.huber_loss(q, y, reduction="sum", delta=CLIP) / B
        part.backward()
        total += part.detach()
    return th.grad, total.reshape(1)


def _stacks(d, idx):
    """Frames, map, action, reward and terminal flag of ring transitions."""
    cap = d["frames"].shape[0]
    slot = lambda k: (d["head"] + k) % cap
    k = idx[:, None] + torch.arange(2, device="cuda")  # newest frame of s and s'
    l = k[..., None] + torch.arange(-3, 1, device="cuda")  # [n, 2, 4]
    starts = (d["ep"][slot(l.clamp(min=0))] != 0) | (l <= 0)
    # a frame stays if no later frame of the stack starts an episode
    later = starts.flip(-1).cumsum(-1).flip(-1) - starts.long()
    ok = (l >= 0) & (later == 0)
    fmap = torch.where(ok, slot(l.clamp(min=0)), -1)
    x = d["frames"][fmap.clamp(min=0)] * ok[..., None, None].to(torch.uint8)
    return (x[:, 0], x[:, 1], fmap, d["action"][slot(idx)], d["reward"][slot(idx)],
            (d["ep"][slot(idx + 1)] != 0).to(torch.uint8))


def _mix(z):
    z = (z ^ (z >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
    z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
    return z ^ (z >> np.uint64(31))


def _greedy(q, eps, seed, A):
    """The documented epsilon-greedy draws (SplitMix64 on a counter)."""
    e = np.arange(q.shape[0], dtype=np.uint64)
    G = np.uint64(0x9E3779B97F4A7C15)
    seed = np.uint64(seed & (2 ** 64 - 1))
    with np.errstate(over="ignore"):
        u = _mix(seed + (np.uint64(2) * e + np.uint64(1)) * G)
        v = _mix(seed + (np.uint64(2) * e + np.uint64(2)) * G)
        rnd = ((v >> np.uint64(32)) * np.uint64(A)) >> np.uint64(32)
    explore = (u >> np.uint64(11)) < np.uint64(math.floor(float(np.float32(eps)) * 2 ** 53))
    best = q.argmax(1).cpu().numpy()
    return torch.from_numpy(np.where(explore, rnd.astype(np.int64), best).astype(np.int32))


def exact(case, seed):
    kind = case["kind"]
    d = _inputs(case, seed)
    if kind in ("act", "act_noalloc", "q"):
        p = _split(d["theta"].double(), case["A"])
        q = torch.cat([_q64(p, x) for x in d["states"].split(CHUNK)])
        if kind == "q":
            return dict(q=q)
        return dict(actions=_greedy(q, case["eps"], seed, case["A"]), q=q)
    if kind == "learn":
        idx = d["idx"]
        if case["ring"]:
            s, s2, _, a, r, term = _stacks(d, idx)
        else:
            s, s2, a, r, term = (d[k][idx] for k in ("s", "s2", "action", "reward", "term"))
        grads, loss = _step64(d["theta"], d["target"], case["A"], s, s2, a, r, term)
        return dict(grads=grads, loss=loss)
    if kind == "grouped":
        out = []
        for i in range(case["G"]):
            idx = d["idx"][i * case["b"]:(i + 1) * case["b"]]
            rows = (d[k][idx] for k in ("s", "s2", "action", "reward", "term"))
            out.append(_step64(d["theta"][i], d["target"], case["A"], *rows))
        return dict(grads=torch.stack([x for x, _ in out]), loss=torch.cat([x for _, x in out]))
    if kind == "gather":
        s, s2, fmap, a, r, term = _stacks(d, d["idx"])
        return dict(s=s, s2=s2, frame_map=fmap, a=a, r=r, term=term)
    if kind == "server":
        G, alpha, k = case["G"], 0.01, 5.0
        x, st = d["loss"].double(), d["stats"]
        n, mean, var = st[:, 0], st[:, 1], st[:, 2]
        dx = x - mean
        keep = ~((x > mean) & (dx * dx > k * k * var))
        stats = torch.stack([n + 1, mean + alpha * dx, (1 - alpha) * (var + alpha * dx * dx)], 1)
        th, h = d["theta"].double(), d["accum"].double()
        # lr and eps as the fp32 arguments hold them
        lr, eps = float(np.float32(0.01)), float(np.float32(1e-6))
        for i in range(G):
            if keep[i]:
                gi = d["grads"][i].double()
                h = h + gi * gi
                th = th - lr * gi / (eps + h.sqrt())
        version = keep.sum().reshape(1)
        C = min(G, 16)
        return dict(theta=th, accum=h, replicas=None, stats=stats, keep=keep.to(torch.uint8),
                    applied=keep.to(torch.uint8), version=version, held=version.expand(C).clone())
    R, m, cap = case["rings"], case["m"], case["capacity"]
    rs = {"frames": torch.zeros((R, cap, 84, 84), dtype=torch.uint8, device="cuda"),
          "ep": torch.zeros((R, cap), dtype=torch.uint8, device="cuda"),
          "action": torch.zeros((R, cap), dtype=torch.int32, device="cuda"),
          "reward": torch.zeros((R, cap), dtype=torch.float32, device="cuda")}
    for key, t in rs.items():
        t[:, :m] = d[key].transpose(0, 1)
    return rs
