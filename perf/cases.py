"""The work that a user of this library has it do, as cases that can be timed: what a pass is, what it is given, what it
returns, what it cannot do without and how far two correct results may differ.

A case is one of five kinds of use, all through the public calls of the package:

  act      one batched Q evaluation with epsilon-greedy selection (dqn_act), W states that are on the device already
  gather   one minibatch drawn and assembled (replay_sample_gather) for a training loop of the caller's own
  train    the train steps between two synchronisation points: dqn_sync_target, then `steps` train steps, either
           dqn_train_step_sampled (the next minibatch prepared ahead) or replay_sample_gather + dqn_train_step, then the
           parameters read back, as a program does to save or evaluate them
  rounds   the synchronized sampler and the trainer driven from one thread: per round four dqn_act_push_step and one
           dqn_train_step_sampled, between two synchronisation points; the Q rows and the parameters come back
  alg1     the whole of Algorithm 1 (dqn_alg1_run) for one target period, sampler and trainer threads and both streams

Sizes: W from a single environment to 256, minibatches from 16 to 512, both precisions, Double DQN, both target settings.
"""
import math

import numpy as np
import torch

import paper_2111_01264_amd as P

# Layers of the Q-network: (weights, fan in, multiply-adds per state); the last layer depends on the number of actions.
_LAYERS = ((32 * 256, 256, 400 * 32 * 256), (64 * 512, 512, 81 * 64 * 512), (64 * 576, 576, 49 * 64 * 576), (512 * 3136, 3136, 512 * 3136))
_BIASES = (32, 64, 64, 512)
_FRAME = 84 * 84
_PIXEL_T, _BACKGROUND = 838861, 40     # 5 % of the pixels uniform, the rest background
_EPSILON = 0.1
_POOL = 16                             # different states / frames that the rounds cycle through


def _num_params(A):
    return sum(n for n, _, _ in _LAYERS) + sum(_BIASES) + 513 * A


def _steps(B, precision):
    """Train steps of a pass: a stretch of the schedule that is long next to reading the parameters back once (1 ms)."""
    return max(100, min(250, 32000 // B)) if precision == "bf16" else max(30, min(60, 8000 // B))


def _case(name=None, **kw):
    c = dict(kind="act", precision="bf16", A=18, W=0, B=0, steps=1, frames=0, double=False, use_target=True, sampled=True)
    c.update(kw)
    if name:
        c["name"] = name
    return c


def _train(name=None, **kw):
    kw.setdefault("steps", _steps(kw["B"], kw.get("precision", "bf16")))
    kw.setdefault("frames", 100000)
    return _case(name, kind="train", **kw)


def listed():
    return [
        # one environment in full precision: the smallest call, nothing but latency (an evaluation episode, a first test)
        _case("act_w1_fp32", precision="fp32", A=4, W=1),
        # a round of the eight synchronized samplers of the paper's main experiments
        _case("act_w8_bf16", W=8),
        # vectorised environments, the largest round that the benchmark's sweep acts for
        _case("act_w128_bf16", W=128),
        # a minibatch for the caller's own training loop, at the sweep's middle size
        _case("gather_b256", kind="gather", B=256, frames=100000),
        # the small full-precision configuration: 4 actions, a replay memory of 10,000 frames, minibatch 32
        _train("train_b32_fp32", precision="fp32", A=4, B=32, frames=10000),
        # the paper's training: minibatch 32 from a replay memory of a million frames
        _train("train_b32_bf16", B=32, frames=1000000),
        # an odd minibatch through the separate calls, with theta^- as it is in standard DQN
        _train("train_b45_bf16_separate", A=6, B=45, sampled=False),
        # full precision at a large minibatch
        _train("train_b256_fp32", precision="fp32", B=256),
        # Double DQN at the size of its configuration
        _train("train_b256_double_bf16", B=256, double=True),
        # the largest minibatch of the sweep
        _train("train_b512_bf16", B=512),
        # synchronized execution with six actions, acting and training interleaved by one thread
        _case("rounds_w8_b32_bf16", kind="rounds", A=6, W=8, B=32, steps=100, frames=100000),
        # the paper's program: eight samplers, minibatch 32, a train step every four timesteps
        _case("alg1_w8_b32_bf16", kind="alg1", W=8, B=32, steps=500, frames=100000),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 0.49)))))))


def draw(rng):
    A = rng.choice((3, 4, 6, 9, 14, 18, 18, 18))
    precision = rng.choice(("bf16", "bf16", "fp32"))
    kind = rng.choice(("act", "act", "act", "gather", "train", "train", "train", "train", "rounds", "alg1"))
    if kind == "act":
        return _case(precision=precision, A=A, W=_log_int(rng, 1, 256), use_target=rng.random() < 0.75)
    if kind == "gather":
        return _case(kind="gather", A=A, B=_log_int(rng, 16, 512), frames=8 * rng.randint(2000, 12000))
    if kind == "train":
        B = _log_int(rng, 16, 512 if precision == "bf16" else 256)
        return _train(precision=precision, A=A, B=B, double=rng.random() < 0.3, sampled=rng.random() < 0.75, frames=8 * rng.randint(2000, 12000))
    if kind == "rounds":
        W = rng.choice((2, 4, 5, 8, 10, 16, 32))
        return _case(kind="rounds", A=A, W=W, B=_log_int(rng, 16, 128), steps=rng.randint(40, 100), frames=W * rng.randint(2000, 6000))
    W = rng.choice((2, 4, 5, 8, 10))
    return _case(kind="alg1", A=A, W=W, B=_log_int(rng, 16, 64), steps=4 * rng.randint(50, 250), frames=W * rng.randint(4000, 10000))


# ---- what a program has in hand -----------------------------------------------------------------------------------

_STREAMS = []


def _streams():
    """The program's act stream and train stream: made once, as every program of this kind does."""
    if not _STREAMS:
        _STREAMS.extend((torch.cuda.Stream(), torch.cuda.Stream()))
    return _STREAMS


class Agent:
    """A context, and what goes with it, given back when the object goes."""

    def __init__(self, case, seed):
        self.case, self.seed = case, seed
        self.ctx = self.rb = self.alg1 = None
        self.train_steps = self.act_steps = 0
        act, train = _streams()
        cfg = P.dqn_config()
        cfg.num_actions, cfg.max_batch, cfg.max_envs = case["A"], max(case["B"], 1), max(case["W"], 1)
        cfg.precision = P.DQN_PRECISION_BF16 if case["precision"] == "bf16" else P.DQN_PRECISION_FP32
        cfg.double_dqn, cfg.centered = int(case["double"]), 1
        cfg.gamma, cfg.huber_delta, cfg.lr, cfg.rms_alpha, cfg.rms_eps = 0.99, 1.0, 2.5e-4, 0.95, 0.01
        cfg.seed = seed
        self.ctx = P.dqn_create(cfg, act, train)
        theta = initial_parameters(seed, case["A"])
        P.dqn_set_params(self.ctx, P.DQN_PARAMS_ONLINE, theta)
        P.dqn_set_params(self.ctx, P.DQN_PARAMS_TARGET, theta)

    def __del__(self):
        if not callable(getattr(P, "dqn_destroy", None)):
            return      # the interpreter is ending and has taken the package apart
        if self.alg1 is not None:
            P.dqn_alg1_destroy(self.alg1)
        if self.rb is not None:
            P.replay_destroy(self.rb)
        if self.ctx is not None:
            P.dqn_destroy(self.ctx)


def initial_parameters(seed, A):
    """Every tensor uniform in +-1/sqrt(fan in); the output biases are spread evenly, as the action values of a network that
    has learned something are, so that the greedy action is no matter of rounding."""
    rng = np.random.default_rng(seed)
    parts = []
    for (n, fan, _), nb in zip(_LAYERS + ((512 * A, 512, 0),), _BIASES + (A,)):
        parts.append(rng.uniform(-1, 1, n).astype(np.float32) / np.float32(math.sqrt(fan)))
        parts.append(rng.uniform(-1, 1, nb).astype(np.float32) / np.float32(math.sqrt(fan)))
    parts[-1] = rng.permutation(np.linspace(-0.5, 0.5, A)).astype(np.float32)
    return np.concatenate(parts)


def _frames(n, seed, first, stream=None):
    f = torch.empty((n, 84, 84), dtype=torch.uint8, device="cuda")
    P.synth_frames(f, n, first, 1, seed, 2, _PIXEL_T, _BACKGROUND, stream)
    return f


def _threshold(p):
    return int(p * (1 << 24))


def _outcomes(n, seed, first, A, p_reward, p_term, stream=None):
    a = torch.empty(n, dtype=torch.int32, device="cuda")
    r = torch.empty(n, dtype=torch.float32, device="cuda")
    t = torch.empty(n, dtype=torch.uint8, device="cuda")
    P.synth_transitions(a, r, t, n, first, 1, seed, A, _threshold(p_reward), _threshold(p_reward), _threshold(p_term), stream)
    return a, r, t


def _fill(agent, lanes, staging):
    """A replay memory filled to the brim: `frames` experiences in `lanes` lanes, a terminal state every thousand (Double DQN's
    configuration: every hundred)."""
    case, seed = agent.case, agent.seed
    act, train = _streams()
    per_lane = case["frames"] // lanes
    chunk = min(5000, per_lane)
    agent.rb = P.replay_create(per_lane * lanes, lanes, min(per_lane, max(staging, chunk)), seed, act, train)
    p_reward, p_term = (0.1, 0.01) if case["double"] else (0.05, 0.001)
    with torch.cuda.stream(act):
        for lo in range(0, per_lane, chunk):
            n = min(chunk, per_lane - lo)
            for lane in range(lanes):
                first = lane * per_lane + lo
                f = torch.empty((n, 84, 84), dtype=torch.uint8, device="cuda")
                P.synth_frames(f, n, first, 1, seed, 0, _PIXEL_T, _BACKGROUND, act)
                P.replay_push(agent.rb, lane, f, *_outcomes(n, seed, first, case["A"], p_reward, p_term, act), n)
            P.replay_flush(agent.rb, 0)
    torch.cuda.synchronize()


def _minibatch_buffers(B):
    s = torch.empty((B, 4, 84, 84), dtype=torch.uint8, device="cuda")
    return dict(s=s, s2=torch.empty_like(s), a=torch.empty(B, dtype=torch.int32, device="cuda"),
                r=torch.empty(B, dtype=torch.float32, device="cuda"), d=torch.empty(B, dtype=torch.float32, device="cuda"))


def prepare(case, seed):
    agent = Agent(case, seed)
    W, B, A = case["W"], case["B"], case["A"]
    if case["kind"] == "act":
        agent.states = _frames(4 * W, seed, 0).view(W, 4, 84, 84)
        agent.actions = torch.zeros(W, dtype=torch.int32, device="cuda")
        agent.q = torch.zeros((W, A), dtype=torch.float32, device="cuda")
    elif case["kind"] == "gather":
        _fill(agent, 8, 1)
        agent.mb = _minibatch_buffers(B)
        agent.idx = torch.zeros(B, dtype=torch.int64, device="cuda")
    elif case["kind"] == "train":
        _fill(agent, 8, 1)
        agent.loss = torch.zeros(1, dtype=torch.float32, device="cuda")
        agent.mb = None if case["sampled"] else _minibatch_buffers(B)
    elif case["kind"] == "rounds":
        n = 4 * case["steps"]
        _fill(agent, W, n)
        agent.loss = torch.zeros(1, dtype=torch.float32, device="cuda")
        states = _frames(_POOL * W * 4, seed, 0).view(_POOL, W, 4, 84, 84)
        agent.states = [states[k] for k in range(_POOL)]
        frames = _frames(_POOL * W, seed, 1 << 40).view(_POOL, W, 84, 84)
        _, r, t = _outcomes(_POOL * W, seed, 1 << 41, A, 0.05, 0.001)
        agent.stepped = [(frames[k], r.view(_POOL, W)[k], t.view(_POOL, W)[k]) for k in range(_POOL)]
        agent.actions = torch.zeros((n, W), dtype=torch.int32, device="cuda")
        agent.q = torch.zeros((n, W, A), dtype=torch.float32, device="cuda")
        agent.rows = [(agent.actions[k], agent.q[k]) for k in range(n)]
    else:
        act, train = _streams()
        period = _period(case)
        agent.rb = P.replay_create(case["frames"] // W * W, W, period // W, seed, act, train)
        ac = P.dqn_alg1_config()
        ac.W, ac.C, ac.F, ac.B, ac.epsilon = W, period, 4, B, _EPSILON
        ac.t_reward_neg, ac.t_reward_pos, ac.t_term = _threshold(0.05), _threshold(0.05), _threshold(0.001)
        ac.concurrent, ac.synchronized, ac.env_step_ns, ac.env_seed = 1, 1, 0, seed
        agent.alg1 = P.dqn_alg1_create(agent.ctx, agent.rb, ac)
        for _ in range(2):
            P.dqn_alg1_prepopulate(agent.alg1, period)
    torch.cuda.synchronize()
    return agent


def _period(case):
    """Timesteps between two synchronisation points: four per train step, whole rounds of W."""
    unit = 4 * case["W"] // math.gcd(4, case["W"])
    return max(1, 4 * case["steps"] // unit) * unit


# ---- one pass --------------------------------------------------------------------------------------------------------

def run(agent):
    return _RUN[agent.case["kind"]](agent, agent.case)


def _run_act(agent, case):
    P.dqn_act(agent.ctx, agent.states, case["W"], _EPSILON, agent.act_steps, int(case["use_target"]), agent.actions, agent.q)
    agent.act_steps += 1
    return agent.actions, agent.q


def _run_gather(agent, case):
    mb = agent.mb
    P.replay_sample_gather(agent.rb, case["B"], agent.train_steps, None, mb["s"], mb["s2"], mb["a"], mb["r"], mb["d"], agent.idx)
    agent.train_steps += 1
    return mb["s"], mb["s2"], mb["a"], mb["r"], mb["d"], agent.idx


def _run_train(agent, case):
    ctx, rb, B, n, mb = agent.ctx, agent.rb, case["B"], case["steps"], agent.mb
    P.dqn_sync_target(ctx, rb, 0)
    for i in range(n):
        if mb is None:
            P.dqn_train_step_sampled(ctx, rb, B, agent.train_steps, i + 1 < n, agent.loss)
        else:
            P.replay_sample_gather(rb, B, agent.train_steps, None, mb["s"], mb["s2"], mb["a"], mb["r"], mb["d"], None)
            P.dqn_train_step(ctx, mb["s"], mb["a"], mb["r"], mb["s2"], mb["d"], B, agent.loss)
        agent.train_steps += 1
    return P.dqn_get_params(ctx, P.DQN_PARAMS_ONLINE)


def _run_rounds(agent, case):
    ctx, rb, W, B, n = agent.ctx, agent.rb, case["W"], case["B"], case["steps"]
    P.dqn_sync_target(ctx, rb, 0)
    before = None      # what the samplers' previous step produced
    for i in range(n):
        P.dqn_train_step_sampled(ctx, rb, B, agent.train_steps, i + 1 < n, agent.loss)
        agent.train_steps += 1
        for k in range(4 * i, 4 * i + 4):
            actions, q = agent.rows[k]
            if before is None:
                P.dqn_act(ctx, agent.states[k % _POOL], W, _EPSILON, agent.act_steps, 1, actions, q)
            else:
                f, a, r, t = before
                P.dqn_act_push_step(ctx, rb, f, a, r, t, agent.states[k % _POOL], W, _EPSILON, agent.act_steps, 1, actions, q)
            f, r, t = agent.stepped[k % _POOL]
            before = f, actions, r, t
            agent.act_steps += 1
    P.replay_push_step(rb, *before)
    # (the actions follow from the Q rows and the draws; training draws the values of a row together, and which of two near
    # equal ones is taken may hang on rounding)
    return agent.q, P.dqn_get_params(ctx, P.DQN_PARAMS_ONLINE)


def _run_alg1(agent, case):
    P.dqn_alg1_run(agent.alg1, _period(case))
    return P.dqn_get_params(agent.ctx, P.DQN_PARAMS_ONLINE)


_RUN = {"act": _run_act, "gather": _run_gather, "train": _run_train, "rounds": _run_rounds, "alg1": _run_alg1}


# ---- what a pass cannot do without, and how near two results are --------------------------------------------------------

def _forward_flops(A):
    return 2.0 * (sum(m for _, _, m in _LAYERS) + 512 * A)


def _act_work(case):
    """The states and one network's parameters read once, the actions and Q rows written."""
    W, A = case["W"], case["A"]
    e = 2 if case["precision"] == "bf16" else 4
    return W * 4 * _FRAME + e * _num_params(A) + W * (4 + 4 * A), W * _forward_flops(A)


def _train_work(case):
    """The minibatch's frames read once (five per transition), both networks' parameters read, theta and the two accumulators
    read and written; forward on s and s', gradients of the weights of every layer and of the inputs of all but the first."""
    B, A = case["B"], case["A"]
    e = 2 if case["precision"] == "bf16" else 4
    fwd = _forward_flops(A)
    flops = B * ((3 if case["double"] else 2) * fwd + 2 * fwd - 2.0 * _LAYERS[0][2])
    return B * (5 * _FRAME + 12) + (24 + e) * _num_params(A), flops


def work(case):
    kind, n = case["kind"], case["steps"]
    if kind == "gather":
        return {"bytes": case["B"] * (5 * _FRAME + 8 * _FRAME + 12 + 8), "flops": 0}
    if kind == "act":
        b, f = _act_work(case)
        return {"bytes": b, "flops": f}
    b, f = _train_work(case)
    acts = 4 * n if kind == "rounds" else _period(case) // case["W"] if kind == "alg1" else 0
    trains = _period(case) // 4 if kind == "alg1" else n
    ab, af = _act_work(case) if acts else (0, 0)
    pushed = 2 * acts * case["W"] * _FRAME * 2      # into the temporary buffers, and from there into the replay memory
    return {"bytes": trains * b + acts * ab + pushed + 4 * _num_params(case["A"]), "flops": trains * f + acts * af}


def tolerance(case):
    """Four times what was seen when each case ran a second time with the hidden channels of every layer in another order: the
    same network, every sum in another order.  Training spreads such differences (a ReLU or, in Double DQN, a maximising action
    that falls the other way once), the parameters themselves move by 3 % in these stretches.  Worst of 150 cases and seeds:
    parameters fp32 rel 3.2e-4, max 0.03; bf16 rel 1.2e-3, max 0.09; bf16 Double DQN rel 4.1e-3, max 0.21; Q rows of an act
    step fp32 below 4e-8; bf16 rel 7e-6, max 5e-5, where an activation rounded the other way moves the network's part of a row
    by up to 2^-9 (the part is a fifth of the row), which is what the bf16 figure below allows."""
    if case["kind"] == "gather":
        return "exact"
    if case["kind"] == "act":
        return {"rel": 1e-6, "max": 1e-5} if case["precision"] == "fp32" else {"rel": 5e-4, "max": 5e-3}
    if case["precision"] == "fp32":
        return {"rel": 1.3e-3, "max": 0.12}
    return {"rel": 1.6e-2, "max": 0.9} if case["double"] else {"rel": 5e-3, "max": 0.4}
