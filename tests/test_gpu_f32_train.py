"""Full-precision train step against the fp64 oracle at the minibatch sizes where its kernels change shape: one sample, a pair,
the last small-batch size and its neighbours, the last one whose samples are run in sevenths / thirds / halves, several samples per
workgroup with a ragged last range; and, at 96 and 101, through the replay memory, where the minibatch exists only as replay slots.

On inputs where no ReLU can flip (see test_gpu_bf16_backward.py) what is left is fp32 rounding: a gradient element is a sum of
up to 400 B products whose accumulator chain is at most 5,000 additions long; their roundings (2^-24 of the running sum) add like
a random walk to 2^-24 * sqrt(5000) = 4e-6 of the largest partial sum, and the factors of up to four layers, dL/dQ and the slice
sums add in the same way: 1e-5 of a tensor's largest element.  Asserted: ten times that.
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

import paper_2111_01264_amd as P
from datagen import synth
from oracle import dqn as odqn
from oracle.replay import OracleReplay
from tests.gpu_util import blob_slices, dev, make_cfg, rel_err

TOL = 1e-4
REWARDS = np.array([-30.0, -2.0, 2.0, 30.0], dtype=np.float32)


def check_step(ctx, orc, A, B, double_dqn, theta, theta_t, s, a, r, s2, d, loss, lr, eps):
    """Q rows, loss, gradient and update of the library's first step against the oracle's on the same minibatch."""
    wloss, q_sa, _ = orc.train_step(s, a, r, s2, d)
    q_on, q_nt, _ = P.dqn_get_train_q(ctx, B, A, bool(double_dqn))
    assert rel_err(q_on, q_sa) <= TOL
    assert rel_err(q_nt, odqn.forward(orc.desc, theta_t.astype(np.float64), odqn.scale_states(s2))[0]) <= TOL
    assert abs(float(loss.item()) - wloss) <= TOL * abs(wloss)
    g = P.dqn_get_params(ctx, P.DQN_PARAMS_GRAD)
    th = P.dqn_get_params(ctx, P.DQN_PARAMS_ONLINE)
    errs = {name: rel_err(g[slc], orc.last_grad[slc]) for name, slc in blob_slices(A).items()}
    print("B=%d per-tensor max-norm gradient errors: %s" % (B, " ".join("%s %.1e" % kv for kv in errs.items())))
    for name, slc in blob_slices(A).items():
        assert errs[name] <= TOL, (name, errs[name])
        # |d(update)/dg| <= lr / eps for the first step from zero state; plus half an ulp of theta
        bound = lr / eps * TOL * np.abs(orc.last_grad[slc]).max() + 2.0 ** -24 * np.abs(theta[slc]).max()
        got, want = th[slc].astype(np.float64) - theta[slc], orc.theta[slc] - theta[slc]
        assert np.abs(got - want).max() <= bound, ("update", name)


@pytest.mark.parametrize("B,split,double_dqn", [(1, True, 0), (2, False, 1), (18, True, 0), (31, True, 1), (33, True, 0), (42, False, 0), (64, True, 0), (65, True, 1), (131, True, 0), (257, False, 1)])
def test_f32_train_step_max_norm_no_relu_flips(B, split, double_dqn):
    A, seed, lr = 6, 5200 + B, 2.5e-5
    cfg = make_cfg(A, max_batch=B, max_envs=8, precision=P.DQN_PRECISION_FP32, double_dqn=double_dqn, seed=seed)
    cfg.lr, cfg.huber_delta = lr, 10.0
    ctx = P.dqn_create(cfg, torch.cuda.Stream(), torch.cuda.Stream())
    try:
        theta = synth.margin_params(seed, A, split)
        theta_t = synth.margin_params(seed + 1, A, split)
        P.dqn_set_params(ctx, P.DQN_PARAMS_ONLINE, theta)
        P.dqn_set_params(ctx, P.DQN_PARAMS_TARGET, theta_t)
        orc = odqn.OracleDQN(A, theta, double_dqn=bool(double_dqn), seed=seed, lr=lr, huber=10.0)
        orc.theta_target = theta_t.astype(np.float64)
        rng = np.random.default_rng(seed)
        s = synth.block_frames(seed + 10, B * 4).reshape(B, 4, 84, 84)
        s2 = synth.block_frames(seed + 20, B * 4).reshape(B, 4, 84, 84)
        a = rng.integers(0, A, size=B).astype(np.int32)
        r = REWARDS[rng.integers(0, 4, size=B)]
        d = (rng.random(B) < 0.2).astype(np.float32)
        loss = torch.zeros(1, dtype=torch.float32, device="cuda")
        P.dqn_train_step(ctx, dev(s), dev(a), dev(r), dev(s2), dev(d), B, loss)
        torch.cuda.synchronize()
        check_step(ctx, orc, A, B, double_dqn, theta, theta_t, s, a, r, s2, d, loss, lr, cfg.rms_eps)
    finally:
        P.dqn_destroy(ctx)


@pytest.mark.parametrize("B,double_dqn", [(96, 0), (101, 1)])
def test_f32_sampled_train_step_max_norm_no_relu_flips(B, double_dqn):
    A, lanes, per_lane, seed, lr = 6, 4, 60, 5600 + B, 2.5e-5
    cfg = make_cfg(A, max_batch=B, max_envs=4, precision=P.DQN_PRECISION_FP32, double_dqn=double_dqn, seed=seed)
    cfg.lr, cfg.huber_delta = lr, 10.0
    sa, st = torch.cuda.Stream(), torch.cuda.Stream()
    ctx = P.dqn_create(cfg, sa, st)
    rb = P.replay_create(lanes * per_lane, lanes, per_lane, seed, sa, st)
    orep = OracleReplay(lanes * per_lane, lanes, seed)
    try:
        theta = synth.margin_params(seed, A, True)
        theta_t = synth.margin_params(seed + 1, A, True)
        P.dqn_set_params(ctx, P.DQN_PARAMS_ONLINE, theta)
        P.dqn_set_params(ctx, P.DQN_PARAMS_TARGET, theta_t)
        orc = odqn.OracleDQN(A, theta, double_dqn=bool(double_dqn), seed=seed, lr=lr, huber=10.0)
        orc.theta_target = theta_t.astype(np.float64)
        rng = np.random.default_rng(seed)
        for lane in range(lanes):
            f = synth.block_frames(seed + 1 + lane, per_lane)
            a = rng.integers(0, A, size=per_lane).astype(np.int32)
            r = REWARDS[rng.integers(0, 4, size=per_lane)]
            d = (rng.random(per_lane) < 0.05).astype(np.uint8)
            P.replay_push(rb, lane, dev(f), dev(a), dev(r), dev(d), per_lane)
            orep.push(lane, f, a, r, d)
        P.replay_flush(rb, 1)
        orep.flush()
        loss = torch.zeros(1, dtype=torch.float32, device="cuda")
        P.dqn_train_step_sampled(ctx, rb, B, 0, 0, loss)
        torch.cuda.synchronize()
        ws, ws2, wa, wr, wd = orep.gather(orep.sample_indices(B, 0))
        check_step(ctx, orc, A, B, double_dqn, theta, theta_t, ws, wa, wr, ws2, wd, loss, lr, cfg.rms_eps)
    finally:
        P.replay_destroy(rb)
        P.dqn_destroy(ctx)
