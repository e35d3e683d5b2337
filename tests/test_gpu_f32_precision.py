"""Precision of the full-precision mode.  Train step: the error of every gradient tensor against the fp64 oracle, as a norm, is no larger than
the error of the same step with every product on the fp32 matrix instruction.

The inputs leave nothing but the backward pass's own rounding: every ReLU has one state for any input (a hidden channel's bias is
larger than the largest weighted sum its inputs can reach, odd channels have it negative) and every TD error is clipped, so dL/dQ is
exactly +-1/B.  Weights have both signs, so the data gradients are sums with cancellation, and since the activations are nearly
constant the weight gradients are, like the bias gradients, sums over all pixels and samples of a data gradient: a rounding
that is not to nearest but always to one side, which a comparison element by element does not see, adds up there.

RECORDED holds the errors of the kernels that computed everything on the fp32 instruction, layer by layer, on the same inputs (both
sides are deterministic); a tenth is allowed on top, for sums of the same precision in another order (fc1.w, whose products
are still made by that instruction, moved by up to 4 % when only the order of its sums changed).

Act step: likewise the network's part of the Q rows (without fc2's biases), on weights as they are initialised.
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

import paper_2111_01264_amd as P
from datagen import synth
from oracle import dqn as odqn
from tests.gpu_util import blob_slices, dev, make_cfg

SLACK = 1.1
SCALE = {"conv1": 0.25, "conv2": 0.2, "conv3": 0.1, "fc1": 0.02, "fc2": 0.02}


def steady_params(seed, A):
    """init_params scaled by SCALE, each hidden bias 0.5 beyond what the channel's inputs can reach (odd channels: negative)."""
    theta = synth.init_params(seed, A).astype(np.float64)
    off, top = 0, 1.0
    for name, shape, _ in synth.layer_shapes(A):
        n = int(np.prod(shape))
        w = theta[off:off + n].reshape(shape[0], -1)
        w *= SCALE[name]
        if name != "fc2":
            reach = np.abs(w).sum(1) * top + 0.5
            theta[off + n:off + n + shape[0]] = reach * np.where(np.arange(shape[0]) % 2, -1.0, 1.0)
            top = 2.0 * reach.max()
        off += n + shape[0]
    return theta.astype(np.float32)


def one_sign_params(seed, A):
    """The same weights with one sign per channel (odd channels negative, their bias too): a data gradient is then a sum of one sign, a
    sample's bias gradient is large, and what is left over the samples, whose errors are clipped to either side, is small."""
    theta = synth.init_params(seed, A).astype(np.float64)
    off = 0
    for name, shape, _ in synth.layer_shapes(A):
        n = int(np.prod(shape))
        w = theta[off:off + n].reshape(shape[0], -1)
        sign = np.where(np.arange(shape[0]) % 2, -1.0, 1.0) if name != "fc2" else np.ones(shape[0])
        w[:] = np.abs(w) * SCALE[name] * sign[:, None]
        if name != "fc2":
            theta[off + n:off + n + shape[0]] = 0.5 * sign
        off += n + shape[0]
    return theta.astype(np.float32)


SEEDS = 4


def gradient_errors(B, double_dqn, params=steady_params):
    """Root mean square over the seeds: a single draw of 32 bias gradients scatters by a third."""
    runs = [step_errors(B, double_dqn, 6400 + B + 1000 * k, params) for k in range(SEEDS)]
    return {name: float(np.sqrt(np.mean([e[name] ** 2 for e in runs]))) for name in runs[0]}


def step_errors(B, double_dqn, seed, params):
    A = 6
    cfg = make_cfg(A, max_batch=B, max_envs=1, precision=P.DQN_PRECISION_FP32, double_dqn=double_dqn, seed=seed)
    ctx = P.dqn_create(cfg, torch.cuda.Stream(), torch.cuda.Stream())
    try:
        theta, theta_t = params(seed, A), params(seed + 1, A)
        P.dqn_set_params(ctx, P.DQN_PARAMS_ONLINE, theta)
        P.dqn_set_params(ctx, P.DQN_PARAMS_TARGET, theta_t)
        orc = odqn.OracleDQN(A, theta, double_dqn=bool(double_dqn), seed=seed)
        orc.theta_target = theta_t.astype(np.float64)
        rng = np.random.default_rng(seed)
        s = synth.block_frames(seed + 10, B * 4).reshape(B, 4, 84, 84)
        s2 = synth.block_frames(seed + 20, B * 4).reshape(B, 4, 84, 84)
        a = rng.integers(0, A, size=B).astype(np.int32)
        r = np.array([-300.0, 300.0], dtype=np.float32)[rng.integers(0, 2, size=B)]     # |Q| stays below 100: every error is clipped
        d = np.zeros(B, dtype=np.float32)
        P.dqn_train_step(ctx, dev(s), dev(a), dev(r), dev(s2), dev(d), B, None)
        torch.cuda.synchronize()
        g = P.dqn_get_params(ctx, P.DQN_PARAMS_GRAD).astype(np.float64)
        _, q_sa, _ = orc.train_step(s, a, r, s2, d)
        assert np.abs(q_sa).max() < 100.0
        return {name: float(np.linalg.norm(g[slc] - orc.last_grad[slc]) / np.linalg.norm(orc.last_grad[slc])) for name, slc in blob_slices(A).items()}
    finally:
        P.dqn_destroy(ctx)


CASES = [(16, 0), (32, 0), (64, 1), (128, 0), (131, 0), (256, 1), (512, 0)]
RECORDED = {   # conv1.w conv1.b conv2.w conv2.b conv3.w conv3.b fc1.w fc1.b fc2.w fc2.b
    16: (4.39e-07, 2.86e-07, 3.58e-07, 2.73e-07, 3.09e-07, 2.14e-07, 9.59e-08, 7.31e-08, 5.07e-08, 0),
    32: (6.18e-07, 3.99e-07, 4.63e-07, 4.11e-07, 3.54e-07, 2.84e-07, 1.13e-07, 7.75e-08, 4.81e-08, 0),
    64: (7.61e-07, 4.9e-07, 5.05e-07, 3.98e-07, 4.7e-07, 3.97e-07, 1.8e-07, 1.29e-07, 8.33e-08, 0),
    128: (9.09e-07, 3.51e-07, 4.55e-07, 3.01e-07, 3.86e-07, 2.95e-07, 2e-07, 9.11e-08, 7.48e-08, 0),
    131: (1.01e-06, 4.68e-07, 6.77e-07, 4.07e-07, 5.74e-07, 3.65e-07, 2.85e-07, 1.35e-07, 1.06e-07, 9.94e-08),
    256: (1.36e-06, 5.28e-07, 7.46e-07, 3.82e-07, 5.85e-07, 3.53e-07, 3.21e-07, 1.12e-07, 1.01e-07, 0),
    512: (1.64e-06, 4.21e-07, 8.25e-07, 3.48e-07, 6.7e-07, 3.04e-07, 4.52e-07, 1.14e-07, 9.62e-08, 0),
}


@pytest.mark.parametrize("B,double_dqn", CASES)
def test_f32_gradient_errors(B, double_dqn):
    errs = gradient_errors(B, double_dqn)
    print("B=%d " % B + " ".join("%s %.2e" % kv for kv in errs.items()))
    for (name, err), bound in zip(errs.items(), RECORDED[B]):
        assert err <= SLACK * bound, (name, err, bound)


ONE_SIGN_RECORDED = {
    16: (8.87e-07, 3.29e-05, 2.64e-06, 6.91e-06, 3.45e-06, 3.59e-06, 2.1e-07, 9.43e-08, 5.6e-08, 0),
    32: (3.13e-07, 7.42e-08, 1.41e-07, 5.59e-08, 1.39e-07, 4.77e-08, 1.07e-07, 6.54e-08, 5.45e-08, 0),
    64: (9.34e-07, 1.35e-07, 4.21e-07, 8.43e-08, 3.88e-07, 9.46e-08, 1.75e-07, 1.14e-07, 1.11e-07, 0),
    128: (1.64e-06, 1.94e-07, 8.12e-07, 1.57e-07, 7.14e-07, 2.49e-07, 2.69e-07, 1.43e-07, 8.99e-08, 0),
    131: (2.2e-06, 4.06e-07, 2e-06, 2.47e-07, 1.49e-06, 3.24e-07, 3.45e-07, 1.94e-07, 1.27e-07, 9.94e-08),
    256: (4.5e-06, 1.44e-06, 1.98e-05, 1.39e-06, 2.12e-05, 1.39e-06, 5.66e-07, 1.67e-07, 1.13e-07, 0),
    512: (3.05e-06, 2.22e-07, 1.61e-06, 1.8e-07, 1.21e-06, 1.68e-07, 5.08e-07, 1.25e-07, 1.15e-07, 0),
}


@pytest.mark.parametrize("B,double_dqn", CASES)
def test_f32_gradient_errors_weights_of_one_sign(B, double_dqn):
    errs = gradient_errors(B, double_dqn, one_sign_params)
    print("B=%d " % B + " ".join("%s %.2e" % kv for kv in errs.items()))
    for (name, err), bound in zip(errs.items(), ONE_SIGN_RECORDED[B]):
        assert err <= SLACK * bound, (name, err, bound)


ACT_RECORDED = {36: 2.89e-07, 85: 4.10e-07, 128: 4.67e-07, 200: 3.10e-07}      # states: error of the kernels on the fp32 instruction


def act_error(W):
    A, errs = 6, []
    for seed in range(2900 + W, 2900 + W + 1000 * SEEDS, 1000):
        ctx = P.dqn_create(make_cfg(A, max_batch=1, max_envs=W, precision=P.DQN_PRECISION_FP32, seed=seed), torch.cuda.Stream(), torch.cuda.Stream())
        try:
            theta = synth.init_params(seed, A)
            P.dqn_set_params(ctx, P.DQN_PARAMS_ONLINE, theta)
            P.dqn_set_params(ctx, P.DQN_PARAMS_TARGET, theta)
            states = synth.act_states(seed, 0, W)
            actions = torch.empty(W, dtype=torch.int32, device="cuda")
            q = torch.empty((W, A), dtype=torch.float32, device="cuda")
            P.dqn_act(ctx, dev(states), W, 0.0, 0, 1, actions, q)
            torch.cuda.synchronize()
            want = odqn.forward(odqn.nature_desc(A), theta.astype(np.float64), odqn.scale_states(states))[0]
            errs.append(np.linalg.norm(q.cpu().numpy() - want) / np.linalg.norm(want - theta[blob_slices(A)["fc2.b"]]))
        finally:
            P.dqn_destroy(ctx)
    return float(np.sqrt(np.mean(np.square(errs))))


@pytest.mark.parametrize("W", [36, 85, 128, 200])
def test_f32_act_error(W):
    err = act_error(W)
    print("W=%d %.2e" % (W, err))
    assert err <= SLACK * ACT_RECORDED[W], (err, ACT_RECORDED[W])
