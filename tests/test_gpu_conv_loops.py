"""The persistent conv kernels beyond one item per workgroup.  On 256 compute units the bf16 forward runs two or more (network, sample)
items per workgroup from 513 items on, the bf16 data gradients two or more samples from minibatch 513 on, and for some minibatches a
workgroup's items belong to two networks.

  * The gradient of a minibatch of 2 b samples is the mean of the gradients of its halves.  1 / (2 b) is half of 1 / b in fp32 and every later
    operand scales with it exactly, so all data gradients have the same bits but for their exponents, and what differs is the order in which
    the weight gradients' fp32 sums are taken.  Inputs on which no ReLU flips, one action and TD errors of one sign, so that a weight's
    terms are of one sign over the samples and nothing cancels: a sum of n steps is then off by at most n * 2^-23 of itself (the matrix instruction
    cuts off what lies below the last bit of the larger term), n is at most 16 items x 13 steps + 24 slice sums (conv1 at 1024): 2.8e-5.  Asserted:
    3e-5 of a tensor's largest element (seen: 2e-6), where a sample that is left out or taken twice is 6e-4 of it or more.
  * Q rows of a train step are, bit for bit, those of dqn_act on the same states and networks in rounds of 128 (halves of a sample on eight
    wavefronts, no loop; fc1's kernel is the same from 33 states on).
  * dqn_train_step_sampled (frames by descriptor) is, bit for bit, replay_sample_gather + dqn_train_step at such sizes."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

import paper_2111_01264_amd as P
from datagen import synth
from tests.gpu_util import blob_slices, dev, fill_replay_from_host, make_cfg

A = 6


def shares(items):
    """(first, end) of every workgroup's items: two workgroups per compute unit, as equal as can be."""
    grid = 2 * torch.cuda.get_device_properties(0).multi_processor_count
    base, more = divmod(items, min(items, grid))
    ends = np.cumsum([base + (j < more) for j in range(min(items, grid))])
    return [(e - base - (j < more), e) for j, e in enumerate(ends)]


def minibatch(seed, B, rewards):
    rng = np.random.default_rng(seed)
    s = synth.block_frames(seed + 10, B * 4).reshape(B, 4, 84, 84)
    s2 = synth.block_frames(seed + 20, B * 4).reshape(B, 4, 84, 84)
    return [s, rng.integers(0, A, size=B).astype(np.int32), rewards[rng.integers(0, len(rewards), size=B)].astype(np.float32), s2,
            (rng.random(B) < 0.2).astype(np.float32)]


@pytest.mark.parametrize("B,precision", [(514, P.DQN_PRECISION_BF16), (770, P.DQN_PRECISION_BF16), (1024, P.DQN_PRECISION_BF16),
                                         (770, P.DQN_PRECISION_FP32)])
def test_gradient_of_a_minibatch_is_the_mean_of_its_halves(B, precision):
    assert max(e - f for f, e in shares(B)) > 1
    seed = 5200 + B
    cfg = make_cfg(A, max_batch=B, max_envs=1, precision=precision, seed=seed)
    cfg.huber_delta = 10.0
    ctx = P.dqn_create(cfg, torch.cuda.Stream(), torch.cuda.Stream())
    try:
        theta = synth.margin_params(seed, A, True)
        P.dqn_set_params(ctx, P.DQN_PARAMS_TARGET, synth.margin_params(seed + 1, A, True))
        batch = minibatch(seed, B, np.array([-2.0, -3.0, -4.0]))     # |Q| < 0.4 (margin_params): every TD error is 1.2 or more
        batch[1][:] = 2                                              # (fc2's weights have both signs)
        loss = torch.zeros(1, dtype=torch.float32, device="cuda")

        def step(lo, hi):
            P.dqn_set_params(ctx, P.DQN_PARAMS_ONLINE, theta)
            s, a, r, s2, d = (dev(v[lo:hi]) for v in batch)
            P.dqn_train_step(ctx, s, a, r, s2, d, hi - lo, loss)
            torch.cuda.synchronize()
            q = P.dqn_get_train_q(ctx, hi - lo, A, False)
            return P.dqn_get_params(ctx, P.DQN_PARAMS_GRAD).astype(np.float64), float(loss.item()), q[0].copy(), q[1].copy()

        g, l, q, qt = step(0, B)
        (g0, l0, q0, qt0), (g1, l1, q1, qt1) = step(0, B // 2), step(B // 2, B)
        assert np.abs(q).max() < 0.4 and np.abs(qt).max() < 0.4
        assert np.array_equal(q, np.concatenate([q0, q1])) and np.array_equal(qt, np.concatenate([qt0, qt1]))
        assert abs(l - (l0 + l1) / 2) <= 1e-5 * abs(l)
        errs = {}
        for name, slc in blob_slices(A).items():
            assert np.abs(g[slc]).max() > 0, name
            errs[name] = np.abs(g[slc] - (g0[slc] + g1[slc]) / 2).max() / np.abs(g[slc]).max()
        print("B=%d against the mean of its halves: %s" % (B, " ".join("%s %.1e" % kv for kv in errs.items())))
        for name, e in errs.items():
            assert e <= 3e-5, (name, e)
    finally:
        P.dqn_destroy(ctx)


CHANGES = [(343, 0), (511, 0), (205, 1), (512, 1), (1023, 1)]      # (minibatch, Double DQN): a workgroup's items span two networks


@pytest.mark.parametrize("B,double_dqn", CHANGES)
def test_q_rows_where_a_workgroup_changes_its_network(B, double_dqn):
    nets = 3 if double_dqn else 2
    changes = {e // B for f, e in shares(nets * B) if f // B != (e - 1) // B}
    assert changes, "no workgroup changes its network"
    seed = 6100 + B
    ctx = P.dqn_create(make_cfg(A, max_batch=B, max_envs=128, precision=P.DQN_PRECISION_BF16, double_dqn=double_dqn, seed=seed), torch.cuda.Stream(),
                       torch.cuda.Stream())
    try:
        P.dqn_set_params(ctx, P.DQN_PARAMS_ONLINE, synth.init_params(seed, A))
        P.dqn_set_params(ctx, P.DQN_PARAMS_TARGET, synth.init_params(seed + 1, A))
        s, a, r, s2, d = (dev(v) for v in minibatch(seed, B, np.array([-1.0, 0.0, 1.0])))
        actions = torch.empty(128, dtype=torch.int32, device="cuda")
        q = torch.empty((128, A), dtype=torch.float32, device="cuda")

        def acted(states, use_target):     # in rounds of 128, the last one moved back (33 rows or more, whatever B is)
            rows = np.empty((B, A), np.float32)
            for lo in range(0, B, 128):
                lo = min(lo, B - 128)
                P.dqn_act(ctx, states[lo:lo + 128], 128, 0.0, 0, use_target, actions, q)
                torch.cuda.synchronize()
                rows[lo:lo + 128] = q.cpu().numpy()
            return rows

        want = [acted(s, 0), acted(s2, 1)] + ([acted(s2, 0)] if double_dqn else [])
        P.dqn_train_step(ctx, s, a, r, s2, d, B, torch.zeros(1, dtype=torch.float32, device="cuda"))
        torch.cuda.synchronize()
        got = P.dqn_get_train_q(ctx, B, A, bool(double_dqn))
        for net, w in enumerate(want):
            assert np.array_equal(got[net], w), ("network", net, np.flatnonzero((got[net] != w).any(1))[:8])
    finally:
        P.dqn_destroy(ctx)


@pytest.mark.parametrize("B,double_dqn", [(205, 1), (343, 0), (770, 0), (1024, 1)])
def test_minibatch_by_descriptor_equals_the_assembled_one(B, double_dqn):
    seed, lanes, per_lane = 7700 + B, 4, 400
    results = []
    for sampled in (False, True):
        st = torch.cuda.Stream()
        ctx = P.dqn_create(make_cfg(A, max_batch=B, max_envs=1, precision=P.DQN_PRECISION_BF16, double_dqn=double_dqn, seed=seed), st, st)
        rb = P.replay_create(lanes * per_lane, lanes, per_lane, seed, st, st)
        try:
            P.dqn_set_params(ctx, P.DQN_PARAMS_ONLINE, synth.init_params(seed, A))
            P.dqn_set_params(ctx, P.DQN_PARAMS_TARGET, synth.init_params(seed + 1, A))
            fill_replay_from_host(rb, seed, lanes, per_lane, A, chunk=per_lane, p_neg=0.3, p_pos=0.3, p_term=0.03)
            s = torch.empty((B, 4, 84, 84), dtype=torch.uint8, device="cuda")
            s2 = torch.empty_like(s)
            a = torch.empty(B, dtype=torch.int32, device="cuda")
            r, d = torch.empty(B, dtype=torch.float32, device="cuda"), torch.empty(B, dtype=torch.float32, device="cuda")
            loss = torch.zeros(1, dtype=torch.float32, device="cuda")
            for step in range(2):
                if sampled:
                    P.dqn_train_step_sampled(ctx, rb, B, step, step == 0, loss)
                else:
                    P.replay_sample_gather(rb, B, step, None, s, s2, a, r, d, None)
                    P.dqn_train_step(ctx, s, a, r, s2, d, B, loss)
                torch.cuda.synchronize()
            results.append((float(loss.item()), P.dqn_get_params(ctx, P.DQN_PARAMS_ONLINE).copy(), P.dqn_get_params(ctx, P.DQN_PARAMS_GRAD).copy()))
        finally:
            torch.cuda.synchronize()
            P.replay_destroy(rb)
            P.dqn_destroy(ctx)
    (l0, t0, g0), (l1, t1, g1) = results
    assert l0 == l1 and np.array_equal(t0, t1) and np.array_equal(g0, g1)
    assert np.abs(g0).max() > 0
