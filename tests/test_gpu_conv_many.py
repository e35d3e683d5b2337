"""The bf16 conv tower's variants agree bit for bit: Q rows of W states at once -- thirds and halves of a sample (up to 85 and 128 states on 256
compute units), whole samples, and above that the persistent workgroups of half the size (one item each up to 512, then unequal
shares) -- against the rows of the same states in rounds of whole samples (fc1's kernel is the same from 33 states on, so every row is
the same sum).  The append that rides along with the persistent kernel (above 256 states) leaves in the replay memory what
replay_push_step does."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

import paper_2111_01264_amd as P
from datagen import synth
from tests.gpu_util import dev, make_cfg

A, SEED, N = 6, 411, 1030


def outcomes(step):
    """Frames, actions, rewards and terminals of the two lanes at `step`: no two alike, none zero throughout."""
    return [dev(v) for v in (synth.frames(SEED, synth.STREAM_REPLAY, np.arange(2 * step, 2 * step + 2, dtype=np.uint64)),
                             np.array([1 + step % 5, 5 - step % 5], np.int32), np.array([step + 0.5, -step - 0.25], np.float32),
                             np.array([step == 6, step == 8], np.uint8))]


@pytest.fixture(scope="module")
def act():
    streams = torch.cuda.Stream(), torch.cuda.Stream()
    ctx = P.dqn_create(make_cfg(A, max_batch=1, max_envs=1024, precision=P.DQN_PRECISION_BF16, seed=SEED), *streams)
    rb = P.replay_create(64, 2, 32, SEED, *streams)
    theta = synth.init_params(SEED, A)
    P.dqn_set_params(ctx, P.DQN_PARAMS_ONLINE, theta)
    P.dqn_set_params(ctx, P.DQN_PARAMS_TARGET, theta)
    states = dev(synth.block_frames(SEED, N * 4).reshape(N, 4, 84, 84))
    push = outcomes(0)

    def rows(lo, hi, ride=False):
        W = hi - lo
        actions = torch.empty(W, dtype=torch.int32, device="cuda")
        q = torch.full((W, A), np.nan, dtype=torch.float32, device="cuda")
        if ride:
            P.dqn_act_push_step(ctx, rb, *push, states[lo:hi], W, 0.0, 0, 1, actions, q)
        else:
            P.dqn_act(ctx, states[lo:hi], W, 0.0, 0, 1, actions, q)
        torch.cuda.synchronize()
        return q.cpu().numpy()

    whole = np.concatenate([rows(lo, min(lo + 200, N - 130)) for lo in range(0, N - 130, 200)] + [rows(N - 130, N)])
    yield rows, whole, ctx, states, streams
    P.replay_destroy(rb)
    P.dqn_destroy(ctx)


@pytest.mark.parametrize("W,ride", [(85, False), (86, False), (127, False), (128, True), (256, False), (257, False), (300, True), (511, False),
                                    (512, False), (513, False), (770, False), (1024, False)])
def test_act_rows_do_not_depend_on_the_variant(act, W, ride):
    rows, whole = act[:2]
    first = N - W if W % 2 else 0
    assert np.array_equal(rows(first, first + W, ride), whole[first:first + W])


@pytest.mark.parametrize("W", [128, 257, 300, 1024])
def test_the_append_that_rides_along(act, W):
    _, _, ctx, states, streams = act
    steps, seen = 12, []
    actions = torch.empty(W, dtype=torch.int32, device="cuda")
    q = torch.empty((W, A), dtype=torch.float32, device="cuda")
    for ride in (False, True):
        rb = P.replay_create(64, 2, 32, SEED, *streams)
        try:
            for step in range(steps):
                if ride:
                    P.dqn_act_push_step(ctx, rb, *outcomes(step), states[:W], W, 0.0, step, 1, actions, q)
                else:
                    P.replay_push_step(rb, *outcomes(step))
            torch.cuda.synchronize()
            P.replay_flush(rb, 1)
            n = P.replay_num_valid(rb)
            assert n == 2 * (steps - 4)
            got = [torch.full((n, 4, 84, 84), 255, dtype=torch.uint8, device="cuda"), torch.full((n, 4, 84, 84), 255, dtype=torch.uint8, device="cuda"),
                   torch.full((n,), -7, dtype=torch.int32, device="cuda"), torch.full((n,), np.nan, device="cuda"), torch.full((n,), np.nan, device="cuda")]
            torch.cuda.synchronize()
            idx = dev(np.array([lane * 32 + 3 + k for lane in range(2) for k in range(steps - 4)], np.int64))
            P.replay_sample_gather(rb, n, 0, idx, *got, None)
            torch.cuda.synchronize()
            seen.append([x.cpu().numpy() for x in got])
        finally:
            torch.cuda.synchronize()
            P.replay_destroy(rb)
    s, s2, a, r, d = seen[1]
    assert all(np.array_equal(x, y) for x, y in zip(*seen))
    assert a.min() >= 1 and len(set(r.tolist())) == len(r) and d.sum() == 2       # what was pushed, not the marker of an invalid row
    newest = synth.frames(SEED, synth.STREAM_REPLAY, np.arange(2 * 3, 2 * (steps - 1), 2, dtype=np.uint64))
    assert np.array_equal(s[:steps - 4, 3], newest)
