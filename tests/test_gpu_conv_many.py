"""The bf16 conv tower's variants agree bit for bit: Q rows of W states at once -- thirds and halves of a sample (up to 85 and 128 states on 256
compute units), whole samples, and above that the persistent workgroups of half the size (one item each up to 512, then unequal
shares) -- against the rows of the same states in rounds of whole samples (fc1's kernel is the same from 33 states on, so every row is
the same sum).  With the append riding along where the persistent kernel acts."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

import paper_2111_01264_amd as P
from datagen import synth
from tests.gpu_util import dev, make_cfg

A, SEED, N = 6, 411, 1030


@pytest.fixture(scope="module")
def act():
    streams = torch.cuda.Stream(), torch.cuda.Stream()
    ctx = P.dqn_create(make_cfg(A, max_batch=1, max_envs=1024, precision=P.DQN_PRECISION_BF16, seed=SEED), *streams)
    rb = P.replay_create(64, 2, 32, SEED, *streams)
    theta = synth.init_params(SEED, A)
    P.dqn_set_params(ctx, P.DQN_PARAMS_ONLINE, theta)
    P.dqn_set_params(ctx, P.DQN_PARAMS_TARGET, theta)
    states = dev(synth.block_frames(SEED, N * 4).reshape(N, 4, 84, 84))
    push = [dev(v) for v in (synth.frames(SEED, synth.STREAM_REPLAY, np.arange(2, dtype=np.uint64)), np.zeros(2, np.int32),
                             np.zeros(2, np.float32), np.zeros(2, np.uint8))]

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
    yield rows, whole
    P.replay_destroy(rb)
    P.dqn_destroy(ctx)


@pytest.mark.parametrize("W,ride", [(85, False), (86, False), (127, False), (128, True), (256, False), (257, False), (300, True), (511, False),
                                    (512, False), (513, False), (770, False), (1024, False)])
def test_act_rows_do_not_depend_on_the_variant(act, W, ride):
    rows, whole = act
    first = N - W if W % 2 else 0
    assert np.array_equal(rows(first, first + W, ride), whole[first:first + W])
