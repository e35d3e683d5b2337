"""Act parity where the act step's kernels change shape: the last and first numbers of states run in sevenths, thirds, halves of a
sample and whole (36/37, 85/86, 128/129 on 256 compute units), and the first whose fc1 workgroups are ordered by XCD (129; a ragged
last row tile at 161).  Q rows against the fp64 oracle with the tolerances of the act tests: fp32 1e-4, bf16 2e-2 of the largest value."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

import paper_2111_01264_amd as P
from datagen import synth
from oracle import dqn as odqn
from tests.gpu_util import dev, make_cfg


@pytest.mark.parametrize("precision,tol", [(P.DQN_PRECISION_FP32, 1e-4), (P.DQN_PRECISION_BF16, 2e-2)])
@pytest.mark.parametrize("W", [36, 37, 85, 86, 128, 129, 161])
def test_act_q_rows(W, precision, tol):
    A, seed = 6, 900 + W
    ctx = P.dqn_create(make_cfg(A, max_batch=1, max_envs=W, precision=precision, seed=seed), torch.cuda.Stream(), torch.cuda.Stream())
    try:
        theta = synth.init_params(seed, A)
        P.dqn_set_params(ctx, P.DQN_PARAMS_ONLINE, theta)
        P.dqn_set_params(ctx, P.DQN_PARAMS_TARGET, theta)
        states = synth.act_states(seed, 0, W)
        actions = torch.empty(W, dtype=torch.int32, device="cuda")
        q = torch.empty((W, A), dtype=torch.float32, device="cuda")
        P.dqn_act(ctx, dev(states), W, 0.0, 0, 1, actions, q)
        torch.cuda.synchronize()
        _, want = odqn.OracleDQN(A, theta, seed=seed).act(states, 0.0, 0)
        got = q.cpu().numpy()
        assert np.abs(got - want).max() <= tol * np.abs(want).max()
        gap = np.sort(want, axis=1)
        clear = gap[:, -1] - gap[:, -2] > 2 * tol * np.abs(want).max()
        assert np.array_equal(actions.cpu().numpy()[clear], want.argmax(1)[clear])
    finally:
        P.dqn_destroy(ctx)
