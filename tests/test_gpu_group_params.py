"""Every variant of the fused conv kernels takes each network's own parameters: Q(s, .; theta), Q(s', .; theta^-) and, with Double DQN,
Q(s', .; theta) of one train step against the fp64 oracle, with weights AND biases of theta and theta^- all different (elsewhere the
two start equal or share their biases at the small minibatches).  Sizes, on 256 compute units: the last minibatch in sevenths,
thirds and halves of a sample for two networks (18, 42, 64; bf16 has no halves) and for three (12, 28, 42), the first one after each,
and whole samples whose ranges cross from one network to the next (130 and 86 by one item; 300).
Tolerances as in the act tests: fp32 1e-4, bf16 2e-2 of the largest value; a bias of another network moves Q by its own size."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

import paper_2111_01264_amd as P
from datagen import synth
from oracle import dqn as odqn
from tests.gpu_util import blob_slices, dev, make_cfg


def params(seed, A):
    theta = synth.init_params(seed, A)
    rng = np.random.default_rng(seed + 77)
    for name, slc in blob_slices(A).items():
        if name.startswith("conv") and name.endswith(".b"):
            theta[slc] = rng.uniform(-0.5, 0.5, slc.stop - slc.start).astype(np.float32)
    return theta


@pytest.mark.parametrize("precision,tol", [(P.DQN_PRECISION_FP32, 1e-4), (P.DQN_PRECISION_BF16, 2e-2)])
@pytest.mark.parametrize("B,double_dqn", [(1, 0), (18, 0), (19, 0), (42, 0), (43, 0), (64, 0), (65, 0), (130, 0), (300, 0), (12, 1), (13, 1), (28, 1), (29, 1), (42, 1),
                                          (43, 1), (86, 1), (300, 1)])
def test_q_of_every_network(B, double_dqn, precision, tol):
    A, seed = 6, 3100 + B
    ctx = P.dqn_create(make_cfg(A, max_batch=B, max_envs=1, precision=precision, double_dqn=double_dqn, seed=seed), torch.cuda.Stream(), torch.cuda.Stream())
    try:
        theta, theta_t = params(seed, A), params(seed + 1, A)
        P.dqn_set_params(ctx, P.DQN_PARAMS_ONLINE, theta)
        P.dqn_set_params(ctx, P.DQN_PARAMS_TARGET, theta_t)
        s = synth.block_frames(seed + 10, B * 4).reshape(B, 4, 84, 84)
        s2 = synth.block_frames(seed + 20, B * 4).reshape(B, 4, 84, 84)
        zeros = np.zeros(B, dtype=np.float32)
        P.dqn_train_step(ctx, dev(s), dev(zeros.astype(np.int32)), dev(zeros), dev(s2), dev(zeros), B, None)
        got = P.dqn_get_train_q(ctx, B, A, bool(double_dqn))
        desc = odqn.nature_desc(A)
        for what, q, th, x in (("Q(s; theta)", got[0], theta, s), ("Q(s'; theta^-)", got[1], theta_t, s2), ("Q(s'; theta)", got[2], theta, s2)):
            if q is None or (what == "Q(s'; theta)" and not double_dqn):
                continue
            want = odqn.forward(desc, th.astype(np.float64), odqn.scale_states(x))[0]
            assert np.abs(q - want).max() <= tol * np.abs(want).max(), (what, np.abs(q - want).max(), np.abs(want).max())
    finally:
        P.dqn_destroy(ctx)
