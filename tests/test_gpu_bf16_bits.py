"""The bits of bf16 training: what a train step computes does not depend on how its reductions are spread over lanes and workgroups,
so a stretch of steps gives the recorded parameters, gradient and loss bit for bit.  tests/golden/bf16_train_sha256.txt was recorded with
the optimiser kernel that adds the conv layers' slices with eight lanes per weight (eight sums, each over every eighth slice, and a tree).
Sizes: one, some and all of conv2's and conv3's slices; fifths (up to 51), halves (70, 256) and whole samples (512) in the data gradients;
thirds, halves, whole samples and the persistent workgroups in the forward.  (dqn_train_step: no descriptors here.)"""
import hashlib
import os

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

import paper_2111_01264_amd as P
from datagen import synth
from tests.gpu_util import dev, make_cfg

GOLDEN = os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden", "bf16_train_sha256.txt")
CASES = [(1, 0), (5, 1), (9, 0), (32, 0), (45, 0), (70, 1), (256, 1), (512, 0)]


def digest(B, double_dqn, steps=3):
    """sha256 over the parameters, the last gradient and the last loss of `steps` train steps on seeded inputs."""
    A, seed = 6, 7300 + B
    ctx = P.dqn_create(make_cfg(A, max_batch=B, max_envs=1, precision=P.DQN_PRECISION_BF16, double_dqn=double_dqn, seed=seed),
                       torch.cuda.Stream(), torch.cuda.Stream())
    try:
        P.dqn_set_params(ctx, P.DQN_PARAMS_ONLINE, synth.init_params(seed, A))
        P.dqn_set_params(ctx, P.DQN_PARAMS_TARGET, synth.init_params(seed + 1, A))
        rng = np.random.default_rng(seed)
        loss = torch.zeros(1, dtype=torch.float32, device="cuda")
        for step in range(steps):
            s = synth.block_frames(seed + 10 + step, B * 4).reshape(B, 4, 84, 84)
            s2 = synth.block_frames(seed + 20 + step, B * 4).reshape(B, 4, 84, 84)
            a = rng.integers(0, A, size=B).astype(np.int32)
            r = rng.integers(-1, 2, size=B).astype(np.float32)
            d = (rng.random(B) < 0.2).astype(np.float32)
            P.dqn_train_step(ctx, dev(s), dev(a), dev(r), dev(s2), dev(d), B, loss)
            torch.cuda.synchronize()
        h = hashlib.sha256()
        for part in (P.dqn_get_params(ctx, P.DQN_PARAMS_ONLINE), P.dqn_get_params(ctx, P.DQN_PARAMS_GRAD), loss.cpu().numpy()):
            h.update(np.ascontiguousarray(part, dtype=np.float32).tobytes())
        return h.hexdigest()
    finally:
        P.dqn_destroy(ctx)


@pytest.mark.parametrize("B,double_dqn", CASES)
def test_bf16_train_bits(B, double_dqn):
    with open(GOLDEN) as f:
        want = dict(line.split() for line in f if line.strip() and not line.startswith("#"))
    assert digest(B, double_dqn) == want["b%d_double%d" % (B, double_dqn)]
