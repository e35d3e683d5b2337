"""dqn_set_params / dqn_get_params: what goes in comes out, element for element, for every blob that can be set and every remainder of the
blob's length over the sixteen-byte vectors and the pieces in which it leaves the device."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

import paper_2111_01264_amd as P
from tests.gpu_util import make_cfg


@pytest.mark.parametrize("precision", [P.DQN_PRECISION_FP32, P.DQN_PRECISION_BF16])
@pytest.mark.parametrize("A", [1, 2, 3, 4, 18, 31, 32])
def test_round_trip(A, precision):
    ctx = P.dqn_create(make_cfg(A, max_batch=1, max_envs=1, precision=precision), torch.cuda.Stream(), torch.cuda.Stream())
    try:
        rng = np.random.default_rng(A)
        n = P.dqn_num_params(ctx)
        blobs = {w: rng.standard_normal(n).astype(np.float32) for w in (P.DQN_PARAMS_ONLINE, P.DQN_PARAMS_TARGET, P.DQN_PARAMS_RMS_V, P.DQN_PARAMS_RMS_M)}
        for w, v in blobs.items():
            P.dqn_set_params(ctx, w, v)
        for w, v in blobs.items():
            assert np.array_equal(P.dqn_get_params(ctx, w), v)
    finally:
        P.dqn_destroy(ctx)
