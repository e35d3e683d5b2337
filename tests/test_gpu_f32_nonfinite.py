"""Full precision with infinities, NaN and values at the end of the fp32 range: the act step shows them as fp32 arithmetic does.

The conv kernels split fp32 values into bf16 parts, which infinities, NaN and values above the largest bf16 (3.39e38) do not have; what
such a value leads to must still be what a network evaluated in fp32 gives: a positive infinity passes the ReLUs and shows in Q, a NaN
becomes 0 in the next ReLU (fmax).  The reference evaluates layer by layer in float64 and rounds every layer's sums to float32:
which sums are infinite or NaN does not depend on the order of the additions here (infinite operands, or overflow among terms of
one sign).  Finite Q values are compared to 1e-4 of the row's largest finite one, as elsewhere.
Sizes: the smallest number of states of every variant of the conv kernel (sevenths, thirds, halves, whole samples, several per workgroup)."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

import paper_2111_01264_amd as P
from datagen import synth
from tests.gpu_util import blob_slices, dev, make_cfg

A = 4


def reference_q(theta, states):
    """Q rows and the activations below them, every layer's result rounded to float32."""
    sl, x = blob_slices(A), states.astype(np.float64)
    with np.errstate(all="ignore"):
        acts = []
        for (name, shape, _), stride in zip(synth.layer_shapes(A)[:3], (4, 2, 1)):
            w = theta[sl[name + ".w"]].astype(np.float64).reshape(shape)
            b = theta[sl[name + ".b"]].astype(np.float64)
            k, out = shape[2], (x.shape[2] - shape[2]) // stride + 1
            y = np.zeros((len(x), shape[0], out, out))
            for p in range(k):
                for q in range(k):
                    win = x[:, :, p:p + stride * (out - 1) + 1:stride, q:q + stride * (out - 1) + 1:stride]
                    for c in range(shape[1]):
                        y += w[None, :, c, p, q, None, None] * win[:, None, c]
            y = y.astype(np.float32).astype(np.float64)
            if name == "conv1":
                y = y / 255.0
            x = np.fmax((y + b[None, :, None, None]).astype(np.float32), np.float32(0)).astype(np.float64)
            acts.append(x)
        h = x.reshape(len(x), -1)

        def dense(name, h):   # row by row of the weights: a product of an infinity with a zero must be formed
            w = theta[sl[name + ".w"]].astype(np.float64).reshape(-1, h.shape[1])
            y = np.stack([(h * wr).sum(1) for wr in w], axis=1).astype(np.float32)
            return (y + theta[sl[name + ".b"]]).astype(np.float32)

        return dense("fc2", np.fmax(dense("fc1", h), np.float32(0)).astype(np.float64)), acts


def params(kind, seed):
    theta = synth.init_params(seed, A)
    sl = blob_slices(A)

    def t(name):
        return theta[sl[name]]

    kind, aligned = kind.replace(" aligned", ""), "aligned" in kind
    if aligned:      # one sign per output channel: an infinity stays one instead of meeting another of the opposite sign
        for name, n in (("conv2.w", 64), ("conv3.w", 64), ("fc1.w", 512), ("fc2.w", A)):
            w = t(name).reshape(n, -1)
            w[:] = np.abs(w) * np.where(np.arange(n) % 2, np.float32(-1), np.float32(1))[:, None]
    if kind == "conv1.b=inf":
        t("conv1.b")[3] = np.inf
    elif kind == "conv2.b=inf":
        t("conv2.b")[5] = np.inf
    elif kind == "conv3.b=inf":
        t("conv3.b")[7] = np.inf
    elif kind == "conv1.w=inf":
        t("conv1.w")[256 * 9 + 17] = np.inf
    elif kind == "conv2.w=-inf":
        t("conv2.w")[512 * 11 + 100] = -np.inf
    elif kind == "conv3.w=nan":
        t("conv3.w")[576 * 20 + 33] = np.nan
    elif kind == "beyond bf16":       # finite all the way: weights between the largest bf16 and the largest fp32 on small activations
        t("conv1.w")[:] *= np.float32(1e-18)
        t("conv1.b")[:] *= np.float32(1e-18)
        w = t("conv2.w")
        w[:] = np.sign(w) * np.float32(3.399e38) * np.float32(1e-20)
        w[::97] *= np.float32(1e20)
        t("conv3.w")[:] *= np.float32(1e-19)
        t("conv2.b")[:] = 0
    elif kind == "overflow":          # bright states overflow in conv2, black ones do not
        t("conv1.w")[:] = np.abs(t("conv1.w")) * np.float32(1e20)
        t("conv1.b")[:] = np.abs(t("conv1.b"))
        w = t("conv2.w").reshape(64, -1)
        w[::2] = np.abs(w[::2]) * np.float32(1e20)
        w[1::2] = -np.abs(w[1::2])
        w3 = t("conv3.w").reshape(64, 64, 9)
        w3[:] = np.abs(w3)
        w3[1::2] *= -1
        for name in ("fc1.w", "fc2.w"):
            t(name)[:] = np.abs(t(name))
    return theta


KINDS = ["conv1.b=inf", "conv1.b=inf aligned", "conv2.b=inf", "conv2.b=inf aligned", "conv3.b=inf aligned", "conv1.w=inf", "conv1.w=inf aligned",
         "conv2.w=-inf", "conv2.w=-inf aligned", "conv3.w=nan", "beyond bf16", "overflow"]


def same_values(got, want, what):
    assert np.array_equal(np.isnan(got), np.isnan(want)), (what, "NaN", got, want)
    inf = np.isinf(want)
    assert np.array_equal(np.isinf(got), inf) and np.array_equal(got[inf], want[inf]), (what, "infinities", got, want)
    fin = np.isfinite(want)
    if fin.any():
        assert np.abs(got[fin].astype(np.float64) - want[fin]).max() <= 1e-4 * max(np.abs(want[fin].astype(np.float64)).max(), 1e-30), (what, got, want)


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("W", [1, 37, 86, 129, 300])
def test_act_with_nonfinite_values(W, kind):
    seed = 4400
    ctx = P.dqn_create(make_cfg(A, max_batch=1, max_envs=W, precision=P.DQN_PRECISION_FP32, seed=seed), torch.cuda.Stream(), torch.cuda.Stream())
    try:
        theta = params(kind, seed)
        P.dqn_set_params(ctx, P.DQN_PARAMS_ONLINE, theta)
        P.dqn_set_params(ctx, P.DQN_PARAMS_TARGET, theta)
        few = np.maximum(synth.act_states(seed, 0, 3), 1)      # no zero byte: which products of an infinity are NaN would hang on pixels otherwise
        few[1] = 0                                             # and one black state
        want3, _ = reference_q(theta, few)
        pick = np.arange(W) % 3
        actions = torch.empty(W, dtype=torch.int32, device="cuda")
        q = torch.empty((W, A), dtype=torch.float32, device="cuda")
        P.dqn_act(ctx, dev(few[pick]), W, 0.0, 0, 1, actions, q)
        torch.cuda.synchronize()
        same_values(q.cpu().numpy(), want3[pick], kind)
    finally:
        P.dqn_destroy(ctx)
