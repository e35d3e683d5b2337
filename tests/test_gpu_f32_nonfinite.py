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


# ---- gradients ------------------------------------------------------------------------------------------------------

def f32(x):
    return x.astype(np.float32).astype(np.float64)


def reference_gradient(theta, state, action, dq):
    """name -> gradient of one sample whose dLoss/dQ[action] is dq, every product formed (a data gradient's filter taps that fall
    outside the output too: as products with zero), every layer's sums rounded to float32."""
    sl = blob_slices(A)

    def tensor(name, shape):
        return theta[sl[name]].astype(np.float64).reshape(shape)

    with np.errstate(all="ignore"):
        _, acts = reference_q(theta, state[None])
        a1, a2, a3 = (x[0] for x in acts)
        w1, w2 = tensor("fc1.w", (512, 3136)), tensor("fc2.w", (A, 512))
        h = np.fmax((f32((a3.reshape(-1) * w1).sum(1)) + theta[sl["fc1.b"]]).astype(np.float32), np.float32(0)).astype(np.float64)
        g = {}
        g["fc2.w"], g["fc2.b"] = np.zeros((A, 512)), np.zeros(A)
        g["fc2.w"][action], g["fc2.b"][action] = dq * h, dq
        dzh = np.where(h > 0, f32(dq * w2[action]), 0.0)
        g["fc1.w"], g["fc1.b"] = dzh[:, None] * a3.reshape(-1)[None], dzh
        dz = np.where(a3 > 0, f32((dzh[:, None] * w1).sum(0)).reshape(64, 7, 7), 0.0)
        x0 = state.astype(np.float64) / 255.0
        for name, shape, stride, x, below in (("conv3", (64, 64, 3, 3), 1, a2, a2), ("conv2", (64, 32, 4, 4), 2, a1, a1), ("conv1", (32, 4, 8, 8), 4, x0, None)):
            k, out = shape[2], dz.shape[1]
            g[name + ".b"] = f32(dz).sum((1, 2))
            gw = np.zeros(shape)
            for p in range(k):
                for q in range(k):
                    win = x[:, p:p + stride * (out - 1) + 1:stride, q:q + stride * (out - 1) + 1:stride]
                    for c in range(shape[1]):
                        gw[:, c, p, q] = (dz * win[None, c]).sum((1, 2))
            g[name + ".w"] = gw
            if below is None:
                break
            w, size = tensor(name + ".w", shape), x.shape[1]
            pad = np.zeros((64, out + 2 * (k // stride - 1), out + 2 * (k // stride - 1)))
            o0 = k // stride - 1
            pad[:, o0:o0 + out, o0:o0 + out] = dz
            dx = np.zeros_like(x)
            n = size // stride
            for py in range(stride):
                for px in range(stride):
                    acc = np.zeros((shape[1], n, n))
                    for p2 in range(k // stride):
                        for q2 in range(k // stride):
                            tap = pad[:, o0 - p2:o0 - p2 + n, o0 - q2:o0 - q2 + n]
                            for o in range(64):
                                acc += w[o, :, stride * p2 + py, stride * q2 + px][:, None, None] * tap[o][None]
                    dx[:, py::stride, px::stride] = acc
            dz = np.where(below > 0, f32(dx), 0.0)
    return {name: v.reshape(-1) for name, v in g.items()}


def gradient_params(kind, seed):
    if kind == "fc2.w=inf aligned":          # dL/d(fc1's output) infinite for the samples with action 0
        theta = params("aligned", seed)
        theta[blob_slices(A)["fc2.w"]][6] = np.inf
    elif kind.startswith("fc1.w=inf"):       # one element of dL/d(act3) infinite: channel 62 of the last pixel
        theta = params("aligned" if "aligned" in kind else "", seed)
        theta[blob_slices(A)["fc1.w"]][3136 * 8 + 62 * 49 + 48] = np.inf
    else:
        theta = params(kind, seed)
    return theta


GRADIENT_KINDS = ["fc2.w=inf aligned", "fc1.w=inf", "fc1.w=inf aligned", "conv1.b=inf aligned", "conv2.b=inf aligned", "conv3.b=inf aligned",
                  "conv2.w=-inf aligned", "conv3.w=nan", "beyond bf16"]


@pytest.mark.parametrize("kind", GRADIENT_KINDS)
@pytest.mark.parametrize("B,sampled", [(1, False), (5, False), (64, False), (130, False), (300, False), (101, True)])
def test_gradient_with_nonfinite_values(B, sampled, kind):
    seed = 4400
    cfg = make_cfg(A, max_batch=B, max_envs=1, precision=P.DQN_PRECISION_FP32, seed=seed)
    cfg.huber_delta = 1.0
    st = torch.cuda.Stream()
    ctx = P.dqn_create(cfg, st, st)
    rb = None
    try:
        theta = gradient_params(kind, seed)
        P.dqn_set_params(ctx, P.DQN_PARAMS_ONLINE, theta)
        P.dqn_set_params(ctx, P.DQN_PARAMS_TARGET, synth.init_params(seed, A))
        few, few_a = np.maximum(synth.act_states(seed, 0, 3), 1), np.array([0, 1, 2], dtype=np.int32)
        if sampled:       # one lane of six frames, none of them terminal: two transitions
            n = 6
            rb = P.replay_create(n, 1, n, seed, st, st)
            frames = few.reshape(12, 84, 84)[:n]
            acts = np.array([0, 0, 0, 0, 1, 0], dtype=np.int32)
            P.replay_push(rb, 0, dev(frames), dev(acts), dev(np.full(n, -1000.0, dtype=np.float32)), dev(np.zeros(n, dtype=np.uint8)), n)
            P.replay_flush(rb, 1)
            s, a, r = (torch.empty(shape, dtype=t, device="cuda") for shape, t in (((B, 4, 84, 84), torch.uint8), (B, torch.int32), (B, torch.float32)))
            s2, d, idx = torch.empty_like(s), torch.empty_like(r), torch.empty(B, dtype=torch.int64, device="cuda")
            P.replay_sample_gather(rb, B, 0, None, s, s2, a, r, d, idx)
            torch.cuda.synchronize()
            pick = idx.cpu().numpy() - 3
            few, few_a = np.stack([frames[0:4], frames[1:5]]), acts[3:5]
            P.dqn_train_step_sampled(ctx, rb, B, 0, 0, None)
        else:
            pick = np.arange(B) % 3
            P.dqn_train_step(ctx, dev(few[pick]), dev(few_a[pick]), dev(np.full(B, -1000.0, dtype=np.float32)), dev(few[pick]), dev(np.ones(B, dtype=np.float32)),
                             B, None)
        torch.cuda.synchronize()
        g = P.dqn_get_params(ctx, P.DQN_PARAMS_GRAD)
        # a finite or positively infinite Q is above every target here: dLoss/dQ is 1/B; a negative infinity gives -1/B, a NaN too (fmax, then fmin)
        q, _ = reference_q(theta, few)
        dq = np.where(q[np.arange(len(few)), few_a] > -1e30, 1.0, -1.0).astype(np.float32) / np.float32(B)
        refs = [reference_gradient(theta, few[k], few_a[k], np.float64(dq[k])) for k in range(len(few))]
        with np.errstate(all="ignore"):
            for name, slc in blob_slices(A).items():
                want = sum(refs[k][name] * count for k, count in enumerate(np.bincount(pick, minlength=len(few))) if count)
                same_values(g[slc], want, "%s %s" % (kind, name))
    finally:
        if rb is not None:
            P.replay_destroy(rb)
        P.dqn_destroy(ctx)
