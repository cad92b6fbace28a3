"""GPU parity of score_losses / local_step for the MLP workload against the oracle."""
import numpy as np
import pytest

import oracle
import synth
from gpu_helpers import Harness, assert_losses_close, assert_tensors_close

pytestmark = pytest.mark.gpu
CFG = synth.workload("mlp")


@pytest.fixture(scope="module")
def h():
    import torch
    import paper_2508_08540_amd as bls
    ctx = bls.Context(0)
    yield Harness(torch, bls, ctx, bls.Model.mlp(), oracle.MLP())
    ctx.close()


@pytest.fixture(scope="module")
def data():
    x, y = synth.image_pool(CFG["id"], CFG["pool"], CFG["classes"])
    return synth.mlp_init(CFG["id"]), x, y


def _zeros(p):
    return {k: np.zeros_like(v) for k, v in p.items()}


def test_scores_match_oracle(h, data):
    p, x, y = data
    ref = oracle.score_losses(h.oracle_model, p, {}, x, y)
    assert_losses_close(h.score(p, {}, x, y), ref)
    assert_losses_close(h.score(p, {}, x[:1], y[:1]), ref[:1])
    assert h.score(p, {}, x[:0], y[:0]).size == 0          # empty pool is a no-op


def test_zero_head_scores_are_log_classes_and_select_first_k(h, data):
    p, x, y = data
    p = dict(p)
    p["fc2.weight"] = np.zeros_like(p["fc2.weight"])
    p["fc2.bias"] = np.zeros_like(p["fc2.bias"])
    got = h.score(p, {}, x, y)
    np.testing.assert_allclose(got, np.log(10.0), rtol=1e-6)


def test_gradients_match_oracle(h, data):
    # lr = 0 with a zero momentum vector leaves the gradient of the batch-mean loss in the momentum buffer
    p, x, y = data
    sel = oracle.topk_by_loss(oracle.score_losses(h.oracle_model, p, {}, x, y).astype(np.float32), CFG["k"])
    ids = sel[:CFG["batch"]]
    losses, grads, _ = oracle.loss_and_grads(h.oracle_model, p, {}, x[ids], y[ids])
    newp, _, mom, sl = h.local_step(p, {}, _zeros(p), x, y, sel, CFG["batch"], 1, lr=0.0, mu=0.9)
    assert_losses_close(sl[0], losses)
    assert_tensors_close(mom, grads, 1e-4, "gradients")
    for k in p:
        np.testing.assert_array_equal(newp[k], p[k].astype(np.float64))


def test_full_workload_steps(h, data):
    p, x, y = data
    sel = oracle.topk_by_loss(oracle.score_losses(h.oracle_model, p, {}, x, y).astype(np.float32), CFG["k"])
    args = dict(batch=CFG["batch"], tau=CFG["tau"], lr=CFG["lr"])
    rp, _, rm, rl = oracle.local_step(h.oracle_model, p, {}, _zeros(p), x, y, sel, momentum=0.0, **args)
    gp, _, gm, gl = h.local_step(p, {}, _zeros(p), x, y, sel, mu=0.0, **args)
    assert_losses_close(gl, rl, rtol=2e-4)
    # compare the movement of the parameters, not the parameters (which barely change)
    delta = lambda a: {k: a[k] - p[k].astype(np.float64) for k in p}
    assert_tensors_close(delta(gp), delta(rp), 3e-4, "parameter change after tau steps")


def test_wrap_momentum_weight_decay(h, data):
    p, x, y = data
    sel = np.array([7, 200, 9, 41, 11], dtype=np.int32)
    mom0 = {k: 0.01 * synth.normal(5, i, v.size).reshape(v.shape) for i, (k, v) in enumerate(p.items())}
    args = dict(batch=3, tau=4, lr=0.05)
    rp, _, rm, rl = oracle.local_step(h.oracle_model, p, {}, mom0, x, y, sel, momentum=0.9, weight_decay=1e-4, **args)
    gp, _, gm, gl = h.local_step(p, {}, mom0, x, y, sel, mu=0.9, wd=1e-4, **args)
    assert_losses_close(gl, rl, rtol=2e-4)
    assert_tensors_close(gm, rm, 3e-4, "momentum")
    delta = lambda a: {k: a[k] - p[k].astype(np.float64) for k in p}
    assert_tensors_close(delta(gp), delta(rp), 3e-4, "parameter change")


def test_noops_and_errors(h, data):
    p, x, y = data
    newp, _, mom, _ = h.local_step(p, {}, _zeros(p), x, y, np.arange(4), 2, 0, lr=0.1)
    for k in p:
        np.testing.assert_array_equal(newp[k], p[k].astype(np.float64))
    with pytest.raises(h.bls.BlsError):
        h.local_step(p, {}, _zeros(p), x, y, np.arange(4), 0, 1, lr=0.1)
    with pytest.raises(h.bls.BlsError):
        h.local_step(p, {}, _zeros(p), x, y, np.arange(4), 2, 1, lr=float("nan"))


@pytest.mark.parametrize("hw,channels,hidden,classes,batch", [
    (5, 3, 16, 2, 1),        # 75 inputs: no 16-byte loads, fewer inputs than one step of all waves; one sample
    (9, 3, 80, 64, 17),     # 243 inputs: one past a 16 x 16 tile of samples, hidden units past a block of 64, most classes
    (16, 1, 272, 10, 33),    # 256 inputs: one workgroup of columns, filled; two feature quads per lane
    (18, 1, 1024, 3, 16),    # 324 inputs: a second workgroup of columns, nearly empty; the largest hidden layer
    (8, 2, 48, 7, 257),      # a second block of 256 samples in the weight gradient, with one sample
])
def test_gradients_and_update_at_the_edges_of_the_kernels(hw, channels, hidden, classes, batch):
    import torch
    import paper_2508_08540_amd as bls
    ctx = bls.Context(0)
    try:
        h = Harness(torch, bls, ctx, bls.Model.mlp(hw, channels, hidden, classes), oracle.MLP())
        x, y = synth.image_pool(3, 40, classes, hw=hw, channels=channels)
        p = synth.mlp_init(3, hw * hw * channels, hidden, classes)
        assert_losses_close(h.score(p, {}, x, y), oracle.score_losses(h.oracle_model, p, {}, x, y))
        sel = np.arange(37, 3, -1, dtype=np.int32)      # shorter than the largest batch: it wraps inside one batch
        mom0 = {k: 0.01 * synth.normal(5, i, v.size).reshape(v.shape) for i, (k, v) in enumerate(p.items())}
        rp, _, rm, rl = oracle.local_step(h.oracle_model, p, {}, mom0, x, y, sel, batch, 1, 0.05, momentum=0.9, weight_decay=1e-2)
        gp, _, gm, gl = h.local_step(p, {}, mom0, x, y, sel, batch, 1, lr=0.05, mu=0.9, wd=1e-2)
        assert_losses_close(gl, rl)
        # momentum = 0.9 * initial + gradient: sums of at most 257 products in fp32, as in the gradient test above
        assert_tensors_close(gm, rm, 1e-4, "momentum")
        # relative to the change itself, which the fp32 parameter quantises to 2^-24 of its size: |p| / |change| < 200 here
        delta = lambda a: {k: a[k] - p[k].astype(np.float64) for k in p}
        assert_tensors_close(delta(gp), delta(rp), 3e-4, "parameter change")
    finally:
        ctx.close()


@pytest.mark.parametrize("hw,channels,hidden,classes,batch", [
    (5, 3, 16, 2, 1),        # 75 inputs, no 16-byte loads; one sample
    (16, 1, 32, 10, 17),     # 256 inputs: one block of inputs, filled; a second group of 16 samples with one of them
    (18, 1, 48, 17, 65),     # 324 inputs: a second block, nearly empty; a second round of samples per wave; more classes than are preloaded
    (8, 2, 16, 7, 128),      # the largest batch whose next first layer rides in the update
    (8, 2, 16, 7, 129),      # the smallest whose does not
    (64, 1, 16, 3, 4),       # 4096 inputs, the most whose partial sums the head still adds up
    (37, 3, 16, 3, 4),       # 4107 inputs
])
def test_steps_whose_first_layer_rides_in_the_update(hw, channels, hidden, classes, batch):
    """Three steps: the partial sums of the second and third come from the update before them.  Criteria as for one step, three times
    as wide."""
    import torch
    import paper_2508_08540_amd as bls
    ctx = bls.Context(0)
    try:
        h = Harness(torch, bls, ctx, bls.Model.mlp(hw, channels, hidden, classes), oracle.MLP())
        x, y = synth.image_pool(3, 300, classes, hw=hw, channels=channels)
        p = synth.mlp_init(3, hw * hw * channels, hidden, classes)
        sel = np.arange(299, 3, -1, dtype=np.int32)
        mom0 = {k: 0.01 * synth.normal(5, i, v.size).reshape(v.shape) for i, (k, v) in enumerate(p.items())}
        rp, _, rm, rl = oracle.local_step(h.oracle_model, p, {}, mom0, x, y, sel, batch, 3, 0.01, momentum=0.9, weight_decay=1e-2)
        gp, _, gm, gl = h.local_step(p, {}, mom0, x, y, sel, batch, 3, lr=0.01, mu=0.9, wd=1e-2)
        assert_losses_close(gl, rl, rtol=2e-4)
        assert_tensors_close(gm, rm, 3e-4, "momentum")
        delta = lambda a: {k: a[k] - p[k].astype(np.float64) for k in p}
        assert_tensors_close(delta(gp), delta(rp), 9e-4, "parameter change")
    finally:
        ctx.close()


@pytest.mark.parametrize("hw,channels,hidden,classes,batch,shift", [
    (5, 3, 16, 2, 1, 0),        # 75 inputs: one part of 256, its last two quarters empty
    (18, 1, 48, 17, 64, 0),     # a second part with one quarter and a remainder; the largest batch of a narrow layer that rides
    (18, 1, 48, 17, 65, 1),     # the smallest that does not; no 16-byte loads
    (18, 1, 96, 17, 65, 1),     # one that does
    (32, 3, 128, 10, 64, 0),    # the measured network
    (16, 1, 96, 10, 128, 0),    # the largest batch whose next first layer rides in the update
    (16, 1, 96, 10, 129, 0),    # the smallest whose does not
    (64, 1, 16, 3, 4, 0),       # 4096 inputs, the most in parts of 256
    (37, 3, 16, 3, 4, 0),       # 4107 inputs
])
def test_one_call_of_three_steps_is_three_calls_of_one(hw, channels, hidden, classes, batch, shift):
    """The partial sums of the first layer are the same whether the update of the step before left them or a launch of its own: same
    weights, momentum and losses, bit for bit."""
    import torch
    import paper_2508_08540_amd as bls
    ctx = bls.Context(0)
    try:
        h = Harness(torch, bls, ctx, bls.Model.mlp(hw, channels, hidden, classes), oracle.MLP())
        h.shift = shift
        x, y = synth.image_pool(4, 3 * batch + 5, classes, hw=hw, channels=channels)
        p = synth.mlp_init(4, hw * hw * channels, hidden, classes)
        mom = {k: 0.01 * synth.normal(6, i, v.size).reshape(v.shape) for i, (k, v) in enumerate(p.items())}
        sel = np.arange(x.shape[0] - 1, -1, -1, dtype=np.int32)
        together = h.local_step(p, {}, mom, x, y, sel, batch, 3, lr=0.01, mu=0.9, wd=1e-2)
        q, m = p, mom
        for j in range(3):
            q, _, m, losses = h.local_step(q, {}, m, x, y, sel[j * batch:(j + 1) * batch], batch, 1, lr=0.01, mu=0.9, wd=1e-2)
            np.testing.assert_array_equal(losses[0], together[3][j])
        for k in p:
            np.testing.assert_array_equal(q[k], together[0][k])
            np.testing.assert_array_equal(m[k], together[2][k])
    finally:
        ctx.close()
