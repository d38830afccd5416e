"""The padding of stored rows and channels stays zero: nothing that a step, another pack's step or a diverged member left
behind may reach a member's results through it."""
import numpy as np
import pytest
import torch

import workloads as wl
from paper_2002_02885_amd import binding
from tests import parity_util as pu
from tests import test_gpu_parity as tp

pytestmark = pytest.mark.gpu

KINDS = {"sgd": None, "momentum": {"kind": "momentum"}, "adagrad": {"kind": "adagrad"}, "adam": {"kind": "adam"}}


def _fill_static_scratch_with_nan(dtype):
    """A step on NaN in the library's static scratch array: 16 splits' worth of partial sums of 64 x 64 weights, all NaN."""
    pk = binding.Pack(16384, (1, 1, 64), dtype, [[("linear", 64)]], seed=1)
    x = torch.full((16384, 64), float("nan"), device="cuda", dtype=torch.bfloat16 if dtype == "bf16" else torch.float32)
    y = torch.zeros(16384, device="cuda", dtype=torch.int32)
    pk.step_static(x.data_ptr(), y.data_ptr(), np.zeros(1, np.float32))
    assert np.isnan(pk.read_loss()[0]) and pk.workspace_bytes() > 16 * 64 * 64 * 4
    pk.destroy()


# rows of 30, 36, 50 and 20 features are stored as 32, 40, 56 and 24, and a batch of 2000 splits the weight gradients: what the
# products leave unwritten in the scratch array would be added into the weights' padding and so reach every output
@pytest.mark.parametrize("opt", ["sgd", "momentum", "adagrad", "adam"])
@pytest.mark.parametrize("dtype,features,hidden,classes", [(wl.F32, 30, [50, 20], 7), (wl.F32, 36, [50], 19), (wl.BF16, 30, [50], 7), (wl.BF16, 30, [], 19)])
def test_split_weight_gradients_of_padded_rows(dtype, features, hidden, classes, opt):
    w = wl.custom(f"split_{features}_{classes}", 31 + classes, dtype, 2000, (1, 1, features), [wl.mlp(hidden, classes) if hidden else [("linear", classes)]],
                  n_classes=classes, steps=3, lr=[0.02 if opt in ("sgd", "momentum") else 0.002])
    if KINDS[opt]:
        w.meta["optimizers"] = [KINDS[opt]]
    gpu = (tp._check_f32(w) if dtype == wl.F32 else tp._check_bf16(w))[0]
    _fill_static_scratch_with_nan(dtype)
    pk = binding.Pack(w.B, w.in_shape, w.dtype, w.models, w.batch)
    pk.write_weights(0, w.weights[0])
    if KINDS[opt]:
        pk.set_optimizer(0, KINDS[opt])
    x, y = pu.device_inputs(w)
    for _ in range(w.steps):
        pk.step_static(x.data_ptr(), y.data_ptr(), w.lr)
    assert np.array_equal(pk.read_weights(0).view(np.uint32), gpu["blobs"][0].view(np.uint32))
    assert np.array_equal(pk.read_loss(), gpu["loss"][-1].astype(np.float32))
    pk.destroy()


def _checkpoint(pk, opt):
    slots = {"sgd": 0, "momentum": 1, "adagrad": 1, "adam": 2}[opt]
    return pk.read_weights(0), [pk.read_opt_state(0, s) for s in range(slots)]


def _load(pk, ckpt):
    pk.write_weights(0, ckpt[0])
    for s, (state, steps) in enumerate(ckpt[1]):
        pk.write_opt_state(0, s, state, steps)


# an infinite pixel makes infinite and NaN gradients; the first convolution over 1 to 3 channels stores 9 to 27 weights in rows
# of 32, the others 9 or 12 channels in groups of 16
@pytest.mark.parametrize("opt", ["sgd", "momentum", "adagrad", "adam"])
@pytest.mark.parametrize("dtype", [wl.F32, wl.BF16])
@pytest.mark.parametrize("shape,layers", [((8, 8, 3), wl.small_cnn((8, 16, 16), 10)), ((8, 8, 1), wl.small_cnn((9, 12, 16), 10)),
                                          ((6, 6, 5), [("conv3x3", 9, 1), ("relu",), ("conv3x3", 12, 2), ("tanh",), ("linear", 11), ("relu",), ("linear", 3)])])
def test_checkpoint_loaded_after_a_divergence_trains_as_if_there_had_been_none(shape, layers, dtype, opt):
    B, lr = 4, np.array([0.01], np.float32)
    x = torch.rand((B,) + shape, device="cuda").to(torch.bfloat16 if dtype == wl.BF16 else torch.float32)
    y = torch.randint(0, 3, (B,), device="cuda", dtype=torch.int32)
    bad = x.clone()
    bad.view(-1)[::7] = float("inf")

    def pack():
        pk = binding.Pack(B, shape, dtype, [layers], seed=5)
        if KINDS[opt]:
            pk.set_optimizer(0, KINDS[opt])
        return pk

    pk = pack()
    pk.step(x.data_ptr(), y.data_ptr(), lr)
    ckpt = _checkpoint(pk, opt)
    got = []
    for diverges in (False, True):
        pk = pack()
        if diverges:
            pk.step(bad.data_ptr(), y.data_ptr(), lr)
            assert not np.all(np.isfinite(pk.read_weights(0)))
        _load(pk, ckpt)
        for _ in range(2):
            pk.step(x.data_ptr(), y.data_ptr(), lr)
        after = _checkpoint(pk, opt)
        got.append([after[0], pk.read_loss()] + [s for s, _ in after[1]])
        pk.destroy()
    for a, b in zip(*got):
        assert np.all(np.isfinite(a)) and np.array_equal(a, b)
