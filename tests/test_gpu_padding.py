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
