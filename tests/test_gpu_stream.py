"""Pooling and input-loader kernels at the sizes where their splits have remainders, against the float64 oracle."""
import pytest

import workloads as wl
from tests import test_gpu_parity as tp

pytestmark = pytest.mark.gpu


# (side, channels): fewer pixels than slices, one more than a round of four slices, channel vectors that fill no block,
# an image smaller than a block of the backward kernel, odd channel counts (stored padded)
@pytest.mark.parametrize("dtype", [wl.F32, wl.BF16])
@pytest.mark.parametrize("side,channels,in_c", [(1, 8, 1), (3, 72, 2), (6, 33, 3), (12, 40, 5), (19, 24, 4)])
def test_pool_and_loader_remainders(dtype, side, channels, in_c):
    models = [[("conv3x3", channels, 1), (act,), ("gap",), ("linear", 7)] for act in ("relu", "tanh")]
    models.append([("conv3x3", channels + 9, 2), ("relu",), ("gap",), ("linear", 7)])
    w = wl.custom(f"pool_{side}_{channels}", 60 + side, dtype, 70, (side, side, in_c), models, batch=[70, 65, 67], n_classes=7, steps=1)
    tp._check_f32(w) if dtype == wl.F32 else tp._check_bf16(w)


# (classes, rows): more rows than a block takes and not a multiple of it, one row, classes at the edges of a group of lanes
# and beyond what the lanes keep in registers
@pytest.mark.parametrize("classes,rows", [(17, [70, 1, 7]), (32, [67, 8, 9]), (33, [5, 4, 64]), (64, [13]), (256, [66]), (257, [65, 3])])
def test_loss_in_blocks_of_rows(classes, rows):
    models = [[("linear", 24), ("tanh",), ("linear", classes)]] * len(rows)
    w = wl.custom(f"loss_{classes}", 80 + classes, wl.F32, max(rows), (1, 1, 40), models, batch=rows, n_classes=classes, steps=2)
    tp._check_f32(w)


# splits of the weight gradients' reductions: fewer than the sixteen that are requested together, some more, twice and some
# more; 33 channels give a bias that is no whole vectors, 40 one that is
@pytest.mark.parametrize("rows,side", [(5, 14), (20, 16), (70, 16)])
def test_split_weight_gradients_are_added_up(rows, side):
    models = [[("conv3x3", 8, 1), ("relu",), ("conv3x3", channels, 1), ("tanh",), ("gap",), ("linear", 7)] for channels in (33, 40)]
    w = wl.custom(f"splits_{rows}", 90 + rows, wl.F32, rows, (side, side, 3), models, n_classes=7, steps=2)
    tp._check_f32(w)
