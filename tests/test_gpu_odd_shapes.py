"""Shapes that fill neither a 16-byte vector nor a chunk nor a tile, on the padded layouts and the general gather of the
convolutions: the device against the CPU oracle, with the tolerances of the other parity tests."""
import numpy as np
import pytest
import torch

import workloads as wl
from paper_2002_02885_amd import binding
from tests import parity_util as pu
from tests import test_gpu_parity as tp
from tests.test_plan_check_host import odd_layers

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,classes", [((6, 5, 3), 3), ((9, 4, 9), 19), ((3, 3, 16), 5), ((1, 1, 13), 17)])
def test_members_of_odd_shapes_f32(shape, classes):
    w = wl.custom(f"odd{shape}", 21, wl.F32, 5, shape, odd_layers(shape[2], classes), batch=[5, 3, 2, 5, 4], n_classes=classes, steps=2)
    tp._check_f32(w, production_form=True)


@pytest.mark.parametrize("make", [
    lambda: wl.custom("odd_bf16", 22, wl.BF16, 70, (7, 9, 3), odd_layers(3, 19)[1:], batch=[70, 64, 66, 70], n_classes=19, steps=2),
    lambda: wl.custom("odd_mlp_bf16", 23, wl.BF16, 67, (1, 1, 203), [wl.mlp([130, 51], 21), wl.mlp([33], 21), [("linear", 21)]], batch=[67, 65, 64], n_classes=21, steps=2),
    lambda: wl.custom("odd_cnn_bf16", 24, wl.BF16, 66, (14, 14, 1), [wl.small_cnn((24, 48, 96), 10)] * 2, batch=[66, 64], steps=2),
])
def test_members_of_odd_shapes_bf16(make):
    tp._check_bf16(make(), production_form=True)


def test_odd_resnets_f32_several_tiles_and_splits():
    tp._check_f32(wl.config5(K=2, B=6, size=19, widths=(20, 40, 72, 72), n_classes=37, steps=2, dtype=wl.F32))


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_members_on_unaligned_blocks_of_their_own_equal_members_alone(dtype):
    """Blocks of 3 rows of 13 features begin where they like; the padded copy gives each member the bits it has alone."""
    layers, B = wl.mlp([21], 5), 3
    rng = np.random.default_rng(3)
    x, y = rng.standard_normal((3 * B, 13)).astype(np.float32), rng.integers(0, 5, 3 * B).astype(np.int32)
    lr = np.full(3, 0.05, np.float32)
    dev = lambda a: (torch.from_numpy(a).to(torch.bfloat16) if dtype == "bf16" and a.dtype == np.float32 else torch.from_numpy(a)).cuda()
    pk = binding.Pack(B, (1, 1, 13), dtype, [layers] * 3, seed=1)
    pk.set_input_mode(True)
    solo = [binding.Pack(B, (1, 1, 13), dtype, [layers], seed=1) for _ in range(3)]
    for k in range(3):
        solo[k].write_weights(0, pk.read_weights(k))
    xd, yd = dev(x), dev(y)
    parts = [(dev(x[k * B:(k + 1) * B].copy()), dev(y[k * B:(k + 1) * B].copy())) for k in range(3)]
    for _ in range(2):
        pk.step(xd.data_ptr(), yd.data_ptr(), lr)
        for k in range(3):
            solo[k].step(parts[k][0].data_ptr(), parts[k][1].data_ptr(), lr[:1])
    for k in range(3):
        assert np.array_equal(pk.read_weights(k), solo[k].read_weights(0))


def test_weights_loaded_after_a_member_diverged_train_as_if_it_never_had():
    """An infinite rate turns everything it touches into NaN, padding between channels included; loading weights cures it."""
    layers, shape, B = [("conv3x3", 9, 1), ("relu",), ("conv3x3", 11, 2), ("relu",), ("linear", 5), ("relu",), ("linear", 3)], (6, 6, 5), 4
    x, y = torch.rand((B,) + shape, device="cuda"), torch.randint(0, 3, (B,), device="cuda", dtype=torch.int32)
    blob = binding.Pack(B, shape, "f32", [layers], seed=5).read_weights(0)
    got = []
    for first in (0.01, np.inf):
        pk = binding.Pack(B, shape, "f32", [layers], seed=5)
        pk.step(x.data_ptr(), y.data_ptr(), np.array([first], np.float32))
        pk.write_weights(0, blob)
        for _ in range(2):
            pk.step(x.data_ptr(), y.data_ptr(), np.array([0.01], np.float32))
        got.append(pk.read_weights(0))
    assert np.all(np.isfinite(got[0])) and np.array_equal(got[0], got[1])


# 251 x 250 pixels: the weight gradient over them goes element by element on padded channels; 256 x 256: whole chunks of
# channels on the staged-tile and halo kernels
@pytest.mark.parametrize("dtype", [wl.F32, wl.BF16])
@pytest.mark.parametrize("shape,widths", [((251, 250, 5), (9, 12)), ((256, 256, 8), (64, 32))])
def test_maps_of_more_than_60000_pixels(shape, widths, dtype):
    layers = [("conv3x3", widths[0], 1), ("relu",), ("conv3x3", widths[1], 1), ("tanh",), ("conv3x3", widths[1], 2), ("relu",), ("gap",), ("linear", 7)]
    w = wl.custom(f"large_map_{shape[0]}", 25, dtype, 1, shape, [layers], n_classes=7, steps=1)
    tp._check_f32(w, trials=1) if dtype == wl.F32 else tp._check_bf16(w, trials=1)


@pytest.mark.parametrize("dtype,widths", [("bf16", (24, 40, 48)), ("f32", (20, 24, 40))])
def test_lean_tiles_of_the_general_gather_give_the_same_bits(dtype, widths, monkeypatch):
    """Forward passes, input gradients of both strides and shortcuts over maps that are no power of two: the form with four
    workgroups per compute unit against the one with two, several chunks and partial tiles of rows and columns."""
    w = wl.config5(K=3, B=9, size=23, widths=widths, n_classes=7, steps=2, dtype=dtype)
    monkeypatch.setenv("PACK_MIN_TILES", "1")       # 128-row tiles, as a larger pack would have
    monkeypatch.setenv("PACK_LEAN64_CHUNKS", "0")
    regular = pu.run_gpu(w, 2)
    monkeypatch.setenv("PACK_LEAN64_CHUNKS", "100000")
    lean = pu.run_gpu(w, 2)
    assert any(t == (128, 64, True) for t in lean["tiles"]) and not any(t == (128, 64, True) for t in regular["tiles"])
    tp._same_bits(regular, lean)
    for k in range(w.K):
        assert np.array_equal(regular["grads"][k], lean["grads"][k])


def test_every_tile_of_single_precision_weight_gradients_of_the_general_gather_gives_the_same_bits(monkeypatch):
    """Full rows of 128 channels, strides 1 and 2, chunks that straddle images: 128 x 128, 128 x 64 and lean 64 x 64 tiles."""
    layers = [("conv3x3", 128, 1), ("relu",), ("conv3x3", 128, 1), ("relu",), ("conv3x3", 256, 2), ("relu",), ("gap",), ("linear", 7)]
    w = wl.custom("gather_dw", 31, wl.F32, 11, (7, 9, 3), [layers] * 2, batch=[11, 10], n_classes=7, steps=1)
    runs = {}
    for least in (100000, 1, 8, 16, 24, 32, 48, 64, 96, 128, 192, 256):
        monkeypatch.setenv("PACK_MIN_TILES", str(least))
        pk = binding.Pack(w.B, w.in_shape, w.dtype, w.models, w.batch)
        tiles = {pk.launch_tile(i) for i in range(pk.num_launches()) if pk.launch_name(i).startswith("gemm_conv_dw")}
        pk.destroy()
        assert len(tiles) == 1
        runs.setdefault(tiles.pop(), least)
    assert set(runs) == {(64, 64, True), (128, 128, False), (128, 64, False)}
    out = []
    for least in runs.values():
        monkeypatch.setenv("PACK_MIN_TILES", str(least))
        out.append(pu.run_gpu(w, 1))
    for other in out[1:]:
        tp._same_bits(out[0], other)
        for k in range(w.K):
            assert np.array_equal(out[0]["grads"][k], other["grads"][k])
