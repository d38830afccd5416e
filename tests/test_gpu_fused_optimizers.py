"""Optimisers with state applied in the kernels that produce the gradients: the same bits as the separate update launch, for
whole and partial tiles, split reductions (vectors and single elements), convolutions that are not split, mixed members."""
import numpy as np
import pytest
import torch

import workloads as wl
from paper_2002_02885_amd import binding

pytestmark = pytest.mark.gpu
KINDS = ("adam", "sgd", "momentum", "adagrad", "adam")
STATES = {"sgd": 0, "momentum": 1, "adagrad": 1, "adam": 2}


@pytest.mark.parametrize("large_tiles", [False, True])            # True: the tile shapes of a large pack
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("B,shape,layers", [
    (40, (1, 1, 530), wl.mlp([257, 64], 7)),                       # short reductions: lean 64 x 64 tiles, apart lean 128 x 128
    (700, (1, 1, 300), wl.mlp([200], 19)),                         # longer ones: the pipelined tiles, partial ones
    (700, (1, 1, 60), wl.mlp([200], 19)),
    (2000, (1, 1, 30), wl.mlp([50, 20], 7)),                       # split reductions, biases of no whole vector
    (6, (14, 14, 3), [("conv3x3", 20, 1), ("relu",), ("res_begin",), ("conv3x3", 24, 2), ("relu",), ("conv3x3", 24, 1), ("res_end",), ("gap",), ("linear", 10)]),
    (16, (16, 16, 8), [("conv3x3", 64, 1), ("relu",), ("conv3x3", 64, 1), ("relu",), ("conv3x3", 64, 2), ("tanh",), ("linear", 33)]),
])
def test_fused_and_separate_updates_give_the_same_bits(B, shape, layers, dtype, large_tiles, monkeypatch):
    if large_tiles:
        monkeypatch.setenv("PACK_MIN_TILES", "1")
    rng = np.random.default_rng(B)
    x = torch.from_numpy(rng.random((B,) + shape, dtype=np.float32)).to(torch.bfloat16 if dtype == "bf16" else torch.float32).cuda()
    y = torch.from_numpy(rng.integers(0, 7, B).astype(np.int32)).cuda()
    K, lr = len(KINDS), np.array([1e-3, 1e-2, 1e-3, 1e-2, 1e-4], np.float32)

    def train():
        pk = binding.Pack(B, shape, dtype, [layers] * K, [B, B, B - 1, B, 1], seed=3)
        for k, kind in enumerate(KINDS):
            pk.set_optimizer(k, {"kind": kind})
        for _ in range(3):
            pk.step(x.data_ptr(), y.data_ptr(), lr)
        out = [pk.read_loss()] + [pk.read_weights(k) for k in range(K)] + [pk.read_grads(k) for k in range(K)]
        for k, kind in enumerate(KINDS):
            for s in range(STATES[kind]):
                state, steps = pk.read_opt_state(k, s)
                assert steps == 3
                out.append(state)
        n = pk.num_launches()
        tiles = {pk.launch_tile(i) for i in range(n) if pk.launch_name(i).startswith("gemm_lin_dw")}
        pk.destroy()
        return out, n, tiles

    fused, n, fused_tiles = train()
    monkeypatch.setenv("PACK_NO_FUSED_UPDATE", "1")
    separate, m, separate_tiles = train()
    if large_tiles and shape[0] == 1:
        if B == 40:
            assert (64, 64, True) in fused_tiles and (128, 128, True) in separate_tiles
        elif B == 700:
            assert (128, 128 if shape[2] == 300 else 64, False) in fused_tiles
    assert n <= m and all(np.isfinite(a).all() for a in fused)
    for i, (a, b) in enumerate(zip(fused, separate)):
        assert np.array_equal(np.asarray(a, np.float32).view(np.uint32), np.asarray(b, np.float32).view(np.uint32)), i
