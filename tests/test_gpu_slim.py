"""The slim form of the dense products (a workgroup's waves share the reduction): at the edges of its tiles, chunks and
waves against 64-bit sums of the same operands, against the staged tiles, and when a member's optimiser changes its form."""
import numpy as np
import pytest
import torch

import workloads as wl
from paper_2002_02885_amd import binding
from tests import parity_util as pu

pytestmark = pytest.mark.gpu


def _dev(a, dtype):
    return (torch.from_numpy(a).to(torch.bfloat16) if dtype == "bf16" and a.dtype == np.float32 else torch.from_numpy(a)).cuda()


# rows, features, width, classes: one element, the last and first of tiles of 32 and 64, chunks of 32 (fp32) and 64 (bf16)
# indices, eight waves' chunks and one more, rows of no whole vector, the largest product of the form
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("B,D,H,classes", [(1, 1, 1, 17), (31, 63, 33, 18), (32, 64, 32, 20), (33, 65, 31, 33), (64, 255, 65, 101), (65, 257, 64, 64),
                                           (100, 513, 127, 19), (128, 1030, 1023, 37), (256, 520, 512, 100), (256, 36, 500, 31)])
def test_products_of_the_slim_form(B, D, H, classes, dtype):
    """Two linear layers without an activation between them: every product of the step is one the test can add up."""
    rng = np.random.default_rng(B + D)
    K = 2
    layers = [("linear", H), ("linear", classes)]
    x = rng.standard_normal((B, D)).astype(np.float32)
    y = rng.integers(0, classes, B).astype(np.int32)
    q = (lambda a: torch.from_numpy(np.asarray(a, np.float32)).to(torch.bfloat16).double().numpy()) if dtype == "bf16" else (lambda a: np.asarray(a, np.float64))
    n = [H * D, H, classes * H, classes]
    pk = binding.Pack(B, (1, 1, D), dtype, [layers] * K, [B, max(1, B - 1)])
    tiles = [pk.launch_tile(i)[:2] for i in range(pk.num_launches()) if pk.launch_name(i) in ("gemm_lin_fwd", "gemm_lin_dx")]
    assert len(tiles) == 3 and all(t == (32, 32) for t in tiles)
    pk.keep_grads(True)
    for k in range(K):
        w = rng.standard_normal(sum(n)).astype(np.float32) * 0.1
        pk.write_weights(k, q(w).astype(np.float32))
    blobs = [pk.read_weights(k).astype(np.float64) for k in range(K)]
    xd, yd = _dev(x, dtype), _dev(y, dtype)
    pk.step(xd.data_ptr(), yd.data_ptr(), np.zeros(K, np.float32))
    for k in range(K):
        rows = pk.batch[k]
        W1, b1, W2, b2 = np.split(blobs[k], np.cumsum(n)[:3])
        W1, W2, X = W1.reshape(H, D), W2.reshape(classes, H), q(x[:rows])
        h = X @ W1.T + b1
        z = q(h) @ W2.T + b2
        e = np.exp(z - z.max(1, keepdims=True))
        dz = (e / e.sum(1, keepdims=True) - np.eye(classes)[y[:rows]]) / rows
        dh = q(dz) @ W2
        grads = np.concatenate([(q(dh).T @ X).ravel(), dh.sum(0) if dtype == "f32" else q(dh).sum(0), (q(dz).T @ q(h)).ravel(), q(dz).sum(0)])
        # fp32: sums of up to 2000 products, each term's error below 2^-24 * sqrt(n), and the softmax's exponentials.  bf16: the
        # same sums decide now and then how a stored value rounds (half a bit of 8), which a 2-norm over few values shows
        tol = 5e-6 if dtype == "f32" else 6e-3
        assert pu.rel_l2(pk.read_logits(k).astype(np.float64), z) < tol
        got = pk.read_grads(k).astype(np.float64)
        for a, b in zip(np.split(got, np.cumsum(n)[:3]), np.split(grads, np.cumsum(n)[:3])):
            assert np.linalg.norm(a - b) <= tol * np.linalg.norm(b) + 1e-9
    pk.destroy()


# members of one width: 32 x 32 tiles alone; together, the slim form's 64 x 64 (bfloat16 forward, long reductions) and the
# staged tiles of 64 x 64, 128 x 64 and (bfloat16) 128 x 128, each with partial tiles and a partial last share
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("B,D,H,K,tiles", [(33, 2600, 505, 40, ((32, 32), (64, 64))), (250, 140, 230, 20, ((64, 64),) * 2), (200, 784, 500, 32, ((128, 64),) * 2),
                                           (126, 36, 1000, 64, ((128, 64), (128, 128))), (256, 1030, 500, 70, ((128, 64), (128, 128)))])
def test_every_tile_of_the_form_gives_a_member_the_same_bits(B, D, H, K, tiles, dtype):
    rng = np.random.default_rng(B)
    model = wl.mlp([H], 17)
    x, y = _dev(rng.standard_normal((B, D)).astype(np.float32), dtype), _dev(rng.integers(0, 17, B).astype(np.int32), dtype)
    batch = [B] + [B - int(k % 3) for k in range(1, K)]
    pk = binding.Pack(B, (1, 1, D), dtype, [model] * K, batch, seed=2)
    assert pk.launch_tile([pk.launch_name(i) for i in range(pk.num_launches())].index("gemm_lin_fwd"))[:2] == tiles[dtype == "bf16"]
    solo = {}
    for k in (0, K - 1):
        solo[k] = binding.Pack(batch[k], (1, 1, D), dtype, [model], seed=2)
        solo[k].write_weights(0, pk.read_weights(k))
    for _ in range(2):
        pk.step(x.data_ptr(), y.data_ptr(), np.full(K, 0.01, np.float32))
        for p in solo.values():
            p.step(x.data_ptr(), y.data_ptr(), np.full(1, 0.01, np.float32))
    for k, p in solo.items():
        assert np.array_equal(pk.read_weights(k).view(np.uint32), p.read_weights(0).view(np.uint32)), k
        assert np.array_equal(pk.read_logits(k).view(np.uint32), p.read_logits(0).view(np.uint32)), k
        p.destroy()
    pk.destroy()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_both_tiles_and_any_company_give_a_member_the_same_bits(dtype):
    """Forty members of unlike width take staged tiles in the order of the slim form, one alone takes 32 x 32."""
    rng = np.random.default_rng(4)
    B, D, K = 96, 700, 40
    models = [wl.mlp([int(rng.integers(200, 400)), int(rng.integers(8, 300))], 21) for _ in range(K)]
    batch = [B if k == 0 else int(rng.integers(1, B + 1)) for k in range(K)]
    x, y = _dev(rng.standard_normal((B, D)).astype(np.float32), dtype), _dev(rng.integers(0, 21, B).astype(np.int32), dtype)
    pk = binding.Pack(B, (1, 1, D), dtype, models, batch, seed=2)
    assert any(pk.launch_name(i) == "gemm_lin_fwd" and pk.launch_tile(i)[:2] == (64, 64) for i in range(pk.num_launches()))
    solo = {}
    for k in (0, 7, 39):
        solo[k] = binding.Pack(batch[k], (1, 1, D), dtype, [models[k]], seed=2)
        solo[k].write_weights(0, pk.read_weights(k))
    for _ in range(3):
        pk.step(x.data_ptr(), y.data_ptr(), np.full(K, 0.01, np.float32))
        for p in solo.values():
            p.step(x.data_ptr(), y.data_ptr(), np.full(1, 0.01, np.float32))
    for k, p in solo.items():
        assert np.array_equal(pk.read_weights(k).view(np.uint32), p.read_weights(0).view(np.uint32)), k


def test_a_change_of_optimiser_changes_the_form_of_a_single_precision_member_and_nothing_else():
    """Members under Adam keep the staged tiles: turned over in a live pack, they train like members that always had it."""
    B, D = 40, 300
    rng = np.random.default_rng(5)
    models = [wl.mlp([130], 21)] * 3
    x, y, lr = _dev(rng.standard_normal((B, D)).astype(np.float32), "f32"), _dev(rng.integers(0, 21, B).astype(np.int32), "f32"), np.full(3, 1e-3, np.float32)
    a, b = (binding.Pack(B, (1, 1, D), "f32", models, seed=1) for _ in range(2))
    forms = lambda p: sorted(p.launch_tile(i)[0] for i in range(p.num_launches()) if p.launch_name(i) == "gemm_lin_fwd")
    assert forms(a) == [32, 32]
    for p, order in ((a, ("adam", "momentum", "adam")), (b, ("momentum", "adam", "sgd"))):
        for k, o in enumerate(order):
            p.set_optimizer(k, {"kind": o})
    b.set_optimizer(0, {"kind": "adam"})
    b.set_optimizer(1, {"kind": "momentum"})
    b.set_optimizer(2, {"kind": "adam"})
    assert forms(a) == forms(b) == [64, 64]     # slim and staged problems in one launch
    for k in range(3):
        b.write_weights(k, a.read_weights(k))
    solo = [binding.Pack(B, (1, 1, D), "f32", models[:1], seed=1) for _ in range(3)]
    for k, o in enumerate(("adam", "momentum", "adam")):     # (each alone: one form or the other)
        solo[k].set_optimizer(0, {"kind": o})
        solo[k].write_weights(0, a.read_weights(k))
    for _ in range(3):
        for p in (a, b):
            p.step(x.data_ptr(), y.data_ptr(), lr)
        for k in range(3):
            solo[k].step(x.data_ptr(), y.data_ptr(), lr[k:k + 1])
    for k in range(3):
        assert np.array_equal(a.read_weights(k).view(np.uint32), solo[k].read_weights(0).view(np.uint32)), k
    assert np.array_equal(a.read_loss(), b.read_loss())
    for k in range(3):
        assert np.array_equal(a.read_weights(k).view(np.uint32), b.read_weights(k).view(np.uint32)), k
