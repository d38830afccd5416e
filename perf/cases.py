"""The workloads this library's speed is judged by.

A pass is what a program that uses the library does between two decisions: it trains a pack for a
number of steps, every step on a batch of its own, and takes the results (losses, logits of the last
step, every member's checkpoint).  Two kinds of pass also build their pack, because the programs they
stand for do: a rung of the hyper-parameter search (`Tuner.train_group`) and an epoch over members
with different batch sizes, whose members leave the live pack as they finish.

A case is a dict of plain values; a member list that is not uniform is drawn from the case's `mix`
number.  Learning rates are hyper-parameters and belong to the case; data and initial weights come
from the seed.
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

from paper_2002_02885_amd import binding, tuner

STATES = {"sgd": 0, "momentum": 1, "adagrad": 1, "adam": 2}    # optimisers, and the state arrays each keeps


def _case(name, kind, dtype, K, B, steps, *, features=0, side=0, channels=0, width=0, depth=0, classes=10, uniform=True,
          batches="full", optimizer="sgd", inputs="shared", samples=0, mix=0):
    """kind: mlp | cnn | resnet | rung | epoch.  uniform: all members alike, else widths (and depths) differ.
    batches: full (all members take the whole batch) | scaled (1, 1/2 or 1/4 of it) | any (any part of it down to
    a quarter).  inputs: shared | own (every member its own data)."""
    return {"name": name, "kind": kind, "dtype": dtype, "K": K, "B": B, "steps": steps, "features": features, "side": side,
            "channels": channels, "width": width, "depth": depth, "classes": classes, "uniform": uniform, "batches": batches,
            "optimizer": optimizer, "inputs": inputs, "samples": samples, "mix": mix}


def listed():
    return [
        # two little networks on flat 28 x 28 pictures, the smallest pack of the benchmark: launches and host calls
        _case("mlp-small-f32", "mlp", "f32", 2, 32, 100, features=784, width=128, depth=1),
        # eight equal MLPs on flat colour pictures, the benchmark's pack of equals, for an epoch of 50 000: weights dominate
        _case("mlp-equal-bf16", "mlp", "bf16", 8, 256, 195, features=3072, width=1024, depth=2),
        # thirty-two unlike MLPs with three batch sizes, the benchmark's ragged pack
        _case("mlp-ragged-bf16", "mlp", "bf16", 32, 128, 100, features=3072, width=1024, depth=4, uniform=False, batches="scaled", mix=3),
        # tabular data: a feature count, layer widths and batches that are multiples of nothing, many classes, momentum
        _case("mlp-odd-bf16", "mlp", "bf16", 6, 100, 50, features=1030, width=500, depth=3, classes=101, uniform=False,
              batches="any", optimizer="momentum", mix=5),
        # wide layers in single precision with the optimiser that keeps most state
        _case("mlp-wide-adam-f32", "mlp", "f32", 3, 256, 100, features=3072, width=2048, depth=3, classes=100, optimizer="adam"),
        # a rung of the search: the tuner builds a group of unlike trials (batch size, optimiser, activation), loads their
        # checkpoints, trains them and takes the checkpoints back
        _case("search-rung-bf16", "rung", "bf16", 8, 70, 100, features=3072, width=512, depth=1, optimizer="mixed", mix=7),
        # one epoch over three batch sizes: index schedule, batches gathered on the device, members leaving as they finish
        _case("epoch-leaving-f32", "epoch", "f32", 3, 200, 0, features=784, width=300, depth=2, samples=4000, mix=2),
        # the benchmark's small convolutional networks in single precision
        _case("cnn-f32", "cnn", "f32", 4, 128, 20, side=32, channels=3, width=32),
        # 28 x 28 grey pictures: maps that are no power of two, channel counts that fill no tile, unlike batches, own data
        _case("cnn-odd-bf16", "cnn", "bf16", 5, 100, 20, side=28, channels=1, width=24, batches="any", optimizer="momentum", inputs="own", mix=4),
        # the benchmark's residual networks
        _case("resnet-bf16", "resnet", "bf16", 4, 64, 20, side=64, channels=3, width=64, classes=100),
        # the same at twice the members and twice the batch, every member on its own data: the largest
        _case("resnet-large-bf16", "resnet", "bf16", 8, 128, 6, side=64, channels=3, width=64, classes=100, inputs="own"),
        # residual networks of another width on pictures of another size, single precision, unlike batches
        _case("resnet-odd-f32", "resnet", "f32", 2, 40, 10, side=48, channels=3, width=40, classes=37, batches="any", optimizer="adagrad", mix=6),
    ]


def draw(rng):
    def log(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    def size(lo, hi):
        """A size of the range; every second one a multiple of 16, as people like them."""
        v = log(lo, hi)
        return max(lo, min(hi, 16 * max(1, round(v / 16)))) if rng.random() < 0.5 else v

    while True:
        kind = rng.choice(("mlp", "mlp", "cnn", "resnet", "rung", "epoch"))
        mix = rng.randrange(1 << 20)
        dtype = rng.choice(("bf16", "bf16", "f32"))
        opt = rng.choice(("sgd", "sgd", "sgd", "momentum", "adagrad", "adam"))
        batches = rng.choice(("full", "full", "scaled", "any"))
        inputs = rng.choice(("shared", "shared", "shared", "own"))
        if kind == "mlp":
            c = _case("", kind, dtype, log(1, 30), size(20, 256), rng.choice((20, 50, 100)), features=rng.choice((784, 3072, size(100, 4000))),
                      width=size(64, 2048), depth=rng.randint(1, 4), classes=rng.choice((10, 100, log(2, 200))), uniform=rng.random() < 0.5,
                      batches=batches, optimizer=opt, inputs=inputs, mix=mix)
        elif kind == "cnn":
            c = _case("", kind, dtype, log(1, 8), size(16, 128), rng.choice((5, 10, 20)), side=rng.choice((28, 32, rng.randint(16, 64))),
                      channels=rng.choice((1, 3)), width=size(16, 64), classes=rng.choice((10, log(2, 200))), batches=batches, optimizer=opt,
                      inputs=inputs, mix=mix)
        elif kind == "resnet":
            c = _case("", kind, dtype, log(1, 8), size(16, 128), rng.choice((3, 6, 10)), side=rng.choice((32, 64, rng.randint(24, 72))), channels=3,
                      width=rng.choice((32, 64, 64, size(24, 80))), classes=rng.choice((10, 100, log(2, 200))), batches=batches, optimizer=opt,
                      inputs=inputs, mix=mix)
        elif kind == "rung":
            # (the tuner hands out rows where they lie, and a batch has to be 16-byte aligned: feature counts are multiples of 4)
            c = _case("", kind, dtype, log(2, 16), 70, rng.choice((50, 100)), features=rng.choice((784, 3072, 4 * log(25, 1000))),
                      width=size(64, 1024), depth=rng.randint(1, 3), optimizer="mixed", mix=mix)
        else:
            c = _case("", kind, dtype, log(2, 8), size(64, 256), 0, features=rng.choice((784, 3072, size(100, 2000))), width=size(64, 1024),
                      depth=rng.randint(1, 3), optimizer=opt, samples=log(1000, 5000), mix=mix)
        c.pop("name")
        w = work(c)
        params = sum(_params(m, _in_shape(c)) for m in _members(c)[0])
        # no more work than the largest listed case; single precision and sizes that are multiples of nothing take a smaller share,
        # since an operation costs more there
        share = 1.0 if dtype == "bf16" and all(v % 16 == 0 for v in (c["width"], c["side"])) else 1 / 24
        most = work(listed()[10])
        if w["flops"] <= share * most["flops"] and params <= 40e6:
            return c


# ---- members of a case ---------------------------------------------------------------------------------

def _in_shape(case):
    return (1, 1, case["features"]) if case["kind"] in ("mlp", "rung", "epoch") else (case["side"], case["side"], case["channels"])


def _mlp(widths, classes, act="relu"):
    return [op for w in widths for op in (("linear", w), (act,))] + [("linear", classes)]


def _cnn(w, classes):
    return [("conv3x3", w, 1), ("relu",), ("conv3x3", 2 * w, 1), ("relu",), ("conv3x3", 4 * w, 2), ("relu",), ("gap",), ("linear", classes)]


def _resnet(w, classes):
    ops = [("conv3x3", w, 1), ("relu",)]
    for i in range(4):
        ops += [("res_begin",), ("conv3x3", w << i, 1 if i == 0 else 2), ("relu",), ("conv3x3", w << i, 1), ("res_end",)]
    return ops + [("gap",), ("linear", classes)]


def _members(case):
    """(layer lists, batch sizes, optimisers, learning rates) of the case's members."""
    rng = random.Random(case["mix"])
    models, batch, opts, lr = [], [], [], []
    for _ in range(case["K"]):
        if case["kind"] == "cnn":
            models.append(_cnn(case["width"], case["classes"]))
        elif case["kind"] == "resnet":
            models.append(_resnet(case["width"], case["classes"]))
        elif case["uniform"]:
            models.append(_mlp([case["width"]] * case["depth"], case["classes"]))
        else:
            depth = rng.randint(min(2, case["depth"]), case["depth"])
            models.append(_mlp([max(8, case["width"] >> rng.randint(0, 4)) for _ in range(depth)], case["classes"]))
        b = case["B"]
        if case["batches"] == "scaled":
            b = max(1, b >> rng.randint(0, 2))
        elif case["batches"] == "any":
            b = rng.randint(max(1, b // 4), b)
        batch.append(b)
        opt = rng.choice(tuple(STATES)) if case["optimizer"] == "mixed" else case["optimizer"]
        opts.append(opt)
        lr.append(10.0 ** rng.uniform(*{"sgd": (-4, -2.5), "momentum": (-4.5, -3.5)}.get(opt, (-5.5, -4.5))))
    if max(batch) < case["B"]:
        batch[rng.randrange(case["K"])] = case["B"]
    return models, batch, opts, np.array(lr, dtype=np.float32)


def _trials(case):
    """The trials of a rung: rows of the tuner's search space (the two largest rates left out: some optimisers diverge there)."""
    rng = random.Random(case["mix"])
    return [(rng.randrange(len(tuner.BATCH_SIZES)), rng.randrange(len(tuner.OPTIMIZERS)), rng.randrange(len(tuner.LEARNING_RATES) - 2),
             rng.randrange(len(tuner.ACTIVATIONS))) for _ in range(case["K"])]


def _epoch_batches(case):
    rng = random.Random(case["mix"])
    return [case["B"]] + [max(8, int(case["B"] * rng.choice((0.5, 0.4, 0.25, 0.2)))) for _ in range(case["K"] - 1)]


def _out(n, s):
    return (n - 1) // s + 1


def _layers(layers, shape):
    """(reduction, outputs, output pixels) of every parameterised layer."""
    h, w, c = shape
    for op in layers:
        if op[0] == "linear":
            yield h * w * c, op[1], 1
            h, w, c = 1, 1, op[1]
        elif op[0] == "conv3x3":
            h, w = _out(h, op[2]), _out(w, op[2])
            yield 9 * c, op[1], h * w
            c = op[1]
        elif op[0] == "gap":
            h = w = 1


def _params(layers, shape):
    return sum((k + 1) * n for k, n, _ in _layers(layers, shape))


# ---- one pass ------------------------------------------------------------------------------------------

def _data(case, n, gen):
    """n samples and labels on the GPU: standard normal features, pictures with pixels in [0, 1)."""
    shape = (n,) + _in_shape(case)
    draw_ = torch.randn if case["kind"] in ("mlp", "rung", "epoch") else torch.rand
    x = draw_(shape, device="cuda", generator=gen)
    y = torch.randint(0, case["classes"], (n,), device="cuda", dtype=torch.int32, generator=gen)
    return (x.to(torch.bfloat16) if case["dtype"] == "bf16" else x), y


def _stream():
    return torch.cuda.current_stream().cuda_stream


def _blob(layers, shape, gen, dtype):
    """A checkpoint as a search starts from: uniform weights of the usual scale."""
    parts = []
    for k, n, _ in _layers(layers, shape):
        for size, bound in ((k * n, math.sqrt(6.0 / k)), (n, 1.0 / math.sqrt(k))):
            parts.append((torch.rand(size, device="cuda", generator=gen) * 2 - 1) * bound)
    flat = torch.cat(parts)
    return (flat.to(torch.bfloat16).float() if dtype == "bf16" else flat).cpu().numpy()


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    state = {"case": case}
    if case["kind"] == "rung":
        n = case["steps"] * max(tuner.BATCH_SIZES) + max(tuner.BATCH_SIZES)
        state["x"], state["y"] = _data(case, n, gen)
        state["tuner"] = tuner.Tuner(state["x"].data_ptr(), state["y"].data_ptr(), n, _in_shape(case), case["dtype"],
                                     tuner.mlp_family([case["width"]] * case["depth"], case["classes"]), None, sync=torch.cuda.synchronize)
        state["cfgs"] = _trials(case)
        family = tuner.mlp_family([case["width"]] * case["depth"], case["classes"])
        state["blobs"] = [_blob(family(tuner.ACTIVATIONS[c[3]]), _in_shape(case), gen, case["dtype"]) for c in state["cfgs"]]
        return state
    if case["kind"] == "epoch":
        state["x"], state["y"] = _data(case, case["samples"], gen)
        state["seed"] = seed
        B = case["B"]
        state["bx"] = torch.empty((B,) + _in_shape(case), device="cuda", dtype=state["x"].dtype)
        state["by"] = torch.empty(B, device="cuda", dtype=torch.int32)
        return state
    models, batch, opts, lr = _members(case)
    blocks = case["K"] if case["inputs"] == "own" else 1
    state["batches"] = [_data(case, blocks * case["B"], gen) for _ in range(case["steps"])]
    pk = binding.Pack(case["B"], _in_shape(case), case["dtype"], models, batch, seed=seed, stream=_stream())
    if case["inputs"] == "own":
        pk.set_input_mode(True)
    for k, o in enumerate(opts):
        if o != "sgd":
            pk.set_optimizer(k, {"kind": o})
    state["pack"], state["lr"] = pk, lr
    return state


def _results(state):
    """The losses and logits of the last step and every member's trained weights."""
    pk, members = state["pack"], range(state["case"]["K"])
    return {"loss": pk.read_loss(), "logits": np.concatenate([pk.read_logits(k).ravel() for k in members]),
            "weights": [pk.read_weights(k) for k in members]}


def run(state):
    case = state["case"]
    if case["kind"] == "rung":
        return _run_rung(state)
    if case["kind"] == "epoch":
        return _run_epoch(state)
    pk, lr = state["pack"], state["lr"]
    for x, y in state["batches"]:
        pk.step(x.data_ptr(), y.data_ptr(), lr)
    return _results(state)


def _run_rung(state):
    """A rung as the search runs it: the group's pack is built, trained from the trials' checkpoints and taken apart again."""
    trials = [tuner.Trial(c, b) for c, b in zip(state["cfgs"], state["blobs"])]
    state["tuner"].train_group(trials, state["case"]["steps"])
    return {"loss": np.array([t.loss for t in trials]), "weights": [t.weights for t in trials]}


def _run_epoch(state):
    """One epoch in which every member sees every sample once; a member leaves the live pack when it is through."""
    case = state["case"]
    models, _, opts, lr = _members(case)
    batch = _epoch_batches(case)
    pk = binding.Pack(case["B"], _in_shape(case), case["dtype"], models, batch, seed=state["seed"], stream=_stream())
    for k, o in enumerate(opts):
        if o != "sgd":
            pk.set_optimizer(k, {"kind": o})
    sched = binding.Schedule(case["samples"], batch)
    live, weights, loss = set(range(case["K"])), [None] * case["K"], np.zeros(case["K"], dtype=np.float32)

    def leave(k):
        weights[k] = pk.read_weights(k)
        live.discard(k)
        if live:
            pk.free(k)

    while True:
        nxt = sched.next()
        if nxt is None:
            break
        idx, rows_k, _ = nxt
        for k in [k for k in sorted(live) if rows_k[k] == 0]:
            leave(k)
        rows = [int(rows_k[k]) if k in live else 1 for k in range(case["K"])]
        if len(idx) != pk.B or any(pk.batch[k] != rows[k] for k in live):
            pk.set_batch(len(idx), rows)
        idx_dev = torch.from_numpy(idx).cuda()
        pk.gather_batch(state["x"].data_ptr(), state["y"].data_ptr(), case["samples"], idx_dev.data_ptr(), len(idx),
                        state["bx"].data_ptr(), state["by"].data_ptr())
        pk.step(state["bx"].data_ptr(), state["by"].data_ptr(), lr)
        state["idx"] = idx_dev    # alive until the next batch has been asked for
    for k in sorted(live):
        loss[k] = pk.read_loss()[k]
    for k in sorted(live):
        leave(k)
    pk.destroy()
    return {"loss": loss, "weights": weights}


# ---- what a pass cannot do without ---------------------------------------------------------------------

def work(case):
    """Operations: the matrix products of the steps, 2 per multiply-add (no input gradient for a first layer).  Bytes: per
    step the batch, the float32 weights read and written and so the optimiser state (a step cannot begin before the one
    before it has ended); once per pass every checkpoint taken (and loaded, where the pass builds its pack)."""
    shape, esz = _in_shape(case), 2 if case["dtype"] == "bf16" else 4
    per_row = esz * shape[0] * shape[1] * shape[2] + 4
    if case["kind"] == "rung":
        cfgs = _trials(case)
        models = [tuner.mlp_family([case["width"]] * case["depth"], case["classes"])(tuner.ACTIVATIONS[c[3]]) for c in cfgs]
        opts = [tuner.OPTIMIZERS[c[1]] for c in cfgs]
        rows = [case["steps"] * tuner.BATCH_SIZES[c[0]] for c in cfgs]
        steps, data_rows = [case["steps"]] * len(cfgs), max(rows)
    elif case["kind"] == "epoch":
        models, _, opts, _ = _members(case)
        rows = [case["samples"]] * case["K"]
        steps, data_rows = [math.ceil(case["samples"] / b) for b in _epoch_batches(case)], case["samples"]
    else:
        models, batch, opts, _ = _members(case)
        rows = [case["steps"] * b for b in batch]
        steps, data_rows = [case["steps"]] * case["K"], (sum(rows) if case["inputs"] == "own" else max(rows))
    flops, nbytes = 0.0, float(data_rows * per_row)
    for m, o, r, s in zip(models, opts, rows, steps):
        for i, (k, n, px) in enumerate(_layers(m, shape)):
            flops += 2.0 * r * px * k * n * (2 if i == 0 else 3)
        p = _params(m, shape)
        nbytes += s * p * 8.0 * (1 + STATES[o])
        nbytes += 4.0 * p * (2 + STATES[o] if case["kind"] == "rung" else 1)
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """Measured with the rows of every batch in another order and the loss, the update and the halo form of the convolutions
    done by other kernels, over two passes: training carries the last bits on, so a pass of many steps ends farther apart
    than one sum does.  bfloat16 (a last bit of a sum moves a stored activation or weight by 2^-9): rel 0.005, max 0.08.
    Single precision: rel 1e-5, max 1e-3; Adam divides by the root of the second moment, which lifts the noise of small
    gradients to the size of an update: rel 7e-4, max 0.02."""
    if case["dtype"] == "bf16":
        return {"rel": 0.02, "max": 0.3}
    return {"rel": 4e-3, "max": 0.1} if case["optimizer"] in ("adam", "mixed") else {"rel": 1e-4, "max": 4e-3}
