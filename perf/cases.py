"""Timed cases of the A-SGD hot path, called as a user's program calls it.

A program trains one of three nets (the 28 x 28 MNIST-sized one, the 32 x 32 three-layer one, the AlexNet-style one
with its response-normalised and two-column forms), alone on the GPU or as several replicas of an A-SGD run, in fp32
or in bf16 with fp32 master weights.  A case is one pass of such a program: a training step, a replica's gradient, a
stretch of an A-SGD schedule, or the parameter server's work for one pushed gradient.

    listed()             the cases, with what each stands for
    draw(rng)            one more case of the same ranges
    prepare(case, seed)  what the program holds before the call: plan, parameters, momentum, minibatches
    run(state)           one pass; the results
    work(case)           bytes and operations that a pass cannot do without
    tolerance(case)      how far another correct implementation of the same precision may be off
"""
import math

import numpy as np
import torch

from paper_1312_6186_amd import binding as B
from paper_1312_6186_amd import workloads as wl

# Momentum, weight decay and the dropout seed are the configurations'.  The learning rate is the last stage of a run
# that starts at 0.01 and is cut by ten three times: many passes over one minibatch leave the weights, and with them
# the sparsity of the activations and the size of the gradients, where they were.
LR, MU, WD, DROPOUT_SEED, STALENESS_SEED = 1e-5, 0.9, 5e-4, 3003, 4005


def listed():
    return [
        # the smallest call: a whole training step of the MNIST-sized net, as launch-bound as this path gets
        {"name": "tiny_f32_step", "kind": "step", "net": "tiny", "dtype": "f32", "batch": 8, "step": "calls"},
        # the CIFAR-sized net as it is configured, one step in one call
        {"name": "small_f32_step", "kind": "step", "net": "small", "dtype": "f32", "batch": 128, "step": "fused"},
        # the same net in bf16 on the last, incomplete minibatch of an epoch
        {"name": "small_bf16_ragged", "kind": "step", "net": "small", "dtype": "bf16", "batch": 93, "step": "calls"},
        # the headline workload: the AlexNet-style net, bf16 with fp32 master weights, 128 images
        {"name": "alexnet_bf16_128", "kind": "step", "net": "alexnet", "dtype": "bf16", "batch": 128, "step": "fused"},
        # the largest minibatch that is configured
        {"name": "alexnet_bf16_256", "kind": "step", "net": "alexnet", "dtype": "bf16", "batch": 256, "step": "fused"},
        # the same net in fp32
        {"name": "alexnet_f32_128", "kind": "step", "net": "alexnet", "dtype": "f32", "batch": 128, "step": "calls"},
        # one replica's gradient at the batch an A-SGD worker has, added to those it has not pushed yet
        {"name": "alexnet_bf16_grad_32", "kind": "grad", "net": "alexnet", "dtype": "bf16", "batch": 32},
        # response normalisation after conv1 and conv2, an odd minibatch
        {"name": "alexnet_lrn_bf16_77", "kind": "step", "net": "alexnet_lrn", "dtype": "bf16", "batch": 77, "step": "calls"},
        # the cited architecture in full: response normalisation and two-column convolutions
        {"name": "alexnet_full_bf16_128", "kind": "step", "net": "alexnet_full", "dtype": "bf16", "batch": 128, "step": "fused"},
        # A-SGD on one GPU: four replicas as concurrent streams, eight pushed gradients, up to three updates stale
        {"name": "asgd_4x32", "kind": "replay", "net": "alexnet", "dtype": "bf16", "batch": 32, "workers": 4, "updates": 8, "stale": 3, "n_sync": 0},
        # the paper's regime: four local steps between two exchanges
        {"name": "asgd_nsync4_4x32", "kind": "replay", "net": "alexnet", "dtype": "bf16", "batch": 32, "workers": 4, "updates": 4, "stale": 3, "n_sync": 4},
        # the parameter server alone: a pushed gradient applied, then a replica's fetch, on the whole parameter vector
        {"name": "server_62M", "kind": "server", "rule": "momentum", "dtype": "bf16", "params": 62378344},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["small_net"] * 3 + ["alexnet"] * 5 + ["grad"] * 2 + ["replay"] * 2 + ["server"] * 2)
    dtype = rng.choice(["f32", "bf16", "bf16"])
    step = rng.choice(["calls", "fused"])
    if kind == "small_net":
        net = rng.choice(["tiny", "small"])
        return {"kind": "step", "net": net, "dtype": dtype, "batch": _log_int(rng, 1, 256) if net == "tiny" else _log_int(rng, 16, 512), "step": step}
    net = rng.choice(["alexnet", "alexnet", "alexnet_lrn", "alexnet_full"])
    if kind == "alexnet":
        return {"kind": "step", "net": net, "dtype": dtype, "batch": _log_int(rng, 16, 256) if dtype == "bf16" else _log_int(rng, 16, 128), "step": step}
    if kind == "grad":
        return {"kind": "grad", "net": net, "dtype": dtype, "batch": rng.randint(16, 64)}
    if kind == "replay":
        workers = rng.randint(2, 4)
        n_sync = rng.choice([0, 0, 2, 4])
        return {"kind": "replay", "net": "alexnet", "dtype": "bf16", "batch": rng.randint(16, 32), "workers": workers, "updates": rng.randint(2, 4) if n_sync else rng.randint(3, 8),
                "stale": rng.randint(0, workers - 1), "n_sync": n_sync}
    return {"kind": "server", "rule": rng.choice(["momentum", "adagrad", "adadelta", "fused"]), "dtype": dtype, "params": _log_int(rng, 10000, 62378344)}


class State(dict):
    """What a program keeps between passes; its plans are released with it."""

    def __del__(self):
        if self.get("plans"):
            torch.cuda.synchronize()
            for p in self["plans"]:
                B.asgd_net_destroy(p)


def _torch_dtype(case):
    return torch.bfloat16 if case["dtype"] == "bf16" else torch.float32


def _abi_dtype(case):
    return B.BF16 if case["dtype"] == "bf16" else B.F32


def _parameters(cfg, batch, gen, dev):
    """He-normal weights and zero biases, and the sum of the gradients that a run under way remembers.

    In these nets the root mean square of a minibatch gradient of 128 images is up to 1.2 (fully connected) or 3
    (convolution) times that of its weights; it falls with the square root of the batch.  mu = 0.9 sums up ten
    gradients, most of which agree.
    """
    w, g = [], []
    for _, wshape, blen, fan_in in wl.param_shapes(cfg["layers"], cfg["in_shape"]):
        n, std = int(np.prod(wshape)), math.sqrt(2.0 / fan_in)
        w += [torch.randn(n, generator=gen, device=dev) * std, torch.zeros(blen, device=dev)]
        g += [torch.randn(n + blen, generator=gen, device=dev) * ((20 if len(wshape) == 4 else 8) * std * math.sqrt(128 / batch))]
    return torch.cat(w), torch.cat(g)


def prepare(case, seed):
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    gen.manual_seed(seed)
    tdt, adt = _torch_dtype(case), _abi_dtype(case)
    s = State(case=dict(case), adt=adt, at=0)
    if case["kind"] == "server":
        n = case["params"]
        s["master"] = torch.randn(n, generator=gen, device=dev) * 0.02
        s["grads"] = torch.randn(n, generator=gen, device=dev) * 0.002
        s["state"] = [torch.rand(n, generator=gen, device=dev) * 1e-5 for _ in range(2 if case["rule"] == "adadelta" else 1)]
        s["copy"] = torch.empty(n, dtype=tdt, device=dev)
        return s
    cfg = wl.CONFIGS[case["net"]]
    batch, shape = case["batch"], tuple(cfg["in_shape"])
    workers = case.get("workers", 1)
    minibatches = case["updates"] * max(1, case["n_sync"]) if case["kind"] == "replay" else 1
    s["plans"] = [B.asgd_net_create(cfg["layers"], batch, shape, adt) for _ in range(workers)]
    for p in s["plans"]:
        B.asgd_net_prepare(p)
    s["master"], s["sum"] = _parameters(cfg, batch, gen, dev)
    s["momentum"] = s["sum"] * -LR
    n = s["master"].numel()
    s["images"] = torch.randn((minibatches, batch) + shape, generator=gen, device=dev).to(tdt)
    s["labels"] = torch.randint(0, cfg["classes"], (minibatches, batch), generator=gen, device=dev, dtype=torch.int32)
    s["loss"] = torch.zeros(minibatches, device=dev)
    s["copy"] = [torch.empty(n, dtype=tdt, device=dev) for _ in range(workers)]
    s["grads"] = [torch.zeros(n, device=dev) for _ in range(workers)]
    if case["kind"] == "replay":
        s["worker"], s["reads"] = B.asgd_schedule_generate(case["updates"], STALENESS_SEED + seed, workers, case["stale"])
        s["log"] = torch.zeros((case["updates"], 3), dtype=torch.int32, device=dev)
        if case["n_sync"]:
            s["local"] = [[torch.zeros(n, device=dev) for _ in range(workers)] for _ in range(3)]   # parameters, momentum, accumulator
    else:
        B.asgd_snapshot(s["master"], s["copy"][0], adt)   # the replica's first fetch
    return s


def run(s):
    case = s["case"]
    s["at"] += 1   # the dropout masks' step
    if case["kind"] == "server":
        w, g, st, c = s["master"], s["grads"], s["state"], s["copy"]
        if case["rule"] == "fused":
            B.asgd_apply_update_snapshot(w, st[0], g, LR, MU, WD, c, s["adt"])
            return {"master": w, "state": st, "copy": c}
        if case["rule"] == "momentum":
            B.asgd_apply_update(w, st[0], g, LR, MU, WD)
        elif case["rule"] == "adagrad":
            B.asgd_apply_update_adagrad(w, st[0], g, LR, 1e-7, WD)
        else:
            B.asgd_apply_update_adadelta(w, st[0], st[1], g, 0.95, 1e-6, WD)
        B.asgd_snapshot(w, c, s["adt"])
        return {"master": w, "state": st, "copy": c}
    if case["kind"] == "replay":
        if case["n_sync"]:
            B.asgd_replay_nsync_run(s["plans"], case["n_sync"], s["master"], s["momentum"], s["local"][0], s["local"][1], s["local"][2], s["copy"], s["grads"],
                                    s["images"], s["labels"], s["worker"], s["reads"], LR, MU, WD, DROPOUT_SEED, s["loss"], s["log"])
        else:
            B.asgd_replay_run(s["plans"], s["master"], s["momentum"], s["copy"], s["grads"], s["images"], s["labels"], s["worker"], s["reads"], LR, MU, WD,
                              DROPOUT_SEED, s["loss"], s["log"])
        return {"losses": s["loss"], "master": s["master"], "momentum": s["momentum"], "log": s["log"]}
    plan, copy, grads = s["plans"][0], s["copy"][0], s["grads"][0]
    if case["kind"] == "grad":
        B.asgd_fwd_bwd(plan, copy, s["images"][0], s["labels"][0], DROPOUT_SEED, s["at"], 0, s["loss"], grads)
        B.asgd_accumulate(s["sum"], grads, False)
        return {"loss": s["loss"], "sum": s["sum"]}
    if case["step"] == "fused":
        B.asgd_train_step_fused(plan, s["master"], s["momentum"], copy, s["images"][0], s["labels"][0], DROPOUT_SEED, s["at"], 0, s["loss"], grads, LR, MU, WD)
    else:
        B.asgd_fwd_bwd(plan, copy, s["images"][0], s["labels"][0], DROPOUT_SEED, s["at"], 0, s["loss"], grads)
        B.asgd_apply_update_snapshot(s["master"], s["momentum"], grads, LR, MU, WD, copy, s["adt"])
    return {"loss": s["loss"], "master": s["master"], "momentum": s["momentum"], "copy": copy}


def _gemm_flops(cfg):
    """Multiply-adds times two of one image, forward and backward (no data gradient below the first layer)."""
    c, h, w = cfg["in_shape"]
    total, first = 0, True
    for l in cfg["layers"]:
        if l[0] == "conv":
            groups = l[5] if len(l) > 5 else 1
            h, w = (h + 2 * l[4] - l[2]) // l[3] + 1, (w + 2 * l[4] - l[2]) // l[3] + 1
            macs = l[1] * (c // groups) * l[2] * l[2] * h * w
            c = l[1]
        elif l[0] == "maxpool":
            h, w = (h - l[1]) // l[2] + 1, (w - l[1]) // l[2] + 1
            continue
        elif l[0] == "fc":
            macs = l[1] * c * h * w
            c, h, w = l[1], 1, 1
        else:
            continue
        total += 2 * macs * (2 if first else 3)
        first = False
    return total


def work(case):
    es = 2 if case["dtype"] == "bf16" else 4
    if case["kind"] == "server":
        n, states = case["params"], 2 if case["rule"] == "adadelta" else 1
        return {"bytes": n * (4 + 8 + 8 * states + es), "flops": n * 6 * (1 + states)}
    cfg = wl.CONFIGS[case["net"]]
    n = wl.param_count(cfg["layers"], cfg["in_shape"])
    image = case["batch"] * int(np.prod(cfg["in_shape"])) * es + case["batch"] * 4
    flops = case["batch"] * _gemm_flops(cfg)
    if case["kind"] == "grad":
        return {"bytes": image + n * (es + 12), "flops": flops}
    if case["kind"] == "step":   # parameters and momentum updated in place, the replica's copy read and rewritten
        return {"bytes": image + n * (16 + 2 * es), "flops": flops}
    # a replay reads the parameters and momentum once and writes them once, each replica leaves its copy and gradient
    local = 20 if case["n_sync"] else 0
    k = case["updates"] * max(1, case["n_sync"])
    return {"bytes": k * image + n * (16 + case["workers"] * (es + 4 + local)), "flops": k * flops}


def tolerance(case):
    """About four times what the path differs from itself by when the channels of every layer are reversed (the same
    sums in another order), over the ranges above.

    A pre-activation that is zero up to rounding, or two pooled values equal up to rounding, may fall either way, and
    a gradient moves with the decision: that, not the rounding of the sums, is what is seen (in bf16 up to 2.6e-3 of
    the updated momentum, single elements by 0.2 of its root mean square; in fp32 up to 1e-4 and 0.03).  A replay
    piles such differences up over its updates (1.4e-2 and 0.75).
    """
    if case["kind"] == "server":   # element by element: an ulp, and where it turns the rounding of the replica's copy a bf16 step
        return {"rel": 3e-5, "max": 0.01}
    if case["kind"] == "replay":
        return {"rel": 0.03, "max": 0.99}
    return {"rel": 0.01, "max": 0.8} if case["dtype"] == "bf16" else {"rel": 5e-4, "max": 0.12}
