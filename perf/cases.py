"""The work that a user of this library has it do, as measurable cases.

Three kinds of pass, all through the library's binding:

  forward   one layer of a pruned network at inference: swconv_forward
  finetune  one training step of a layer with its sparsity pattern fixed: swconv_update_values (the optimizer's
            new values), swconv_forward, swconv_backward on the transformed input that the forward pass left
  prune     one training step of a layer whose pattern changes: swconv_set_weights_device (the pattern and values
            that the last pruning step left on the device), swconv_forward, swconv_backward, swconv_prune_step

Sizes are the repository's own layer configurations (paper_1702_08597_amd/synth.py) and generic ones between and
around them; values are post-ReLU-like activations, N(0, 0.05) weights on iid Bernoulli masks (or the skewed
recipe), and a small normal gradient of the output.
"""
import math
import weakref

import numpy as np
import torch

from paper_1702_08597_amd import binding as sw
from paper_1702_08597_amd import synth

# SGD rate, L1 factor and the two thresholds of the pruning step (the last two are the paper's recommendation)
ETA, LAM, EPS, BETA = 1e-3, 1e-4, 1e-4, 0.1


def _layer(name, kind, **change):
    c = {k: v for k, v in synth.CONFIGS[name].items() if k != "seed"}
    skew = c["density"] is None
    c["density"] = 0.155 if skew else c["density"]  # the skewed recipe draws its own: U[0.01, 0.30] per position
    case = {"kind": kind, "skew": skew, **c}
    case.update(change)
    return case


def listed():
    return [
        # serving one image at a time: three launches of a few microseconds, latency is everything
        {"name": "forward_conv3_n1_f2", **_layer("alexnet_conv3_n1_f2", "forward")},
        # the 3x3 layers of a pruned AlexNet at the batch sizes of the repository's tables
        {"name": "forward_conv3_n32", **_layer("alexnet_conv3_n32_f4", "forward")},
        {"name": "forward_conv4_n64", **_layer("alexnet_conv4_n64_f4", "forward")},
        # a mildly pruned layer: the products outweigh the traffic
        {"name": "forward_conv5_n64_d30", **_layer("alexnet_conv5_n64_f4", "forward", density=0.30)},
        # very uneven positions and rows: what the schedule has to balance
        {"name": "forward_conv4_skewed", **_layer("conv4_skewed_n64_f4", "forward")},
        # the largest layer, the benchmark's workload: everything streams through device memory
        {"name": "forward_vgg56_n32", **_layer("vgg_56_n32_f4", "forward")},
        # the 5x5 layer: few channels, few non-zeros per row
        {"name": "forward_conv2_f2r5", **_layer("alexnet_conv2g_n32_f2r5", "forward")},
        # nothing divides anything: ragged tiles, blocks that span images, rows and channels that fill no slice
        {"name": "forward_ragged", "kind": "forward", "skew": False, "N": 11, "C": 131, "H": 29, "W": 23, "K": 187,
         "m": 4, "r": 3, "pad": 1, "density": 0.07},
        # training steps with the pattern fixed: an AlexNet layer, the largest layer, the 5x5 layer
        {"name": "finetune_conv4_n64", **_layer("alexnet_conv4_n64_f4", "finetune")},
        {"name": "finetune_vgg56_n32", **_layer("vgg_56_n32_f4", "finetune")},
        {"name": "finetune_conv2_f4r5", **_layer("alexnet_conv2g_n32_f4r5", "finetune")},
        # a training step that prunes: the pattern goes back into the plan
        {"name": "prune_conv3_n32", **_layer("alexnet_conv3_n32_f4", "prune")},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """A case of the same ranges: 1 to 64 images of 7 to 64 pixels a side, 16 to 512 channels, densities 0.04 to 0.30."""
    top = work(_layer("vgg_56_n32_f4", "finetune"))
    while True:
        kind = rng.choice(["forward", "forward", "forward", "finetune", "finetune", "prune"])
        m, r = rng.choice([(4, 3), (4, 3), (4, 3), (2, 3), (2, 5), (4, 5)])
        case = {"kind": kind, "skew": rng.random() < 0.15, "N": _log(rng, 1, 64), "C": _log(rng, 16, 512),
                "H": _log(rng, 7, 64), "W": 0, "K": _log(rng, 16, 512), "m": m, "r": r, "pad": r // 2,
                "density": round(math.exp(rng.uniform(math.log(0.04), math.log(0.30))), 3)}
        case["W"] = case["H"] if rng.random() < 0.6 else _log(rng, 7, 64)
        if case["skew"]:
            case["density"] = 0.155
        if r == 5:  # 5x5 layers have few channels
            case["C"], case["K"] = _log(rng, 16, 128), _log(rng, 16, 256)
        w = work(case)
        weights = (m + r - 1) ** 2 * case["K"] * case["C"] * case["density"]
        v_and_m = synth.geometry(**_shape(case))["T"] * (m + r - 1) ** 2 * max(case["C"], case["K"]) * 4
        # no costlier than the largest listed case, its weights and intermediates no larger than theirs
        if w["bytes"] <= top["bytes"] and w["flops"] <= top["flops"] and weights <= 1.6e6 and v_and_m <= 240e6:
            return case


def _shape(case):
    return {k: case[k] for k in ("N", "C", "H", "W", "K", "m", "r", "pad")}


def prepare(case, seed):
    g = synth.geometry(**_shape(case))
    N, C, K = case["N"], case["C"], case["K"]
    if case["skew"]:
        rowptr, colidx, vals = synth.skewed_weights(g["P"], K, C, seed)
    else:
        rowptr, colidx, vals = synth.bernoulli_weights(g["P"], K, C, case["density"], seed)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    s = _State()
    s.kind = case["kind"]
    s.plan = sw.swconv_plan_create(N, C, case["H"], case["W"], K, case["m"], case["r"], case["pad"])
    weakref.finalize(s, sw.swconv_plan_destroy, s.plan)
    sw.swconv_set_weights(s.plan, rowptr, colidx, vals)
    s.x = torch.randn((N, C, case["H"], case["W"]), generator=gen, device="cuda").clamp_(min=0)
    s.out = torch.empty((N, K, g["Ho"], g["Wo"]), device="cuda")
    if s.kind != "forward":
        # a network that is pruned while it trains keeps its CSR arrays at a fixed capacity
        cap = int(0.31 * g["P"] * K * C) + 64 if case["skew"] else int(1.02 * g["P"] * K * C * case["density"]) + 512
        s.vals = _at_capacity(vals, cap)
        # a loss averaged over the batch: small gradients, of which a pruning step drops a small share of the weights
        s.dout = torch.randn(s.out.shape, generator=gen, device="cuda").mul_(1e-4)
        s.din = torch.empty_like(s.x)
        s.dvals = torch.zeros_like(s.vals)
    if s.kind == "prune":
        s.rows = g["P"] * K
        s.rowptr, s.colidx = torch.from_numpy(rowptr).cuda(), _at_capacity(colidx, cap)
        s.updated = torch.zeros_like(s.vals)
        s.new_rowptr, s.new_colidx, s.new_vals = (torch.zeros_like(s.rowptr), torch.zeros_like(s.colidx),
                                                  torch.zeros_like(s.vals))
    return s


def _at_capacity(a, cap):
    full = np.zeros(cap, dtype=a.dtype)
    full[:len(a)] = a
    return torch.from_numpy(full).cuda()


class _State:
    """What the user's program holds for a layer; the plan goes when it goes."""


def run(s):
    stream = torch.cuda.current_stream().cuda_stream
    if s.kind == "prune":
        sw.swconv_set_weights_device(s.plan, stream, s.rowptr.data_ptr(), s.colidx.data_ptr(), s.vals.data_ptr())
    elif s.kind == "finetune":
        sw.swconv_update_values(s.plan, stream, s.vals.data_ptr())
    sw.swconv_forward(s.plan, stream, s.x.data_ptr(), s.out.data_ptr())
    if s.kind == "forward":
        return s.out
    sw.swconv_backward(s.plan, stream, 0, s.dout.data_ptr(), s.din.data_ptr(), s.dvals.data_ptr())
    if s.kind == "finetune":
        return s.out, s.din, s.dvals
    sw.swconv_prune_step(s.rows, s.rowptr.data_ptr(), s.colidx.data_ptr(), s.vals.data_ptr(), s.dvals.data_ptr(), ETA,
                         LAM, EPS, BETA, stream, s.updated.data_ptr(), s.new_rowptr.data_ptr(), s.new_colidx.data_ptr(),
                         s.new_vals.data_ptr())
    return s.out, s.din, s.dvals, s.updated, s.new_rowptr, s.new_colidx, s.new_vals


def work(case):
    """Tensors once in and once out, the CSR arrays once (8 bytes an entry), two operations per non-zero and tile and
    product: one product forward, two backward."""
    g = synth.geometry(**_shape(case))
    nnz = g["P"] * case["K"] * case["C"] * case["density"]
    x = case["N"] * case["C"] * case["H"] * case["W"] * 4
    y = case["N"] * case["K"] * g["Ho"] * g["Wo"] * 4
    nbytes, flops = x + y + 8 * nnz, 2 * nnz * g["T"]
    if case["kind"] != "forward":
        nbytes += y + x + 8 * nnz  # dL/dO in, dL/dI out, values in, their gradient out
        flops *= 3
    if case["kind"] == "prune":
        nbytes += 12 * nnz  # the values in the old pattern and the new arrays
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """Against the layer in 64 bits the outputs measure rel 0.9e-7 to 2.7e-7 and max 0.5e-6 to 6.3e-6 (the skewed
    layer, whose fullest rows sum all 384 channels): four times the largest.  `differ`: whether an entry is pruned is a
    comparison of floats."""
    return {"rel": 1.1e-6, "max": 2.5e-5, "differ": 0.001}
