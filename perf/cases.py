"""The work that programs built on this framework have it do, as a list of cases that can be timed and compared.

A case is a dict of plain values that describes one block (or a chain of blocks), what is done with it and at which size:

  path      "distill"  a training task: `steps` distillation steps of one block (Block.distill_step: teacher forward, student
                       forward, local loss, backward, update), then the trained student and its optimiser state are gathered
            "chain"    the same for all blocks of a network at once (distill_step_all), teacher chain on its own stream
            "labels"   the frozen teacher block alone, forward, writing the labels of a data set's batches
            "network"  the reassembled network, forward (network_forward), student blocks in place of the teacher's
            "select"   Algorithm 1's choice of the student blocks to keep (select_blocks)
  n, h, w   batch, height and width of the input
  teacher   channels of the teacher's 3x3 convolutions, "64-128-128"; the blocks of a chain are separated by "/"
  student   the same for the student's depthwise-separable layers; a leading "full:" keeps the first layer a full convolution
  stride    stride of a block's first layer
  shortcut  0 none, 1 projection shortcut in teacher and student, 2 identity skip around the student's layers
  pool      2: a 2x2 max-pool ends every block
  streams   student streams; 1 = everything on the current stream, 2 = teacher and student of a block on one each,
            more = that many student streams beside the teacher's (chain)
  steps     steps (or forward passes) of one pass, over two batches in turn
  inference network: BatchNorm with the running statistics instead of the batch's

Sizes are those of the benchmark's and the tests' blocks, at the batch sizes they are used with, and generic odd ones.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2012_03096_amd import binding as pb, workloads as wl

VGG16 = "3-64-64/64-128-128/128-256-256-256/256-512-512-512/512-512-512-512"
VGG16_STUDENT = "full:3-64-64/64-128-128/128-256-256-256/256-512-512-512/512-512-512-512"
LR = 0.01


def _case(name, path, n, h, w, teacher, student=None, stride=1, shortcut=0, pool=0, streams=1, steps=1, inference=False):
    return {"name": name, "path": path, "n": n, "h": h, "w": w, "teacher": teacher, "student": student or teacher,
            "stride": stride, "shortcut": shortcut, "pool": pool, "streams": streams, "steps": steps, "inference": inference}


def listed():
    return [
        # the smallest block of the repository (a unit test, a first try): bound by launches and host time
        _case("tiny_block", "distill", 4, 16, 16, "16-16-16", steps=50),
        # one stage of a CIFAR-sized network per task, the usual granularity: VGG's second stage, teacher beside student
        _case("cifar_vgg_block2", "distill", 128, 16, 16, "64-128-128", pool=2, streams=2, steps=20),
        # a downsampling residual block with its projection shortcut
        _case("cifar_resnet_down", "distill", 128, 16, 16, "128-256-256", stride=2, shortcut=1, streams=2, steps=20),
        # the largest single block: ImageNet-sized images, first layer kept a full convolution, the headline benchmark
        _case("imagenet_vgg_block1", "distill", 32, 224, 224, "3-64-64", "full:3-64-64", pool=2, streams=2, steps=5),
        # all five stages trained at the same time from one teacher pass
        _case("cifar_vgg16_all", "chain", 128, 32, 32, VGG16, VGG16_STUDENT, pool=2, streams=3, steps=10),
        # the paper's own granularity: one convolution, two depthwise-separable layers for it, deep and on small maps
        _case("conv_task_512_4x4", "distill", 128, 4, 4, "512-512", "512-512-512", steps=20),
        # the last stage at ImageNet size, 14x14 maps (no multiple of 4)
        _case("imagenet_vgg_block5", "distill", 32, 14, 14, "512-512-512-512", pool=2, steps=10),
        # the epoch's last batch of a network that is nobody's benchmark: odd batch, odd channels, odd maps, identity skip
        _case("ragged_skip_block", "distill", 77, 27, 23, "67-100-67", "67-100-67", shortcut=2, steps=10),
        # labels for a data set from one teacher stage, no student
        _case("labels_56x56", "labels", 32, 56, 56, "128-256-256-256", pool=2, steps=2),
        # the compressed network in use, one image at a time and a batch at a time
        _case("network_one_image", "network", 1, 32, 32, VGG16, VGG16_STUDENT, pool=2, steps=4, inference=True),
        _case("network_batch", "network", 128, 32, 32, VGG16, VGG16_STUDENT, pool=2, steps=4, inference=True),
        # which blocks meet the threshold
        _case("select_blocks", "select", 128, 32, 32, VGG16, VGG16_STUDENT, pool=2),
    ]


def _log(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


_MOST = {}


def _cost(case):
    w = work(case)
    return max(w["bytes"] / 8e12, w["flops"] / 100e12)


def draw(rng):
    """One more case: the same paths and kinds of blocks over the whole range of sizes."""
    if not _MOST:
        _MOST["cost"] = max(_cost(c) for c in listed())
    while True:
        kind = rng.choice(["stage", "stage", "residual", "image", "skip", "task", "labels", "network"])
        n, h = _log(rng, 1, 128), _log(rng, 2, 224)
        w = h if rng.random() < 0.6 else max(1, h + rng.randint(-(h // 4), h // 4))
        if rng.random() < 0.4:
            h, w = -(-h // 4) * 4, -(-w // 4) * 4
        c0, c1 = _log(rng, 16, 512), _log(rng, 16, 512)
        if rng.random() < 0.5:
            c0, c1 = -(-c0 // 16) * 16, -(-c1 // 16) * 16
        pool = 2 if rng.random() < 0.5 and h >= 4 and w >= 4 else 0
        streams = rng.choice([1, 2])
        case = None
        if kind == "stage":
            chans = "-".join(str(v) for v in [c0] + [c1] * rng.choice([2, 3]))
            case = _case("", "distill", n, h, w, chans, pool=pool, streams=streams)
        elif kind == "residual":
            case = _case("", "distill", n, h, w, f"{c0}-{c1}-{c1}", stride=rng.choice([1, 2]), shortcut=1, streams=streams)
        elif kind == "image":
            c0 = rng.choice([1, 3, 3, 3])
            chans = f"{c0}-{min(c1, 64)}-{min(c1, 64)}"
            case = _case("", "distill", n, h, w, chans, "full:" + chans, pool=pool, streams=streams)
        elif kind == "skip":
            case = _case("", "distill", n, h, w, f"{c0}-{c1}-{c0}", f"{c0}-{c1}-{c0}", shortcut=2, pool=pool, streams=streams)
        elif kind == "task":
            case = _case("", "distill", n, h, w, f"{c0}-{c1}", f"{c0}-{c1}-{c1}", streams=streams)
        elif kind == "labels":
            case = _case("", "labels", n, h, w, "-".join(str(v) for v in [c0] + [c1] * rng.choice([1, 2, 3])), pool=pool)
        else:
            h = w = rng.choice([32, 48, 64, 96])
            base = rng.choice([16, 24, 32, 48, 64])
            plan = [[3, base, base], [base, 2 * base, 2 * base], [2 * base, 4 * base, 4 * base], [4 * base, 8 * base, 8 * base]]
            text = "/".join("-".join(str(v) for v in p) for p in plan)
            case = _case("", "network", n, h, w, text, "full:" + text, pool=2, inference=rng.random() < 0.7)
        del case["name"]
        one = _cost(case)
        if n * h * w < 256 * case["stride"] ** 2:    # batch statistics of a handful of values: nobody trains on that
            continue
        if 5e-8 < one <= _MOST["cost"]:
            # as many steps as an ordinary short run has, fewer where one is long
            case["steps"] = max(1, min(20 if case["path"] == "distill" else 4, int(0.5 * _MOST["cost"] / one)))
            return case


# ------------------------------------------------------------------------------------------ descriptors
def _archs(case):
    """[(teacher, student)] of the case's blocks, as the framework's descriptors."""
    out = []
    h, w = case["h"], case["w"]
    for t_text, s_text in zip(case["teacher"].split("/"), case["student"].split("/")):
        full = s_text.startswith("full:")
        tc = [int(v) for v in t_text.split("-")]
        sc = [int(v) for v in s_text.removeprefix("full:").split("-")]
        tl = [wl.Layer(wl.CONV3X3, a, b, case["stride"] if i == 0 else 1, 0) for i, (a, b) in enumerate(zip(tc[:-1], tc[1:]))]
        sl = [wl.Layer(wl.CONV3X3 if full and i == 0 else wl.DWSEP3X3, a, b, case["stride"] if i == 0 else 1, 1)
              for i, (a, b) in enumerate(zip(sc[:-1], sc[1:]))]
        short = case["shortcut"]
        t = wl.Arch(case["n"], tc[0], h, w, tl, shortcut=1 if short == 1 else 0, shortcut_stride=case["stride"], pool=case["pool"])
        s = wl.Arch(case["n"], sc[0], h, w, sl, shortcut=short, shortcut_stride=case["stride"], pool=case["pool"])
        out.append((t, s))
        _, _, h, w = wl.output_shape(t)
    return out


def _random_params(arch, gen):
    """He-normal weights, BatchNorm gamma around 1 and beta around 0, as after some training."""
    out = []
    for shapes in wl.param_shapes(arch):
        layer = []
        for k, shape in enumerate(shapes):
            if len(shape) == 1:
                first = len(shapes[k - 1]) > 1                      # gamma, then beta
                v = 0.5 + torch.rand(shape, generator=gen, device="cuda") if first else 0.1 * torch.randn(shape, generator=gen, device="cuda")
            else:
                v = torch.randn(shape, generator=gen, device="cuda") * math.sqrt(2.0 / math.prod(shape[1:]))
            layer.append(v.cpu().numpy())
        out.append(layer)
    return out


_STREAMS = []


def _streams():
    """The program's streams, made once: the teacher's first, then three for the students."""
    if not _STREAMS:
        for _ in range(4):
            s = torch.cuda.Stream()
            with torch.cuda.stream(s):
                torch.zeros(256, device="cuda").add_(1.0)
            torch.cuda.synchronize()
            _STREAMS.append(s)
    return _STREAMS


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(int(seed))
    archs = _archs(case)
    first = archs[0][0]
    image = case["student"].startswith("full:")
    xs = []
    for _ in range(2):
        x = torch.randn((first.n, first.c, first.h, first.w), generator=gen, device="cuda")
        xs.append(x if image else x.clamp_(min=0))                  # a feature map comes out of a ReLU
    blocks = []
    for t, s in archs:
        tp, sp = _random_params(t, gen), _random_params(s, gen)
        if case["shortcut"] == 1:
            sp[-1] = [a.copy() for a in tp[-1]]                     # the shortcut is kept: a copy of the teacher's
        blocks.append(pb.Block(t, tp, s, sp))
    shapes = [wl.output_shape(t) for t, _ in archs]
    state = {"case": case, "blocks": blocks, "xs": xs, "archs": archs, "streams": _streams(),
             "outs": [[torch.zeros(shape, device="cuda") for shape in shapes] for _ in range(2)]}
    if case["path"] == "chain":
        state["stream_of"], state["order"], _ = pb.schedule_blocks(None, case["streams"], 0, blocks=blocks)
    if case["path"] == "network" and case["inference"]:
        # running statistics as training leaves them: those of a batch
        for use, act, run, nets in ((0, pb.TEACHER_ACT, pb.TEACHER_BN_RUNNING, [t for t, _ in archs]),
                                    (1, pb.STUDENT_ACT, pb.STUDENT_BN_RUNNING, [s for _, s in archs])):
            pb.network_forward(blocks, [use] * len(blocks), xs[0], state["outs"][0])
            for b, net in zip(blocks, nets):
                for l, layer in enumerate(net.layers):
                    mean, rstd = (b.get_tensor(act, l, k, (layer.cout,)) for k in (2, 3))
                    # (a batch that leaves a channel one value has no variance: the start value then)
                    var = np.where(rstd > 100, 1.0, 1.0 / np.maximum(rstd.astype(np.float64), 1e-3) ** 2)
                    b.set_tensor(run, l, 0, mean)
                    b.set_tensor(run, l, 1, var.astype(np.float32))
    torch.cuda.synchronize()
    return state


def _gather(block, arch):
    """The trained student as a program collects it at the end of a task: weights, momentum, running statistics, loss."""
    flat = {"weights": [], "momentum": [], "running": []}
    for l, shapes in enumerate(wl.param_shapes(arch)):
        trained = l < len(arch.layers)
        for k, shape in enumerate(shapes):
            if trained:
                flat["weights"].append(block.get_tensor(pb.STUDENT_PARAM, l, k, shape).reshape(-1))
                flat["momentum"].append(block.get_tensor(pb.STUDENT_MOMENTUM, l, k, shape).reshape(-1))
        for k in range(2):
            flat["running"].append(block.get_tensor(pb.STUDENT_BN_RUNNING, l, k, shapes[-1]))
    return {"loss": block.last_loss(), **{k: np.concatenate(v) for k, v in flat.items()}}


def run(state):
    case, blocks, xs, outs, streams = (state[k] for k in ("case", "blocks", "xs", "outs", "streams"))
    path, steps = case["path"], case["steps"]
    if path == "distill":
        ts, ss = (streams[0], streams[1]) if case["streams"] == 2 else (None, None)
        b = blocks[0]
        for i in range(steps):
            b.distill_step(xs[i % 2], outs[i % 2][0], LR, want_loss=False, student_stream=ss, teacher_stream=ts)
        return {"labels": [o[0] for o in outs[:min(steps, 2)]], **_gather(b, state["archs"][0][1])}
    if path == "chain":
        for i in range(steps):
            o = outs[i % 2]
            pb.distill_step_all(blocks, [xs[i % 2]] + o[:-1], o, LR, streams[1:1 + case["streams"]], state["stream_of"],
                                state["order"], True, streams[0])
        return {"labels": outs[0] + outs[1], "students": [_gather(b, s) for b, (_, s) in zip(blocks, state["archs"])]}
    if path == "labels":
        for i in range(steps):
            blocks[0].teacher_forward(xs[i % 2], outs[i % 2][0])
        return [o[0] for o in outs[:min(steps, 2)]]
    if path == "network":
        for i in range(steps):
            pb.network_forward(blocks, [1] * len(blocks), xs[i % 2], outs[i % 2], bn_mode=int(case["inference"]))
        return [o for o in outs[:min(steps, 2)]]
    use, errors, final = pb.select_blocks(blocks, xs[0], outs[0], outs[1], threshold=0.5)
    return {"use": use, "errors": errors, "final": final, "teacher": outs[0], "network": outs[1]}


# ------------------------------------------------------------------------------------------ work, tolerance
def _forward(arch, batch_statistics):
    """(bytes, flops) of one forward pass.  BatchNorm with the batch's statistics is a barrier: a layer's convolution
    output has to be complete before any of it can be normalised, so it is written once and read once; with running
    statistics layers could follow each other on the chip."""
    n, size, flops = arch.n, 0, 0
    for (ci, hi, wi, co, ho, wo), layer in zip(wl.layer_shapes(arch), arch.layers):
        z = n * co * ho * wo
        flops += 2 * 9 * ci * co * n * ho * wo if layer.kind == wl.CONV3X3 else 2 * (9 + co) * ci * n * ho * wo
        size += 2 * z if batch_statistics else 0
    if arch.shortcut == 1:
        flops += 2 * arch.c * co * n * ho * wo
        size += 2 * z if batch_statistics else 0
    weights = sum(math.prod(s) for shapes in wl.param_shapes(arch) for s in shapes)
    return 4 * (size + weights + n * arch.c * arch.h * arch.w), flops


def _step(teacher, student):
    """(bytes, flops) of one distillation step.  Backward: each layer's convolution output once more, the gradient that
    arrives at its BatchNorm written and read (its two channel sums are another barrier), the block input once more, and
    weights, gradients and momentum."""
    tb, tf = _forward(teacher, True)
    sb, sf = _forward(student, True)
    target = math.prod(wl.output_shape(teacher))
    size, flops = 2 * target, 0
    for l, ((ci, hi, wi, co, ho, wo), layer) in enumerate(zip(wl.layer_shapes(student), student.layers)):
        z = student.n * co * ho * wo
        size += 3 * z
        f = 2 * 9 * ci * co if layer.kind == wl.CONV3X3 else 2 * (9 + co) * ci
        flops += (f if l == 0 and layer.kind == wl.CONV3X3 else 2 * f - (18 * ci if l == 0 else 0)) * student.n * ho * wo
    size += student.n * student.c * student.h * student.w
    size += 4 * sum(math.prod(s) for shapes in wl.param_shapes(student) for s in shapes)
    return tb + sb + 4 * size, tf + sf + flops


def work(case):
    archs, steps = _archs(case), case["steps"]
    outs = [4 * math.prod(wl.output_shape(t)) for t, _ in archs]
    size = flops = 0
    if case["path"] in ("distill", "chain"):
        for t, s in archs:
            b, f = _step(t, s)
            size, flops = size + b, flops + f
    elif case["path"] == "labels":
        size, flops = _forward(archs[0][0], True)
        size += outs[0]
    elif case["path"] == "network":
        for (_, s), o in zip(archs, outs):
            b, f = _forward(s, not case["inference"])
            size, flops = size + b + o, flops + f
    else:                                     # the teacher network, each student block with the teacher behind it, the choice
        for k, ((t, s), o) in enumerate(zip(archs, outs)):
            tb, tf = _forward(t, True)
            sb, sf = _forward(s, True)
            size += (2 + k) * (tb + o) + sb + o
            flops += (2 + k) * tf + sf
        size += 2 * (len(archs) + 1) * outs[-1]
    return {"bytes": steps * size, "flops": steps * flops}


def tolerance(case):
    """About four times the differences measured between fp32 runs whose sums go in another order (other tiles of the
    pointwise kernels, fp32 instead of split-operand teacher convolutions).  Forward passes: rounding only, 2e-6 for one
    block, 1e-5 to 2e-5 for a chain of them.  Training: where a pre-activation rounds to the other side of a ReLU's kink,
    that element's gradient is switched on or off; up to 7e-4 of a single block's momentum after forty steps, 5e-3 in a
    chain of five, in single channels some tens of times that."""
    if case["path"] == "distill":
        return {"rel": 3e-3, "max": 0.2}
    if case["path"] == "chain":
        return {"rel": 2e-2, "max": 0.6}
    return {"rel": 1e-5 if case["path"] == "labels" else 1e-4}
