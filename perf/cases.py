"""The workloads a user of this library runs, as timed cases.

A user builds a `FusedNet` once -- filters packed, buffers allocated, normally captured into a HIP
graph -- and then runs it for one batch of images after another.  A case is one such network at one
batch and image size; a pass is one inference.  The networks are those of the paper's vision
evaluation: ResNet-18 (fp16 and the quantized int8 form), MobileNet-v1, VGG-16, the deep Q-network, an
Inception block with its parallel convolutions combined, and a single residual block.

Parameters and images are random with the distributions such a network meets: N(0, 1) images,
He-normal filters, batch-norm scales around 1; int8 codes uniform over +-127 with shifts that keep
the scale of the activations from layer to layer.
"""
import math

import numpy as np
import torch

from paper_1904_08368_amd.fusion import FusedOp
from paper_1904_08368_amd.stack import FusedNet


# ------------------------------------------------------------------------------- networks
def _conv(name, src, dst, cin, cout, r, stride, pad, relu=True, res=None, bias=False):
    return FusedOp("conv", name, src, dst, cin, cout, r, stride, pad, bias, not bias, relu, res)


def _block(ops, p, src, cin, cout, stride):
    """conv 3x3, conv 3x3 with the shortcut added (a 1x1 conv where the shape changes)."""
    ops.append(_conv(p + ".conv1", src, p + ".t", cin, cout, 3, stride, 1))
    short = src
    if stride != 1 or cin != cout:
        ops.append(_conv(p + ".down", src, p + ".d", cin, cout, 1, stride, 0, relu=False))
        short = p + ".d"
    ops.append(_conv(p + ".conv2", p + ".t", p + ".out", cout, cout, 3, 1, 1, res=short))
    return p + ".out"


def _head(ops, src, c):
    """Global average pool and the 1000-class dense layer."""
    ops.append(FusedOp("avgpool", "avgpool", src, "pooled", c, c))
    ops.append(FusedOp("dense", "fc", "pooled", "logits", c, 1000, bias=True))
    return [src, "logits"]


def _resnet18(case):
    ops = [_conv("conv1", "x", "c1", 3, 64, 7, 2, 3),
           FusedOp("maxpool", "maxpool", "c1", "s1.in", 64, 64, 3, 2, 1)]
    cur, cin = "s1.in", 64
    for stage, cout in enumerate((64, 128, 256, 512), start=1):
        for blk in range(2):
            cur = _block(ops, "l%d.b%d" % (stage, blk), cur, cin, cout, 2 if stage > 1 and blk == 0 else 1)
            cin = cout
    # the quantized network ends at its last feature map: the head runs in floating point elsewhere
    return ops, [cur] if case["dtype"] == "i8" else _head(ops, cur, 512), 3


def _mobilenet_v1(case):
    ops, cur, cin = [_conv("stem", "x", "b0", 3, 32, 3, 2, 1)], "b0", 32
    for i, (cout, s) in enumerate(((64, 1), (128, 2), (128, 1), (256, 2), (256, 1), (512, 2), (512, 1), (512, 1), (512, 1),
                                   (512, 1), (512, 1), (1024, 2), (1024, 1)), start=1):
        ops.append(FusedOp("dwconv", "b%d.dw" % i, cur, "b%d.t" % i, cin, cin, 3, s, 1, bn=True, relu=True))
        ops.append(_conv("b%d.pw" % i, "b%d.t" % i, "b%d" % i, cin, cout, 1, 1, 0))
        cur, cin = "b%d" % i, cout
    return ops, _head(ops, cur, 1024), 3


def _vgg16(case):
    ops, cur, cin = [], "x", 3
    for b, (n, cout) in enumerate(((2, 64), (2, 128), (3, 256), (3, 512), (3, 512)), start=1):
        for j in range(1, n + 1):
            ops.append(_conv("conv%d_%d" % (b, j), cur, "c%d_%d" % (b, j), cin, cout, 3, 1, 1, bias=True))
            cur, cin = "c%d_%d" % (b, j), cout
        ops.append(FusedOp("maxpool", "pool%d" % b, cur, "p%d" % b, cin, cin, 2, 2, 0))
        cur = "p%d" % b
    return ops, [cur], 3


def _dqn(case):
    ops = [_conv("c1", "x", "c1", 4, 32, 8, 4, 0, bias=True), _conv("c2", "c1", "c2", 32, 64, 4, 2, 0, bias=True),
           _conv("c3", "c2", "c3", 64, 64, 3, 1, 0, bias=True),
           FusedOp("dense", "fc1", "c3", "h", 64 * 7 * 7, 512, bias=True, relu=True),
           FusedOp("dense", "fc2", "h", "q", 512, 18, bias=True)]
    return ops, ["h", "q"], 4


def _inception(case):
    ops = [_conv("b1", "x", "b1.out", 256, 128, 1, 1, 0), _conv("b3r", "x", "b3r.out", 256, 128, 1, 1, 0),
           _conv("b3", "b3r.out", "b3.out", 128, 192, 3, 1, 1), _conv("b5r", "x", "b5r.out", 256, 32, 1, 1, 0),
           _conv("b5", "b5r.out", "b5.out", 32, 96, 5, 1, 2),
           FusedOp("maxpool", "pool", "x", "pool.out", 256, 256, 3, 1, 1), _conv("bp", "pool.out", "bp.out", 256, 64, 1, 1, 0),
           FusedOp("concat", "cat", "b1.out", "cat", 0, 480, srcs=("b1.out", "b3.out", "b5.out", "bp.out"))]
    return ops, ["cat"], 256


def _residual_block(case):
    ops = []
    return ops, [_block(ops, "blk", "x", case["channels"], case["channels"], 1)], case["channels"]


NETS = {"resnet18": _resnet18, "mobilenet_v1": _mobilenet_v1, "vgg16": _vgg16, "dqn": _dqn, "inception": _inception,
        "block": _residual_block}


# ---------------------------------------------------------------------------------- cases
def _case(net, dtype, batch, h, w, captured=True, channels=0, name=None):
    c = {"net": net, "dtype": dtype, "batch": batch, "h": h, "w": w, "captured": captured, "channels": channels}
    return dict(c, name=name) if name else c


def listed():
    return [
        # an agent that asks its Q-network for one action at a time: six tiny launches
        _case("dqn", "f16", 1, 84, 84, name="dqn_f16_b1"),
        # one residual block on one image, called eagerly: what a call costs a program without a captured graph
        _case("block", "f16", 1, 56, 56, captured=False, channels=64, name="block_f16_b1_eager"),
        # image classification one image at a time, where latency counts
        _case("resnet18", "f16", 1, 224, 224, name="resnet18_f16_b1"),
        _case("resnet18", "i8", 1, 224, 224, name="resnet18_i8_b1"),
        _case("mobilenet_v1", "f16", 1, 224, 224, name="mobilenet_f16_b1"),
        # odd batches of images that are neither square nor a multiple of anything (crops, camera frames)
        _case("resnet18", "f16", 7, 197, 251, name="resnet18_f16_b7_odd"),
        _case("mobilenet_v1", "f16", 11, 163, 206, name="mobilenet_f16_b11_odd"),
        # quantized serving at a moderate batch
        _case("resnet18", "i8", 16, 224, 224, name="resnet18_i8_b16"),
        # an Inception block: parallel convolutions in one launch, outputs stored into the concatenation
        _case("inception", "f16", 32, 28, 28, name="inception_f16_b32"),
        # throughput serving
        _case("mobilenet_v1", "f16", 32, 224, 224, name="mobilenet_f16_b32"),
        _case("resnet18", "f16", 32, 224, 224, name="resnet18_f16_b32"),
        # the largest: VGG-16's convolutions, dense contractions of 31 GFLOP per image
        _case("vgg16", "f16", 32, 224, 224, name="vgg16_f16_b32"),
    ]


def draw(rng):
    """One more case: any of the networks, 1 to 32 images of 128 to 256 pixels a side (the deep Q-network's frames
    are always 84 x 84, feature maps of a single block 7 to 64), mostly captured."""
    net, dtype = rng.choice([("resnet18", "f16"), ("resnet18", "f16"), ("resnet18", "i8"), ("resnet18", "i8"),
                             ("mobilenet_v1", "f16"), ("mobilenet_v1", "f16"), ("vgg16", "f16"), ("dqn", "f16"),
                             ("inception", "f16"), ("block", "f16"), ("block", "i8")])
    batch = min(32, int(math.exp(rng.uniform(0.0, math.log(33.0)))))
    captured = rng.random() < 0.8
    if net == "dqn":
        return _case(net, dtype, batch, 84, 84, captured)
    if net in ("inception", "block"):
        side = lambda: int(math.exp(rng.uniform(math.log(7.0), math.log(65.0))))
        h, w = side(), side()
        return _case(net, dtype, batch, h, w, captured, rng.choice([64, 128, 256, 512]) if net == "block" else 0)
    h, w = rng.randint(128, 256), rng.randint(128, 256)
    if batch * h * w > 32 * 224 * 224:     # (no more work than the largest listed case)
        batch = 32 * 224 * 224 // (h * w)
    return _case(net, dtype, batch, h, w, captured)


# ---------------------------------------------------------------------- state and one pass
def _shift(op):
    """Right shift after which a chained int8 conv has the scale of its input again."""
    return int(round(math.log2(73.3 * math.sqrt(op.cin * op.r * op.r))))


def prepare(case, seed):
    rng = np.random.default_rng(seed)
    ops, outs, cin = NETS[case["net"]](case)
    i8 = case["dtype"] == "i8"
    n, h, w = case["batch"], case["h"], case["w"]

    def normal(shape, mean, std, dtype=np.float32):
        a = rng.standard_normal(shape, dtype=np.float32)
        a *= np.float32(std)
        a += np.float32(mean)
        return a.astype(dtype)

    def codes(shape):
        return rng.integers(-127, 128, size=shape, dtype=np.int8)

    params, shifts = [], []
    for op in ops:
        p = {}
        shape = {"conv": (op.cout, op.cin, op.r, op.r), "dwconv": (op.cin, op.r, op.r), "dense": (op.cout, op.cin)}.get(op.kind)
        if shape and i8:
            p["w"] = codes(shape)
        elif shape:
            fan_in = op.r * op.r * (1 if op.kind == "dwconv" else op.cin)
            p["w"] = normal(shape, 0.0, math.sqrt(2.0 / fan_in), np.float16)
            if op.bias:
                p["bias"] = normal((op.cout,), 0.0, 0.1)
            if op.bn:
                p["scale"], p["shift"] = normal((op.cout,), 1.0, 0.1), normal((op.cout,), 0.0, 0.1)
        params.append(p)
        shifts.append({"s": _shift(op), "l": _shift(op) if op.res else 0} if op.kind == "conv" else {})
    net = FusedNet(ops, params, n, h, w, case["dtype"], shifts=shifts if i8 else None, in_channels=cin,
                   combine=case["net"] == "inception")
    net.load_input(codes((n, cin, h, w)) if i8 else normal((n, cin, h, w), 0.0, 1.0, np.float16))
    if case["captured"]:
        net.capture()
    return {"net": net, "outs": [net.bufs[o] for o in outs], "captured": case["captured"]}


def run(state):
    if state["captured"]:
        state["net"].replay()
    else:
        state["net"].run()
    return state["outs"]


# -------------------------------------------------------------------------- what a pass is
def work(case):
    """Image, filters and results once each; two operations per multiply-accumulate of the contractions."""
    ops, outs, cin = NETS[case["net"]](case)
    es = 1 if case["dtype"] == "i8" else 2
    n = case["batch"]
    hw, ch = {"x": (case["h"], case["w"])}, {"x": cin}
    macs = filters = 0
    for op in ops:
        h, w = hw[op.src]
        if op.kind in ("conv", "dwconv", "maxpool"):
            h, w = ((e + 2 * op.pad - op.r) // op.stride + 1 for e in (h, w))
        elif op.kind != "concat":
            h = w = 1
        hw[op.dst], ch[op.dst] = (h, w), op.cout
        if op.kind in ("conv", "dwconv"):
            k = op.r * op.r * (op.cin if op.kind == "conv" else 1)
            macs += n * h * w * op.cout * k
            filters += op.cout * k
        elif op.kind == "dense":
            macs += n * op.cin * op.cout
            filters += op.cin * op.cout
    results = sum(n * hw[o][0] * hw[o][1] * ch[o] for o in outs)
    return {"bytes": (n * cin * case["h"] * case["w"] + filters + results) * es, "flops": 2.0 * macs}


def tolerance(case):
    """int8 is exact.  fp16: every layer's output is rounded to fp16, and a value that another order of the sums
    rounds differently goes on through the layers behind it, so the deeper the network the further two correct
    implementations are apart.  Stated: about four times what the outputs differ by from the same network in
    64-bit arithmetic between the same fp16 roundings, which is rel 2.9e-5 and max 9.7e-4 for the block of two
    and the Inception block of three convolutions in a row, 2.9e-4 and 9.6e-4 for the Q-network's five layers, 7.9e-4 to 9.2e-4
    and 4.0e-3 to 6.4e-3 for the last feature maps of the 13 to 27 layers of the others."""
    if case["dtype"] == "i8":
        return "exact"
    return {"block": {"rel": 1.2e-4, "max": 4e-3}, "inception": {"rel": 1.2e-4, "max": 4e-3},
            "dqn": {"rel": 1.2e-3, "max": 4e-3}}.get(case["net"], {"rel": 3.6e-3, "max": 2.4e-2})
