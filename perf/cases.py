"""The work a user of this package has it do, as sized cases.

Families and what they stand for:
  infer       the ResNet-50-shaped stack of 53 blocks with folded batch norm, inference, planned arena: serving one
              image, a small batch of an odd image size, a throughput batch.
  bottleneck  one training step over an identity bottleneck (1x1, 3x3, 1x1 + shortcut + ReLU): the benchmark shape, the
              last stage's shape, a small and a ragged batch.
  stage2      one training step over the four bottlenecks of stage 2 (strided 3x3, strided projection, identity blocks).
  stem        one training step over the 7x7 / stride 2 stem (no gradient to the image).
  block       one block through the two calls of the C interface as they stand: forward, L1 gradient, and a backward call
              that masks its own gradient and adds a shortcut gradient; bf16 with channel counts of every kind and the
              fp32 configuration.

A pass of the first four is the prepared sequence that ``runner.Sequencer`` records; a pass of the last is three calls of
``binding``.  All inputs are drawn on the GPU from the seed, from the distributions the workloads use.
"""
import math

import numpy as np
import torch

from paper_2205_10357_amd import binding as B
from paper_2205_10357_amd import runner
from paper_2205_10357_amd import workloads as wl


# ------------------------------------------------------------------------------------------------------------- cases
def listed():
    return [
        # the fp32 correctness configuration: one 3x3 block, batch 1 (smallest call: launches and latency)
        dict(name="block_f32_16", family="block", dtype="f32", n=1, h=16, w=16, c_in=16, c_out=16, k=3, stride=1),
        # one block called through the interface, channels a multiple of 64: masks its own gradient
        dict(name="block_3x3_128", family="block", dtype="bf16", n=32, h=28, w=28, c_in=128, c_out=128, k=3, stride=1),
        # channel counts that are multiples of 8 only, odd image, stride 2
        dict(name="block_3x3_ragged", family="block", dtype="bf16", n=19, h=45, w=37, c_in=72, c_out=104, k=3, stride=2),
        # serving one image: latency of 55 small launches
        dict(name="infer_n1", family="infer", n=1, hw=224),
        # a small batch of images whose size is no multiple of 32
        dict(name="infer_n6_odd", family="infer", n=6, hw=203),
        # throughput inference, the benchmark batch
        dict(name="infer_n128", family="infer", n=128, hw=224),
        # the stem's training step at the benchmark batch
        dict(name="stem_n32", family="stem", n=32, hw=224),
        # the headline benchmark: bottleneck at 14x14, batch 64
        dict(name="bottleneck_14_n64", family="bottleneck", n=64, hw=14, width=256),
        # few images per step: tiles do not fill the chip
        dict(name="bottleneck_14_n7", family="bottleneck", n=7, hw=14, width=256),
        # the last stage's bottleneck: few pixels, long reductions, large weights
        dict(name="bottleneck_7_n48", family="bottleneck", n=48, hw=7, width=512),
        # a stage-2 training step of an odd image size and batch
        dict(name="stage2_n11_odd", family="stage2", n=11, hw=51),
        # the stage-2 training step at the benchmark batch
        dict(name="stage2_n128", family="stage2", n=128, hw=56),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    family = rng.choice(["block", "block", "block_f32", "infer", "infer", "bottleneck", "bottleneck", "stage2", "stem"])
    if family == "block_f32":
        return dict(family="block", dtype="f32", n=rng.randint(1, 4), h=rng.randint(8, 24), w=rng.randint(8, 24), c_in=rng.randint(4, 32),
                    c_out=rng.randint(4, 32), k=rng.choice([1, 3]), stride=rng.choice([1, 2]))
    if family == "block":
        ch = lambda: 64 * rng.randint(1, 4) if rng.random() < 0.5 else 8 * rng.randint(2, 32)
        return dict(family="block", dtype="bf16", n=_log_int(rng, 1, 64), h=rng.randint(7, 56), w=rng.randint(7, 56), c_in=ch(), c_out=ch(),
                    k=rng.choice([1, 3]), stride=rng.choice([1, 1, 2]))
    if family == "infer":
        return dict(family="infer", n=_log_int(rng, 1, 100), hw=rng.randint(128, 240))
    if family == "bottleneck":
        return dict(family="bottleneck", n=_log_int(rng, 2, 96), hw=rng.randint(7, 16), width=rng.choice([128, 256, 256, 512]))
    if family == "stage2":
        return dict(family="stage2", n=_log_int(rng, 4, 100), hw=rng.randint(32, 60))
    return dict(family="stem", n=_log_int(rng, 1, 64), hw=rng.randint(96, 256))


# ------------------------------------------------------------------------------------------------------ geometry
def _ops(case):
    if case["family"] == "infer":
        return wl.resnet50_ops(), 3
    if case["family"] == "stem":
        return [wl.ConvBlock("stem", 3, 64, 7, 2, 3, True, 0, 1, None, 0)], 3
    if case["family"] == "stage2":
        return wl.stage2_ops(True), 256
    ops = []
    wl.bottleneck(ops, "b", 0, 1, 0, 4 * case["width"], case["width"], 1, project=False)
    return ops, 4 * case["width"]


def _workload(case):
    """The case's op list with placeholder arrays; the values are drawn on the GPU afterwards."""
    ops, c = _ops(case)
    zeros = lambda *shape: np.broadcast_to(np.float32(0), shape)
    train = case["family"] != "infer"
    w = wl.Workload(0, case["family"], "bf16", case["n"], case["hw"], case["hw"], c, ops, zeros(case["n"], c, case["hw"], case["hw"]),
                    train=train, need_input_grad=case["family"] not in ("stem", "infer"))
    for o in w.conv_blocks():
        w.params[o.layer] = dict(W=zeros(o.c_out, o.c_in, o.k, o.k), scale=zeros(o.c_out), shift=zeros(o.c_out))
    if train:
        w.target = zeros(case["n"], *w.tensor_shapes()[ops[-1].out])
    return w


def _block_desc(case):
    return B.BlockDesc(case["n"], case["h"], case["w"], case["c_in"], case["c_out"], case["k"], case["k"], case["stride"], case["k"] // 2,
                       B.SOL_F32 if case["dtype"] == "f32" else B.SOL_BF16, B.SOL_RELU)


# ------------------------------------------------------------------------------------------------------- inputs
class _Draw:
    def __init__(self, seed, device="cuda:0"):
        self.g = torch.Generator(device=device)
        self.g.manual_seed(int(seed))
        self.device = device

    def uniform(self, shape, dtype, lo=0.0, hi=1.0):
        return torch.empty(shape, dtype=torch.float32, device=self.device).uniform_(lo, hi, generator=self.g).to(dtype)

    def normal(self, shape, dtype, std=1.0):
        return torch.empty(shape, dtype=torch.float32, device=self.device).normal_(0.0, std, generator=self.g).to(dtype)

    def params(self, c_out, k, c_in, dtype):
        return dict(W=self.normal((c_out, k, k, c_in), dtype, math.sqrt(2.0 / (c_in * k * k))),
                    scale=self.uniform((c_out,), torch.float32, 0.5, 1.5), shift=self.normal((c_out,), torch.float32, 0.1))


def prepare(case, seed):
    d = _Draw(seed)
    if case["family"] == "block":
        return _prepare_block(case, d)
    w = _workload(case)
    seq = runner.Sequencer(w, d.device)
    x = seq.act[0]
    x.copy_(d.normal(x.shape, x.dtype) if case["family"] in ("stem", "bottleneck") else d.uniform(x.shape, x.dtype))
    for o in w.conv_blocks():
        for key, t in d.params(o.c_out, o.k, o.c_in, seq.tdtype).items():
            seq.params[o.layer][key].copy_(t)
    if w.train:
        seq.target.copy_(d.uniform(seq.target.shape, seq.target.dtype))
    seq.prepared()
    return seq


def _prepare_block(case, d):
    desc = _block_desc(case)
    dt = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    xs, ys = (desc.N, desc.H, desc.W, desc.C_in), (desc.N, desc.Ho, desc.Wo, desc.C_out)
    s = dict(desc=desc, x=d.uniform(xs, dt), t=d.uniform(ys, dt), addend=d.normal(xs, dt, 1.0 / math.prod(ys)), **d.params(desc.C_out, desc.KH, desc.C_in, dt))
    for key, shape, t in (("y", ys, dt), ("dy", ys, dt), ("dx", xs, dt), ("dW", s["W"].shape, torch.float32),
                          ("dscale", (desc.C_out,), torch.float32), ("dshift", (desc.C_out,), torch.float32)):
        s[key] = torch.zeros(shape, dtype=t, device=d.device)
    for key, which in (("ws_fwd", B.SOL_PASS_FWD), ("ws_bwd", B.SOL_PASS_BWD)):
        s[key] = torch.empty((max(B.sol_block_workspace_bytes(desc, which), 256),), dtype=torch.uint8, device=d.device)
    return s


# ---------------------------------------------------------------------------------------------------------- pass
def run(state):
    if isinstance(state, dict):
        s = state
        B.sol_block_fwd(s["desc"], s["x"], s["W"], s["scale"], s["shift"], None, s["y"], s["ws_fwd"])
        B.sol_l1_loss_grad(s["desc"].dtype, s["y"], s["t"], s["dy"], s["y"].numel())
        B.sol_block_bwd(s["desc"], s["dy"], s["x"], s["W"], s["y"], s["dx"], s["dW"], s["dscale"], s["dshift"], s["scale"], None,
                        s["addend"], None, None, s["ws_bwd"])
        return {key: s[key] for key in ("y", "dx", "dW", "dscale", "dshift")}
    seq = state
    seq.step_prepared()
    last = seq.act[seq.ops[-1].out]
    if not seq.wl.train:
        return last
    out = {"y": last}
    if seq.wl.need_input_grad:
        out["dx"] = seq.dact[0]
    for layer, g in seq.grads.items():
        out.update({f"{key}{layer}": t for key, t in g.items()})
    return out


# ----------------------------------------------------------------------------------------------- work, tolerance
def work(case):
    """Operands of every block read once and results written once (activations between blocks are stored tensors of the
    interface), 2 * pixels * K * C_out flops per convolution and direction."""
    if case["family"] == "block":
        d = _block_desc(case)
        es = 4 if case["dtype"] == "f32" else 2
        x, y = d.N * d.H * d.W * d.C_in, d.N * d.Ho * d.Wo * d.C_out
        wt = d.C_out * d.KH * d.KW * d.C_in
        fwd = (x + wt + y) * es
        loss = 3 * y * es
        bwd = (2 * y + x + wt + 2 * x) * es + wt * 4                      # dy, y, x, W, addend, dx; dW in fp32
        return dict(bytes=fwd + loss + bwd + 5 * d.C_out * 4, flops=3 * 2 * y * d.KH * d.KW * d.C_in)
    ops, c = _ops(case)
    train = case["family"] != "infer"
    w = wl.Workload(0, case["family"], "bf16", case["n"], case["hw"], case["hw"], c, ops, None, train=train,
                    need_input_grad=case["family"] not in ("stem", "infer"))
    shp = w.tensor_shapes()
    size = {t: case["n"] * a * b * e * 2 for t, (a, b, e) in shp.items()}
    total = 0
    for o in ops:
        total += size[o.inp] + size[o.out]
        if o.op != "conv":
            continue
        wt = o.c_out * o.k * o.k * o.c_in
        total += wt * 2 + o.c_out * 8 + (size[o.res] if o.res is not None else 0)
        if train:
            total += size[o.out] + size[o.inp] + wt * 4 + o.c_out * 12     # weight gradient: dy, x -> dW (fp32)
            if o.inp != 0 or w.need_input_grad:
                total += size[o.inp] + wt * 2                              # data gradient: dx, W
            if o.res is not None:
                total += size[o.res]                                       # shortcut gradient
    if train:
        total += 3 * size[ops[-1].out]
    return dict(bytes=total, flops=w.flops_step())


def tolerance(case):
    """Measured against a pass with fp64 sums and the same roundings at the stores, and against one with the sums in another
    order.  A stored bf16 value that rounds the other way is 1e-5 of a tensor, but the path has steps: where y - t or a
    pre-activation lies within a rounding of zero the gradient of that pixel jumps.  One such pixel of millions is 8e-4 of a
    block's input gradient and up to 0.4 root mean squares of the bottleneck's (its shortcut carries the jump undiluted).  In
    a chain they add up: bottleneck 0.4 %, stage 2 2.5 %; 53 layers of inference, without steps, end 0.9 % apart.  fp32
    blocks: 6e-7."""
    if case["family"] == "block" and case["dtype"] == "f32":
        return dict(rel=2.5e-6)
    return {"block": dict(rel=4e-3, max=1.0), "stem": dict(rel=2e-3, max=1.0), "bottleneck": dict(rel=1.5e-2, max=1.0),
            "stage2": dict(rel=3e-2, max=1.0), "infer": dict(rel=3e-2, max=0.3)}[case["family"]]
