"""The work that users of this library have it do, as cases that can be timed and compared.

Three kinds of program use it: a training loop that steps a stack of layers (`ConvStack`), a program that evaluates a
network forward, and a program that calls the C entry points of one layer itself through the binding.  A case is a plain
dict with a `kind`:

  step     one training step of a stack: forward, backward, momentum-SGD update (what `bench.py`, `caffenet_step.py` and
           configuration 2 of `config_bench.py` time)
  forward  the same network evaluated forward only
  layer    one convolution layer on its own: forward, data gradient, model gradient (configurations 1, 3 and 4)
  partial  the forward pass b_p images at a time (`bp_sweep.py`)
  move     batched lowering and col2im on their own (`movement_bench.py`)

Sizes are those of the repository's own configurations, tests and benchmark or generic odd ones between them.  Values:
inputs N(0,1) (U[-1,1) for the 32 x 32 images), weights and biases N(0, 0.01), upstream gradients N(0,1) -- scaled by
the power of two that keeps repeated steps in their starting distribution -- all drawn on the GPU from the seed.
"""
from __future__ import annotations

import math

import torch

from paper_1606_04487_amd import binding as B
from paper_1606_04487_amd import workloads as wl
from paper_1606_04487_amd.stack import ConvStack

STACKS = {"cifar": wl.cifar_stack, "caffenet": wl.caffenet_stack, "caffenet_full": wl.caffenet_full}
LR, MOMENTUM = 0.01, 0.9


def listed():
    return [
        # Configuration 1: the smallest layer, three calls of a few microseconds: launches and host time are what counts.
        layer("single layer f32 b8", 8, 3, 32, 32, 32, 5, 1, 2, "f32", False),
        # Configuration 2: the CIFAR-style network in the paper's precision at the paper's batch; many small launches.
        {"name": "cifar step f32 b128", "kind": "step", "stack": "cifar", "batch": 128, "dtype": "f32"},
        # The same network in bf16 at a batch that is no power of two (the last batch of an epoch, a split batch).
        {"name": "cifar step bf16 b100", "kind": "step", "stack": "cifar", "batch": 100, "dtype": "bf16"},
        # The batch sweep's smallest point: a step of one image, all latency.
        {"name": "caffenet step bf16 b1", "kind": "step", "stack": "caffenet", "batch": 1, "dtype": "bf16"},
        # A worker's share of a batch when several share it: few tiles per layer.
        {"name": "caffenet step bf16 b16", "kind": "step", "stack": "caffenet", "batch": 16, "dtype": "bf16"},
        # The benchmark's workload.
        {"name": "caffenet step bf16 b256", "kind": "step", "stack": "caffenet", "batch": 256, "dtype": "bf16"},
        # The whole training iteration: normalisation, fully connected layers and dropout among the convolutions.
        {"name": "whole step bf16 b256", "kind": "step", "stack": "caffenet_full", "batch": 256, "dtype": "bf16"},
        # The benchmark's workload in the paper's precision: batched lowering, one product a pass, col2im.
        {"name": "caffenet step f32 b256", "kind": "step", "stack": "caffenet", "batch": 256, "dtype": "f32"},
        # Evaluation of the whole network on a batch of an odd size.
        {"name": "whole forward bf16 b50", "kind": "forward", "stack": "caffenet_full", "batch": 50, "dtype": "bf16"},
        # One layer of no network in the repository: odd image, filters that fill no tile, plain (unpacked) weights.
        layer("odd layer bf16 b37", 37, 96, 30, 27, 192, 3, 1, 1, "bf16", True),
        # The b_p sweep on conv2 in the middle of its range: the explicit path's products and lowering at small sizes.
        {"name": "partial conv2 bf16 b256 bp32", "kind": "partial", "N": 256, "C": 96, "H": 27, "W": 27, "F": 256, "k": 5,
         "s": 1, "p": 2, "dtype": "bf16", "bp": 32},
        # The two data-movement steps on their own, conv4's shape.
        {"name": "lower col2im bf16 conv4 b256", "kind": "move", "N": 256, "C": 384, "H": 13, "W": 13, "F": 384, "k": 3,
         "s": 1, "p": 1, "dtype": "bf16"},
    ]


def layer(name, N, C, H, W, F, k, s, p, dtype, fused):
    return {"name": name, "kind": "layer", "N": N, "C": C, "H": H, "W": W, "F": F, "k": k, "s": s, "p": p, "dtype": dtype,
            "fused": fused}


# ---------------------------------------------------------------------------------------------- the ranges
def spread(rng, lo, hi):
    """A whole number between lo and hi, spread over the logarithm."""
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["step", "step", "step", "step", "forward", "layer", "layer", "layer", "partial", "move"])
    if kind == "step":
        stack, dtype, most = rng.choice([("cifar", "f32", 512), ("cifar", "bf16", 512), ("caffenet", "bf16", 256),
                                         ("caffenet", "bf16", 256), ("caffenet_full", "bf16", 256), ("caffenet", "f32", 200)])
        return {"kind": "step", "stack": stack, "batch": spread(rng, 2, most), "dtype": dtype}
    if kind == "forward":
        return {"kind": "forward", "stack": rng.choice(["cifar", "caffenet", "caffenet_full"]), "batch": spread(rng, 2, 256),
                "dtype": "bf16"}
    if kind == "layer":
        dtype = rng.choice(["bf16", "bf16", "f32"])
        if rng.random() < 0.25:      # a first layer: few channels, a long stride
            k = rng.choice([7, 8, 11])
            c = layer("", spread(rng, 1, 128), 3, rng.randint(64, 227), rng.randint(64, 227), rng.choice([32, 48, 64, 96]),
                      k, 4, 0, dtype, dtype == "bf16")
        else:
            k = rng.choice([1, 3, 3, 5])
            C = rng.choice([3, 32, 64, 96, 128, 192, 256, 384])
            F = rng.choice([32, 64, 96, 128, 192, 200, 256, 384])
            H = rng.randint(max(7, k), 32)
            c = layer("", spread(rng, 1, 128), C, H, rng.randint(max(7, k), 32), F, k, 1, k // 2, dtype, dtype == "bf16")
        del c["name"]
        return c
    if kind == "partial":
        N = spread(rng, 32, 256)
        return {"kind": "partial", "N": N, "C": 96, "H": 27, "W": 27, "F": 256, "k": 5, "s": 1, "p": 2, "dtype": "bf16",
                "bp": spread(rng, 8, N)}
    k, s = rng.choice([(3, 1), (3, 1), (5, 1), (11, 4)])
    C = 3 if s == 4 else rng.choice([32, 64, 96, 256, 384])
    H = rng.randint(100, 227) if s == 4 else rng.randint(8, 32)
    return {"kind": "move", "N": spread(rng, 4, 128), "C": C, "H": H, "W": H + rng.randint(0, 3), "F": 96, "k": k, "s": s,
            "p": 0 if s == 4 else k // 2, "dtype": rng.choice(["bf16", "f32"])}


# ---------------------------------------------------------------------------------------------- state
def code(dtype):
    return B.BF16 if dtype == "bf16" else B.F32


def normal(g, shape, dtype, sigma=1.0):
    return (torch.randn(shape, generator=g, device="cuda", dtype=torch.float32) * sigma).to(B.torch_dtype(dtype))


def stack_layers(case):
    return STACKS[case["stack"]](case["batch"])


def prepare(case, seed):
    g = torch.Generator(device="cuda").manual_seed(int(seed))
    dt = code(case["dtype"])
    st = {"kind": case["kind"]}
    if case["kind"] in ("step", "forward"):
        layers = stack_layers(case)
        net = ConvStack(layers, dtype=dt, ceil_mode=case["stack"] == "cifar", skip_first_dgrad=True)
        L = layers[0]
        shape = (L.N, L.C, L.H, L.W)
        if case["stack"] == "cifar":
            X = (2.0 * torch.rand(shape, generator=g, device="cuda") - 1.0).to(net.tdtype)
        else:
            X = normal(g, shape, dt)
        # weights that bf16 can hold, as a program has them that starts both precisions from one checkpoint
        Ws = [normal(g, w.shape, dt, 0.01).float() for w in net.W]
        bs = [normal(g, b.shape, B.F32, 0.01) for b in net.b]
        net.set_parameters(Ws, bs)
        st.update(net=net, X=X)
        if case["kind"] == "step":
            st["dOut"] = normal(g, net.output_shape(), dt, wl.step_upstream_scale(L.N))
        return st
    flags = B.FLAG_FUSED if case.get("fused") else 0
    d = B.conv_desc(case["N"], case["C"], case["H"], case["W"], case["F"], case["k"], case["k"], case["s"], case["p"], dt, flags)
    X = normal(g, (d.N, d.C, d.H, d.W), dt)
    st.update(desc=d, X=X)
    if case["kind"] == "move":
        st["ld"] = B.conv_dhat_ld(d)
        st["Dhat"] = torch.empty((d.C * d.kh * d.kw, st["ld"]), dtype=X.dtype, device="cuda")
        st["dX"] = torch.empty_like(X)
        return st
    ho, wo = B.conv_output_dims(d)
    st["W"] = normal(g, (d.F, d.C, d.kh, d.kw), dt, 0.01)
    st["b"] = normal(g, (d.F,), B.F32, 0.01)
    st["Y"] = torch.empty((d.N, d.F, ho, wo), dtype=X.dtype, device="cuda")
    if case["kind"] == "partial":
        st["bp"] = case["bp"]
        sub = B.conv_desc(case["bp"], d.C, d.H, d.W, d.F, d.kh, d.kw, d.stride_h, d.pad_h, dt, flags)
        st["ws"] = B.alloc_workspace(sub, B.PASS_FORWARD)
        return st
    st["dY"] = normal(g, st["Y"].shape, dt)
    st["dX"] = torch.empty_like(X)
    st["dW"] = torch.empty(st["W"].shape, dtype=torch.float32, device="cuda")
    st["db"] = torch.empty((d.F,), dtype=torch.float32, device="cuda")
    st["ws"] = [B.alloc_workspace(d, p) for p in (B.PASS_FORWARD, B.PASS_BACKWARD_DATA, B.PASS_BACKWARD_WEIGHTS)]
    return st


# ---------------------------------------------------------------------------------------------- one pass
def run(st):
    kind = st["kind"]
    if kind == "step":
        net = st["net"]
        out = net.step(st["X"], st["dOut"], LR, MOMENTUM)
        got = {"out": out, "W": net.W, "b": net.b}
        # In bf16 the stack's gradients are no measure of anything: a forward sum in another order rounds some outputs the
        # other way, a few ReLUs and pool winners change sides, and the gradients of all layers before them move by 2 to
        # 8 % of their norm (see tolerance()).  There the updated parameters stand for the step, and the `layer` cases,
        # whose inputs are given, hold the gradients themselves.
        if net.dtype == B.F32:
            got.update(dW=net.dW, db=net.db, VW=net.VW, Vb=net.Vb)
        return got
    if kind == "forward":
        return st["net"].forward(st["X"])
    d = st["desc"]
    if kind == "partial":
        return B.conv_forward_partial(d, st["bp"], st["X"], st["W"], st["b"], st["Y"], st["ws"])
    if kind == "move":
        D = B.lower(d, st["X"], st["Dhat"], st["ld"])
        return {"Dhat": D, "dX": B.col2im(d, D, st["dX"], st["ld"])}
    Y = B.conv_forward(d, st["X"], st["W"], st["b"], st["Y"], st["ws"][0])
    dX = B.conv_backward_data(d, st["dY"], st["W"], st["dX"], st["ws"][1])
    dW, db = B.conv_backward_weights(d, st["X"], st["dY"], st["dW"], st["db"], st["ws"][2])
    return {"Y": Y, "dX": dX, "dW": dW, "db": db}


# ---------------------------------------------------------------------------------------------- what a pass needs
def work(case):
    e = 2 if case["dtype"] == "bf16" else 4
    if case["kind"] in ("step", "forward"):
        layers = stack_layers(case)
        first, last = layers[0], layers[-1]
        out_plane = last.Ho * last.Wo
        if last.pool_after:
            po = [B.pool_output_dim(n, 3, 2, case["stack"] == "cifar") for n in (last.Ho, last.Wo)]
            out_plane = po[0] * po[1]
        x, y = first.N * first.C * first.H * first.W * e, last.N * last.F * out_plane * e
        params = sum(L.F * L.K + L.F for L in layers)
        flops = sum(L.gemm_flops for L in layers)
        if case["kind"] == "forward":
            return {"bytes": x + y + params * e, "flops": flops}
        # image and upstream gradient in, output out; every layer's output kept by the forward pass and read by the
        # backward one; masters and velocities read and written, gradients written, in fp32
        kept = sum(L.N * L.F * L.Ho * L.Wo for L in layers) * e
        return {"bytes": x + 2 * y + 2 * kept + 20 * params, "flops": 3 * flops - first.gemm_flops}
    s, p, k = case["s"], case["p"], case["k"]
    ho, wo = (case["H"] + 2 * p - k) // s + 1, (case["W"] + 2 * p - k) // s + 1
    x = case["N"] * case["C"] * case["H"] * case["W"]
    y = case["N"] * case["F"] * ho * wo
    w = case["F"] * case["C"] * k * k
    gemm = 2 * y * case["C"] * k * k
    if case["kind"] == "move":
        dhat = case["C"] * k * k * ((case["N"] * ho * wo + 63) // 64 * 64)
        return {"bytes": 2 * (x + dhat) * e, "flops": x * min(k * k, (-(-k // s)) ** 2)}
    if case["kind"] == "partial":
        return {"bytes": (x + y + w) * e, "flops": gemm}
    return {"bytes": (3 * x + 3 * y + 2 * w) * e + 4 * w, "flops": 3 * gemm}


def tolerance(case):
    """Largest relative error of another correct implementation at the same precision, about four times what was measured.

    bf16: fused against explicit path, i.e. other orders of the fp32 sums and, in the data gradient, one more rounding:
    3e-5 for a forward pass on given inputs, 1.7e-3 for a col2im against fp64, 2.4e-3 for the output of the whole network
    (bf16 roundings that fall the other way, carried through eight layers).  The stack's gradients differ by 0.016 (last
    convolution) to 0.076 (first) between the two paths, at every batch: they are not among a bf16 step's outputs.
    f32 against the same arithmetic in fp64: 2.4e-7 for a layer; for a step 1e-6 in the output and 5e-3 in the gradients,
    because there, too, pool winners and ReLUs change sides where two values differ in the last bits."""
    if case["dtype"] == "bf16":
        return {"rel": 1e-2}
    return {"rel": 2e-2} if case["kind"] == "step" else {"rel": 1e-5}
