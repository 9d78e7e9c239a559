"""The work this library is used for, as cases that can be timed and compared: inference over pruned
layers and networks (single images, serving batches, throughput batches), the dense convolution
beside them, and the pruning step that makes the handles.

A case is a dict of plain values.  ``listed()`` gives the standing cases, ``draw(rng)`` one more of
the same ranges, ``prepare(case, seed)`` what a program holds before the call (device tensors, packed
handles, output buffers), ``run(state)`` one pass through the public entry points, ``work(case)`` the
bytes and operations of a pass, ``tolerance(case)`` how far another correct result may lie away.

Network shapes are those of ``workloads/`` (MobileNetV1, MobileNetV2 and ResNet-50 at 224x224 input);
weights and images are random, scaled so that activations stay of order one from layer to layer.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2109_00170_amd as alcs

# ------------------------------------------------------------------------------- networks

# MobileNetV1 blocks: channels in, channels out, input size of the depthwise layer, its stride
MBV1 = [(32, 64, 112, 1), (64, 128, 112, 2), (128, 128, 56, 1), (128, 256, 56, 2), (256, 256, 28, 1),
        (256, 512, 28, 2), (512, 512, 14, 1), (512, 512, 14, 1), (512, 512, 14, 1), (512, 512, 14, 1),
        (512, 512, 14, 1), (512, 1024, 14, 2), (1024, 1024, 7, 1)]

# MobileNetV2 blocks: channels in, expansion, channels out, input size, stride, how often
MBV2 = [(32, 1, 16, 112, 1, 1), (16, 6, 24, 112, 2, 1), (24, 6, 24, 56, 1, 1), (24, 6, 32, 56, 2, 1),
        (32, 6, 32, 28, 1, 2), (32, 6, 64, 28, 2, 1), (64, 6, 64, 14, 1, 3), (64, 6, 96, 14, 1, 1),
        (96, 6, 96, 14, 1, 2), (96, 6, 160, 14, 2, 1), (160, 6, 160, 7, 1, 2), (160, 6, 320, 7, 1, 1)]

# ResNet-50 stages: blocks, width, channels out, input size of the stage
RESNET = [(3, 64, 256, 56), (4, 128, 512, 56), (6, 256, 1024, 28), (3, 512, 2048, 14)]


def mbv2_blocks():
    return [(ci if i == 0 else co, t, co, h if i == 0 else h // s, s if i == 0 else 1)
            for ci, t, co, h, s, n in MBV2 for i in range(n)]


def resnet_convs():
    """(channels in, channels out, input size, kernel, stride, role) of the bottleneck blocks in order;
    a stage's first block has a 1x1 convolution on its shortcut."""
    out, cin = [], 64
    for stage, (blocks, width, cout, size) in enumerate(RESNET):
        h = size
        for b in range(blocks):
            s = 2 if stage and b == 0 else 1
            if b == 0:
                out.append((cin, cout, h, 1, s, "shortcut"))
            out += [(cin, width, h, 1, 1, "reduce"), (width, width, h, 3, s, "middle"),
                    (width, cout, h // s, 1, 1, "expand")]
            h, cin = h // s, cout
    return out


def prune_layers(net):
    """(channels in, channels out, size, kernel, stride) of the convolutions that a network prunes."""
    if net == "mbv1":
        return [(ci, co, h // s, 1, 1) for ci, co, h, s in MBV1]
    if net == "mbv2":
        return [l for ci, t, co, h, s in mbv2_blocks()
                for l in ([(ci, ci * t, h, 1, 1)] if t > 1 else []) + [(ci * t, co, h // s, 1, 1)]]
    return [(ci, co, h, k, s) for ci, co, h, k, s, role in resnet_convs() if role != "shortcut"]


# ------------------------------------------------------------------------------- the cases

def listed():
    return [
        # one small layer on one image: what a call costs when nothing hides it
        {"name": "layer, one image", "kind": "conv", "cin": 64, "cout": 64, "h": 56, "w": 56, "n": 1, "k": 1, "stride": 1,
         "V": 4, "sparsity": 0.5, "dtype": "f32", "act": "none", "residual": False, "shared": False},
        # the classifier head of a served model: no image, the batch is the pixel axis
        {"name": "classifier head", "kind": "conv", "cin": 2048, "cout": 1000, "h": 1, "w": 1, "n": 128, "k": 1, "stride": 1,
         "V": 8, "sparsity": 0.9, "dtype": "f32", "act": "none", "residual": False, "shared": False},
        # a 3x3 layer of a network nobody rounded to powers of two: ragged groups, odd image, stride 2,
        # every tap pruned by itself
        {"name": "3x3, odd sizes", "kind": "conv", "cin": 100, "cout": 130, "h": 57, "w": 43, "n": 9, "k": 3, "stride": 2,
         "V": 4, "sparsity": 0.8, "dtype": "f32", "act": "relu", "residual": False, "shared": False},
        # activations stored as bfloat16 beside float32 weights, odd image, shortcut added
        {"name": "bfloat16 tensors, odd sizes", "kind": "conv", "cin": 200, "cout": 330, "h": 45, "w": 37, "n": 12, "k": 1,
         "stride": 1, "V": 4, "sparsity": 0.8, "dtype": "bf16", "act": "relu6", "residual": True, "shared": False},
        # a whole MobileNetV1 on one image: on-line inference
        {"name": "MobileNetV1, one image", "kind": "mbv1", "n": 1, "V": 4, "sparsity": 0.8},
        # the same network in a serving batch
        {"name": "MobileNetV1, batch 32", "kind": "mbv1", "n": 32, "V": 4, "sparsity": 0.8},
        # the benchmark's 13 pointwise layers, each on tensors of its own
        {"name": "13 pointwise layers", "kind": "pointwise", "n": 32, "V": 4, "sparsity": 0.9, "dtype": "f32"},
        # the same in 16-bit arithmetic with the wider group that goes with it
        {"name": "13 pointwise layers, 16-bit", "kind": "pointwise", "n": 32, "V": 8, "sparsity": 0.9, "dtype": "bf16_math"},
        # MobileNetV2 with groups of very different lengths, throughput batch
        {"name": "MobileNetV2, batch 128", "kind": "mbv2", "n": 128, "V": 8, "density": 0.15},
        # ResNet-50's bottlenecks, throughput batch, the pattern shared by a filter's nine taps
        {"name": "ResNet-50, batch 64", "kind": "resnet", "n": 64, "V": 4, "sparsity": 0.8, "shared": True},
        # the dense convolution: layers that stay unpruned, and what a pruned one is compared with
        {"name": "dense 3x3", "kind": "dense", "cin": 128, "cout": 128, "h": 28, "w": 28, "n": 64, "k": 3, "stride": 1},
        # one pruning step: scores, latency-constrained selection, packing, and the new network on one image
        {"name": "pruning step, MobileNetV1", "kind": "prune", "net": "mbv1", "V": 4, "budget": 0.3},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _channels(rng, lo, hi):
    c = _log(rng, lo, hi)
    return c if rng.random() < 0.4 else max(8, (c + 4) // 8 * 8)


def _draw_once(rng):
    kind = rng.choice(["conv", "conv", "conv", "head", "pointwise", "mbv1", "mbv2", "resnet", "dense", "prune"])
    if kind == "mbv1":
        return {"kind": kind, "n": _log(rng, 1, 64), "V": rng.choice([4, 4, 8]), "sparsity": round(rng.uniform(0.7, 0.92), 3)}
    if kind == "pointwise":
        dtype = rng.choice(["f32", "bf16", "bf16_math", "bf16_math"])
        return {"kind": kind, "n": _log(rng, 1, 64), "V": rng.choice([4, 8, 16]), "sparsity": round(rng.uniform(0.7, 0.92), 3),
                "dtype": dtype}
    if kind == "mbv2":
        return {"kind": kind, "n": _log(rng, 1, 128), "V": rng.choice([1, 4, 4, 8, 8, 16]), "density": round(rng.uniform(0.1, 0.25), 3)}
    if kind == "resnet":
        return {"kind": kind, "n": _log(rng, 1, 64), "V": rng.choice([4, 4, 8]), "sparsity": round(rng.uniform(0.7, 0.9), 3),
                "shared": rng.random() < 0.5}
    if kind == "prune":
        return {"kind": kind, "net": rng.choice(["mbv1", "mbv2", "resnet"]), "V": rng.choice([4, 4, 8, 16]),
                "budget": round(rng.uniform(0.1, 0.5), 3)}
    if kind == "head":
        return {"kind": "conv", "cin": _channels(rng, 256, 4096), "cout": rng.choice([10, 100, 1000, _channels(rng, 64, 2048)]),
                "h": 1, "w": 1, "n": _log(rng, 1, 256), "k": 1, "stride": 1, "V": rng.choice([2, 4, 8, 16]),
                "sparsity": round(rng.uniform(0.7, 0.95), 3), "dtype": "f32", "act": rng.choice(["none", "relu"]),
                "residual": False, "shared": False}
    size = rng.choice([7, 14, 28, 56, 112, _log(rng, 7, 112)])
    c = {"kind": kind, "cin": _channels(rng, 16, 1024), "cout": _channels(rng, 16, 1024), "h": size,
         "w": size if rng.random() < 0.6 else max(5, int(size * rng.uniform(0.6, 1.4))), "n": _log(rng, 1, 256),
         "k": rng.choice([1, 1, 3]), "stride": rng.choice([1, 1, 1, 2])}
    if kind == "dense":
        return c
    dtype = rng.choice(["f32", "f32", "bf16", "bf16_math"]) if c["k"] == 1 else "f32"
    c.update(V=rng.choice([4, 8, 16] if dtype == "bf16_math" else [1, 2, 4, 4, 4, 8, 8, 16]),
             sparsity=round(rng.uniform(0.5, 0.95), 3), dtype=dtype, act=rng.choice(["none", "relu", "relu6"]),
             residual=rng.random() < 0.3, shared=c["k"] == 3 and rng.random() < 0.5)
    if dtype == "bf16" and c["V"] < 4:
        c["cin"] = min(c["cin"], 639)  # what that entry point takes
    return c


# A drawn single layer stays below this many bytes and operations (the networks are bounded by their batch).
MOST_BYTES, MOST_FLOPS = 6e8, {"conv": 2e10, "dense": 6e10}


def draw(rng):
    while True:
        c = _draw_once(rng)
        if c["kind"] not in MOST_FLOPS:
            return c
        w = work(c)
        if w["bytes"] <= MOST_BYTES and w["flops"] <= MOST_FLOPS[c["kind"]]:
            return c


# ------------------------------------------------------------------------------- weights and masks

def _groups(cout, V):
    return -(-cout // V)


def _kept(total, sparsity):
    return total - int(round(sparsity * total))


def zipf_counts(G, K, density):
    """Kept blocks per group rank, falling like 1 / rank, with the given mean share of K."""
    ranks = np.arange(1, G + 1, dtype=np.float64)
    lo, hi = 0.0, float(K) * G * 4 + 1.0
    for _ in range(100):
        mid = 0.5 * (lo + hi)
        if np.clip(np.rint(mid / ranks), 0, K).mean() < density * K:
            lo = mid
        else:
            hi = mid
    return np.clip(np.rint(hi / ranks), 0, K).astype(np.int64)


class _Rand:
    """Random device tensors from one seed."""

    def __init__(self, seed):
        self.gen = torch.Generator(device="cuda")
        self.gen.manual_seed(int(seed))

    def normal(self, *shape, std=1.0):
        return torch.randn(shape, generator=self.gen, device="cuda").mul_(std)

    def image(self, *shape, dtype=torch.float32):
        return torch.relu_(torch.randn(shape, generator=self.gen, device="cuda")).to(dtype)

    def weights(self, cout, cin, k, density):
        return self.normal(cout, cin, k, k, std=math.sqrt(2.0 / (cin * k * k * density)))

    def mask(self, G, cin, k, sparsity, shared=False):
        """Exactly the given share of the layer's blocks dropped, anywhere in the layer."""
        kk = 1 if shared else k * k
        total = G * cin * kk
        order = torch.randperm(total, generator=self.gen, device="cuda")
        m = torch.zeros(total, dtype=torch.uint8, device="cuda")
        m[order[:_kept(total, sparsity)]] = 1
        m = m.view(G, cin, kk)
        return (m.repeat(1, 1, k * k) if shared else m).reshape(G, cin, k, k).contiguous()

    def mask_zipf(self, G, cin, density):
        """Group lengths by zipf_counts, dealt to the groups at random."""
        counts = torch.from_numpy(zipf_counts(G, cin, density)).cuda()
        counts = counts[torch.randperm(G, generator=self.gen, device="cuda")]
        rank = torch.rand((G, cin), generator=self.gen, device="cuda").argsort(1).argsort(1)
        return (rank < counts[:, None]).to(torch.uint8).view(G, cin, 1, 1).contiguous()


def _out(size, k, s):
    return (size + 2 * ((k - 1) // 2) - k) // s + 1


class _State:
    """What run() works on; frees its handles with itself."""


# ------------------------------------------------------------------------------- prepare

def _prepare_conv(c, R):
    s = _State()
    n, k, dtype = c["n"], c["k"], torch.float32 if c["dtype"] == "f32" else torch.bfloat16
    G = _groups(c["cout"], c["V"])
    W = R.weights(c["cout"], c["cin"], k, max(0.05, 1 - c["sparsity"]))
    s.handle = alcs.alcs_pack_weights_device(W, R.mask(G, c["cin"], k, c["sparsity"], c["shared"]), c["V"])
    if c["dtype"] == "bf16_math":
        s.handle.add_bf16_weights()
    s.X = R.image(n, c["cin"], c["h"], c["w"], dtype=dtype)
    s.bias = R.normal(c["cout"], std=0.1)
    shape = (n, c["cout"], _out(c["h"], k, c["stride"]), _out(c["w"], k, c["stride"]))
    s.Y = torch.empty(shape, dtype=dtype, device="cuda")
    s.residual = R.normal(*shape).to(dtype) if c["residual"] else None
    s.stride, s.act, s.dtype = c["stride"], None if c["act"] == "none" else c["act"], c["dtype"]
    return s


def _run_conv(s):
    if s.dtype == "bf16_math":
        alcs.alcs_sparse_conv_bf16_mfma(s.handle, s.X, s.bias, s.residual, s.Y, stride=s.stride, activation=s.act)
    elif s.dtype == "bf16":
        alcs.alcs_sparse_conv_bf16(s.handle, s.X, s.bias, s.residual, s.Y, stride=s.stride, activation=s.act)
    elif s.act is None and s.residual is None:
        alcs.alcs_sparse_conv(s.handle, s.X, s.bias, s.Y, stride=s.stride)
    else:
        alcs.alcs_sparse_conv_fused(s.handle, s.X, s.bias, s.residual, s.Y, stride=s.stride, activation=s.act)
    return s.Y


def _prepare_dense(c, R):
    s = _State()
    s.W = R.weights(c["cout"], c["cin"], c["k"], 1.0)
    s.X = R.image(c["n"], c["cin"], c["h"], c["w"])
    s.bias = R.normal(c["cout"], std=0.1)
    s.Y = torch.empty((c["n"], c["cout"], _out(c["h"], c["k"], c["stride"]), _out(c["w"], c["k"], c["stride"])), device="cuda")
    s.stride = c["stride"]
    return s


def _run_dense(s):
    alcs.alcs_dense_conv(s.W, s.X, s.bias, s.Y, stride=s.stride)
    return s.Y


def _prepare_pointwise(c, R):
    s = _State()
    V, dens, dtype = c["V"], 1 - c["sparsity"], torch.float32 if c["dtype"] == "f32" else torch.bfloat16
    Ws = [R.weights(co, ci, 1, dens) for ci, co, _, _ in MBV1]
    masks = [R.mask(_groups(co, V), ci, 1, c["sparsity"]) for ci, co, _, _ in MBV1]
    handles = alcs.alcs_pack_network_device(Ws, masks, V)
    if c["dtype"] == "bf16_math":
        for h in handles:
            h.add_bf16_weights()
    s.layers = []
    for h, (ci, co, size, st) in zip(handles, MBV1):
        p = size // st
        s.layers.append((h, R.image(c["n"], ci, p, p, dtype=dtype), R.normal(co, std=0.1),
                         torch.empty((c["n"], co, p, p), dtype=dtype, device="cuda")))
    s.dtype = c["dtype"]
    return s


def _run_pointwise(s):
    if s.dtype == "f32":
        for h, X, _, Y in s.layers:
            alcs.alcs_sparse_conv(h, X, None, Y)
    elif s.dtype == "bf16":
        for h, X, b, Y in s.layers:
            alcs.alcs_sparse_conv_bf16(h, X, b, None, Y, activation="relu")
    else:
        for h, X, b, Y in s.layers:
            alcs.alcs_sparse_conv_bf16_mfma(h, X, b, None, Y, activation="relu")
    return [l[3] for l in s.layers]


def _prepare_mbv1(c, R):
    s = _State()
    n, V, dens = c["n"], c["V"], 1 - c["sparsity"]
    handles = alcs.alcs_pack_network_device([R.weights(co, ci, 1, dens) for ci, co, _, _ in MBV1],
                                            [R.mask(_groups(co, V), ci, 1, c["sparsity"]) for ci, co, _, _ in MBV1], V)
    scratch = torch.empty(max(n * ci * (h // st) ** 2 for ci, _, h, st in MBV1), device="cuda")
    s.X, s.blocks = R.image(n, 32, 112, 112), []
    for h, (ci, co, size, st) in zip(handles, MBV1):
        p = size // st
        s.blocks.append((h, R.normal(ci, 3, 3, std=math.sqrt(2 / 9)), R.normal(ci, std=0.1), R.normal(co, std=0.1),
                         torch.empty((n, co, p, p), device="cuda"), scratch[:n * ci * p * p].view(n, ci, p, p), st))
    return s


def _run_mbv1(s):
    X = s.X
    for h, D, db, b, Y, ws, st in s.blocks:
        alcs.alcs_dw_sparse_conv_fused(h, D, db, X, b, None, Y, dw_stride=st, dw_activation="relu", activation="relu",
                                       workspace=ws)
        X = Y
    return [l[4] for l in s.blocks]


def _prepare_mbv2(c, R):
    s = _State()
    n, V, dens = c["n"], c["V"], c["density"]
    blocks = mbv2_blocks()
    shapes = [l for ci, t, co, _, _ in blocks for l in ([(ci, ci * t)] if t > 1 else []) + [(ci * t, co)]]
    handles = iter(alcs.alcs_pack_network_device([R.weights(co, ci, 1, 2 * dens) for ci, co in shapes],
                                                 [R.mask_zipf(_groups(co, V), ci, dens) for ci, co in shapes], V))
    scratch = torch.empty(max(n * ci * t * (h // st) ** 2 for ci, t, _, h, st in blocks), device="cuda")
    s.X, s.blocks = R.image(n, 32, 112, 112), []
    for ci, t, co, size, st in blocks:
        mid, p = ci * t, size // st
        expand = (next(handles), R.normal(mid, std=0.1), torch.empty((n, mid, size, size), device="cuda")) if t > 1 else None
        s.blocks.append((expand, next(handles), R.normal(mid, 3, 3, std=math.sqrt(2 / 9)), R.normal(mid, std=0.1),
                         R.normal(co, std=0.1), torch.empty((n, co, p, p), device="cuda"),
                         scratch[:n * mid * p * p].view(n, mid, p, p), st, st == 1 and ci == co))
    return s


def _run_mbv2(s):
    X = s.X
    for expand, h, D, db, b, Y, ws, st, add in s.blocks:
        Z = X
        if expand is not None:
            he, be, Z = expand
            alcs.alcs_sparse_conv_fused(he, X, be, None, Z, activation="relu6")
        alcs.alcs_dw_sparse_conv_fused(h, D, db, Z, b, X if add else None, Y, dw_stride=st, dw_activation="relu6",
                                       workspace=ws)
        X = Y
    return [l[5] for l in s.blocks]


def _prepare_resnet(c, R):
    s = _State()
    n, V, dens = c["n"], c["V"], 1 - c["sparsity"]
    convs = resnet_convs()
    handles = alcs.alcs_pack_network_device(
        [R.weights(co, ci, k, dens) for ci, co, _, k, _, _ in convs],
        [R.mask(_groups(co, V), ci, k, c["sparsity"], c["shared"] and k == 3) for ci, co, _, k, _, _ in convs], V)
    s.X, s.convs = R.image(n, 64, 56, 56), []
    for h, (ci, co, size, k, st, role) in zip(handles, convs):
        p = _out(size, k, st)
        s.convs.append((role, h, R.normal(co, std=0.1), torch.empty((n, co, p, p), device="cuda"), st))
    return s


def _run_resnet(s):
    block_in = shortcut = x = s.X
    out = []
    for role, h, b, Y, st in s.convs:
        if role == "shortcut":
            alcs.alcs_sparse_conv_fused(h, block_in, b, None, Y, stride=st)
            shortcut = Y
        elif role == "expand":
            alcs.alcs_sparse_conv_fused(h, x, b, shortcut, Y, activation="relu")
            block_in = shortcut = x = Y
            out.append(Y)
        else:
            alcs.alcs_sparse_conv_fused(h, x, b, None, Y, stride=st, activation="relu")
            x = Y
    return out


def _prepare_prune(c, R):
    s = _State()
    layers, V = prune_layers(c["net"]), c["V"]
    s.V = [V] * len(layers)
    # layers of different scale compete for the blocks, as in a trained network
    scale = torch.rand(len(layers), generator=R.gen, device="cuda").mul_(0.2).add_(0.05).tolist()
    s.W = [R.normal(co, ci, k, k, std=sc) for (ci, co, _, k, _), sc in zip(layers, scale)]
    sizes = [_groups(co, V) * ci * k * k for ci, co, _, k, _ in layers]
    s.starts = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    s.scores = torch.empty(int(s.starts[-1]), device="cuda")
    s.views = [s.scores[int(a):int(b)].view(_groups(co, V), ci, k, k)
               for (ci, co, _, k, _), a, b in zip(layers, s.starts, s.starts[1:])]
    # latency tables as measured on this kind of GPU: a floor and a slope per kept weight
    steps = np.arange(11)
    s.tables = [(steps * 0.1 * (co * ci * k * k), 9.0 + 60.0 * steps / 10.0 * float(k)) for ci, co, _, k, _ in layers]
    none, every = sum(t[0] for _, t in s.tables), sum(t[-1] for _, t in s.tables)
    s.budget = none + c["budget"] * (every - none)
    flags = [torch.ones(m, dtype=torch.uint8, device="cuda") for m in sizes]
    s.workspace = torch.empty(alcs.alcs_pack_workspace_bytes(s.W, flags, s.V), dtype=torch.uint8, device="cuda")
    s.handles = alcs.alcs_pack_network_device(s.W, flags, s.V, workspace=s.workspace)
    s.X = [R.image(1, ci, h, h) for ci, _, h, _, _ in layers]
    s.Y = [torch.empty((1, co, _out(h, k, st), _out(h, k, st)), device="cuda") for _, co, h, k, st in layers]
    s.stride = [st for _, _, _, _, st in layers]
    return s


def _run_prune(s):
    for W, V, view in zip(s.W, s.V, s.views):
        alcs.alcs_block_scores(W, V, scores=view)
    N, mask, t0, t1 = alcs.alcs_project_latency(s.scores, s.starts, s.V, s.tables, 0.0, s.budget, 1e-3)
    masks = [mask[int(a):int(b)] for a, b in zip(s.starts, s.starts[1:])]
    handles = alcs.alcs_pack_network_device(s.W, masks, s.V, workspace=s.workspace)
    for h in s.handles:
        h.free()
    s.handles = handles
    # the new network once over an image (every layer on the image it sees)
    for h, X, Y, st in zip(handles, s.X, s.Y, s.stride):
        alcs.alcs_sparse_conv(h, X, None, Y, stride=st)
    return {"N": N, "mask": mask, "t0": t0, "t1": t1, "scores": s.scores, "kept": np.array([h.nnzb for h in handles]), "Y": s.Y}


PREPARE = {"conv": _prepare_conv, "dense": _prepare_dense, "pointwise": _prepare_pointwise, "mbv1": _prepare_mbv1,
           "mbv2": _prepare_mbv2, "resnet": _prepare_resnet, "prune": _prepare_prune}
RUN = {"conv": _run_conv, "dense": _run_dense, "pointwise": _run_pointwise, "mbv1": _run_mbv1, "mbv2": _run_mbv2,
       "resnet": _run_resnet, "prune": _run_prune}


def prepare(case, seed):
    state = PREPARE[case["kind"]](case, _Rand(seed))
    state.kind = case["kind"]
    return state


def run(state):
    return RUN[state.kind](state)


# ------------------------------------------------------------------------------- work and tolerance

def _conv_work(n, cin, cout, h, w, k, stride, V, kept, elem, residual=False, dw=False):
    """One sparse layer: its input, output, packed weights (and shortcut) once; two operations per kept
    weight and pixel.  dw: a depthwise 3x3 layer in front, whose output need not exist."""
    G = _groups(cout, V)
    kin = 3 if dw else k
    P = _out(h, kin, stride) * _out(w, kin, stride)
    by = elem * n * (cin * h * w + (2 if residual else 1) * cout * P) + 4 * (G + 1) + 4 * kept * (1 + V) + 4 * cout
    fl = 2.0 * n * P * V * kept
    if dw:
        by += 4 * 10 * cin
        fl += 2.0 * 9 * n * P * cin
    return by, fl


def work(case):
    c, kind = case, case["kind"]
    if kind == "dense":
        ho, wo = _out(c["h"], c["k"], c["stride"]), _out(c["w"], c["k"], c["stride"])
        K = c["cin"] * c["k"] ** 2
        return {"bytes": 4.0 * (c["n"] * (c["cin"] * c["h"] * c["w"] + c["cout"] * ho * wo) + c["cout"] * (K + 1)),
                "flops": 2.0 * c["n"] * ho * wo * c["cout"] * K}
    parts = []
    if kind == "conv":
        kk = 1 if c["shared"] else c["k"] ** 2
        kept = _kept(_groups(c["cout"], c["V"]) * c["cin"] * kk, c["sparsity"]) * (c["k"] ** 2 // kk)
        parts.append(_conv_work(c["n"], c["cin"], c["cout"], c["h"], c["w"], c["k"], c["stride"], c["V"], kept,
                                4 if c["dtype"] == "f32" else 2, c["residual"]))
    elif kind == "pointwise":
        for ci, co, h, st in MBV1:
            parts.append(_conv_work(c["n"], ci, co, h // st, h // st, 1, 1, c["V"], _kept(_groups(co, c["V"]) * ci, c["sparsity"]),
                                    4 if c["dtype"] == "f32" else 2))
    elif kind == "mbv1":
        for ci, co, h, st in MBV1:
            parts.append(_conv_work(c["n"], ci, co, h, h, 1, st, c["V"], _kept(_groups(co, c["V"]) * ci, c["sparsity"]), 4, dw=True))
    elif kind == "mbv2":
        for ci, t, co, h, st in mbv2_blocks():
            mid = ci * t
            if t > 1:
                parts.append(_conv_work(c["n"], ci, mid, h, h, 1, 1, c["V"], int(zipf_counts(_groups(mid, c["V"]), ci, c["density"]).sum()), 4))
            parts.append(_conv_work(c["n"], mid, co, h, h, 1, st, c["V"], int(zipf_counts(_groups(co, c["V"]), mid, c["density"]).sum()), 4,
                                    residual=st == 1 and ci == co, dw=True))
    elif kind == "resnet":
        for ci, co, h, k, st, role in resnet_convs():
            parts.append(_conv_work(c["n"], ci, co, h, h, k, st, c["V"], _kept(_groups(co, c["V"]) * ci * k * k, c["sparsity"]), 4,
                                    residual=role == "expand"))
    else:  # prune: weights once, scores and flags written, the kept blocks packed, one image through the layers
        for ci, co, h, k, st in prune_layers(c["net"]):
            blocks = _groups(co, c["V"]) * ci * k * k
            kept = int(c["budget"] * blocks)
            by, fl = _conv_work(1, ci, co, h, h, k, st, c["V"], kept, 4)
            parts.append((by + 4 * co * ci * k * k + 5 * blocks, fl + 2.0 * co * ci * k * k))
    return {"bytes": float(sum(p[0] for p in parts)), "flops": float(sum(p[1] for p in parts))}


def tolerance(case):
    if case.get("dtype", "f32") != "f32":
        return {"rel": 5e-3, "max": 2e-2}  # results rounded to bfloat16: a sum on the edge rounds either way
    return {"rel": 1e-5}  # float32 sums in any order; flags, counts and kept blocks are whole and the same
