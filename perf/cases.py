"""Timed cases of the executor: the calls a program that serves dynamic
networks makes, from one small fp32 network to a whole early-exit ResNet-50
batch, with the layers and routing steps between them on their own.

listed() holds the cases that are always timed, draw(rng) gives one more of
the same ranges; prepare / run / work / tolerance / exact take a case apart:
what a program has in hand before the call, one pass through the public entry
points, the bytes and operations that pass cannot do without, how far another
correct implementation may be off, and the result in 64 bits.
"""

import ctypes
import functools
import math

import numpy as np
import torch
import torch.nn.functional as F

from paper_2307_04963_amd import _lib, runtime
from workloads import configs


def listed():
    return [
        # the smallest whole call: an early-exit MLP in fp32, where launches and latency count
        {"name": "mlp_exit_b64", "kind": "plan", "net": "mlp_exit", "batch": 64},
        # the largest whole call: the early-exit ResNet-50 of the benchmark, in its device host mode
        {"name": "resnet50_exit_b256", "kind": "plan", "net": "resnet50_exit", "batch": 256},
        # the ImageNet stem with its max-pool, every image of a batch
        {"name": "stem_pool_224", "kind": "stem", "n": 256, "H": 224, "W": 224},
        # ResNet-50 stage 1 / ResNet-18 stage 1: 3x3, 64 channels, large images, whole batch, with a residual
        conv("conv3_c64_56", n=256, H=56, W=56, cin=64, cout=64, k=3, stride=1, residual=True),
        # ResNet-50 stage 2: 3x3, 128 channels, the odd number of images that an exit leaves
        conv("conv3_c128_28", n=183, H=28, W=28, cin=128, cout=128, k=3, stride=1, residual=False),
        # SkipNet's first stage: narrow 3x3 layers with a residual
        conv("conv3_c16_32", n=2048, H=32, W=32, cin=16, cout=16, k=3, stride=1, residual=True),
        # the first 3x3 layer of a stage: stride 2, twice the channels
        conv("conv3_s2_128_256", n=529, H=16, W=16, cin=128, cout=256, k=3, stride=2, residual=False),
        # ResNet-18 stage 4: deep 3x3 layers on 4x4 images, few rows left after three exits
        conv("conv3_c512_4", n=255, H=4, W=4, cin=512, cout=512, k=3, stride=1, residual=True),
        # ResNet-50 stage 3: the 1x1 reduction at the head of a bottleneck
        conv("conv1_1024_256_14", n=107, H=14, W=14, cin=1024, cout=256, k=1, stride=1, residual=False),
        # a bottleneck's last 1x1 layer and the next block's first one, at ResNet-50 stage 1
        {"name": "pair_64_256_64_56", "kind": "pair", "n": 256, "H": 56, "W": 56, "cin": 64, "c3": 256, "c1": 64,
         "residual": True},
        # the cell of the bounded loop: a bf16 linear layer with GELU over 4096 samples
        {"name": "linear_2048_1024", "kind": "conv", "n": 4096, "H": 1, "W": 1, "cin": 2048, "cout": 1024, "k": 1,
         "stride": 1, "residual": False, "act": 2},
        # the partition of a decision that carries sample ids, far beyond one workgroup
        {"name": "compact_ids_2^26", "kind": "compact", "n": 1 << 26, "ids": True},
    ]


def conv(name, n, H, W, cin, cout, k, stride, residual, act=1):
    return {"name": name, "kind": "conv", "n": n, "H": H, "W": W, "cin": cin, "cout": cout, "k": k, "stride": stride,
            "residual": residual, "act": act}


MOST_FLOPS, MOST_BYTES = 1.2e11, 1.2e9       # of one drawn layer: below the largest listed whole call


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["plan", "plan", "stem", "pair", "conv3", "conv3", "conv3", "conv3_s2", "conv1", "conv1", "linear",
                       "compact"])
    if kind == "plan":
        net, most = rng.choice([("mlp_exit", 64), ("resnet50_exit", 256)])
        return {"kind": "plan", "net": net, "batch": _log_int(rng, 1, most)}
    if kind == "compact":
        return {"kind": "compact", "n": _log_int(rng, 1 << 8, 1 << 26), "ids": rng.random() < 0.5}
    if kind == "linear":
        return {"kind": "conv", "n": _log_int(rng, 16, 4096), "H": 1, "W": 1, "cin": rng.choice([512, 768, 1024, 2048]),
                "cout": rng.choice([512, 1024, 2048]), "k": 1, "stride": 1, "residual": False, "act": rng.choice([0, 2])}
    if kind == "stem":
        c = {"kind": "stem", "H": rng.randrange(64, 225), "W": 8 * rng.randrange(8, 29)}
    elif kind == "pair":
        s = rng.choice([56, 28, rng.randrange(7, 57)])
        c3 = rng.choice([256, 512])
        c = {"kind": "pair", "H": s, "W": s, "cin": 64 if c3 == 256 else 128, "c3": c3, "c1": c3 // 4,
             "residual": rng.random() < 0.8}
    else:
        k = 1 if kind == "conv1" else 3
        cin = rng.choice([16, 32, 64, 64, 128, 128, 256, 512] if k == 3 else [64, 128, 256, 512, 1024])
        cout = rng.choice([cin // 2, 2 * cin, cin // 4, 4 * cin]) if k == 1 else 2 * cin if kind == "conv3_s2" else cin
        s = rng.choice([56, 32, 28, 16, 14, 8, 7, 4, rng.randrange(4, 57)])
        c = {"kind": "conv", "H": s, "W": s, "cin": cin, "cout": min(2048, max(16, cout)), "k": k,
             "stride": 2 if kind == "conv3_s2" else 1, "residual": kind != "conv3_s2" and rng.random() < 0.5, "act": 1}
    w = work(dict(c, n=1))
    most = max(1, int(min(MOST_FLOPS / w["flops"], MOST_BYTES / w["bytes"], 2048 if c["H"] <= 32 else 256)))
    return dict(c, n=_log_int(rng, 1, most))


# ---- what a program has in hand before the call ---------------------------

@functools.lru_cache(maxsize=None)
def _network(name):
    return configs.build(name)


def _uniform(g, shape, lo, hi):
    return torch.rand(shape, generator=g, device="cuda") * (hi - lo) + lo


def _layer(g, cin, cout, k):
    """Weights of one layer (Kaiming-uniform, bf16) as the program keeps them: packed, with the folded BatchNorm's scale and shift."""
    b = math.sqrt(6.0 / (k * k * cin))
    w = _uniform(g, (cout, k, k, cin), -b, b).bfloat16()
    bits = w.view(torch.int16).cpu().numpy().view(np.uint16)
    packed = torch.from_numpy(runtime.pack_conv_weights(bits).view(np.int16)).cuda()
    return {"w": w, "packed": packed, "scale": _uniform(g, (cout,), 0.5, 1.5), "shift": _uniform(g, (cout,), -0.3, 0.3)}


def _inputs(case, seed):
    g = torch.Generator(device="cuda").manual_seed(1_000_003 * (seed % (1 << 31)) + 17)
    normal = lambda *shape: torch.randn(shape, generator=g, device="cuda")  # noqa: E731
    kind = case["kind"]
    if kind == "plan":
        wl = _network(case["net"])
        x = normal(case["batch"], *wl.in_shape)
        return {"x": x if wl.in_dtype == "f32" else x.bfloat16()}
    if kind == "compact":
        n = case["n"]
        s = {"flags": (torch.rand(n, generator=g, device="cuda") < 0.5).to(torch.uint8), "orig": None}
        if case["ids"]:
            s["orig"] = torch.randperm(n, generator=g, device="cuda").to(torch.int32)
        return s
    n, H, W = case["n"], case["H"], case["W"]
    if kind == "stem":
        return {"x": normal(n, H, W, 3).bfloat16(), "l": _layer(g, 3, 64, 7)}
    x = normal(n, H, W, case["cin"])
    # between layers: what a ReLU leaves; a bounded loop's cell reads states of both signs
    x = (F.relu(x) if H > 1 else x).bfloat16()
    if kind == "pair":
        res = F.relu(normal(n, H, W, case["c3"])).bfloat16() if case["residual"] else None
        return {"x": x, "res": res, "l3": _layer(g, case["cin"], case["c3"], 1), "l1": _layer(g, case["c3"], case["c1"], 1)}
    Ho, Wo = _out(H, case), _out(W, case)
    res = F.relu(normal(n, Ho, Wo, case["cout"])).bfloat16() if case["residual"] else None
    return {"x": x, "res": res, "l": _layer(g, case["cin"], case["cout"], case["k"])}


def _out(size, case):
    k = case["k"]
    return (size + 2 * (k // 2) - k) // case["stride"] + 1


def prepare(case, seed):
    s = _inputs(case, seed)
    s["case"] = dict(case)
    if case["kind"] == "plan":
        wl = _network(case["net"])
        s["plan"] = runtime.Plan.from_workload(wl, case["batch"])
        s["plan"].set_host_mode("device")
        s["logits"], s["records"], _ = s["plan"].outputs(case["batch"])
    elif case["kind"] == "compact":
        n = case["n"]
        # lists of the largest length; entries past the counts stay as they are here
        s["lists"] = [torch.zeros(n, dtype=torch.int32, device="cuda") if k % 2 == 0 or case["ids"] else None for k in range(4)]
        s["counts"] = torch.zeros(2, dtype=torch.int32, device="cuda")
        s["workspace"] = torch.zeros(max(8, _lib.lib.dycl_op_compact_workspace(n)), dtype=torch.uint8, device="cuda")
    elif case["kind"] == "conv":
        c = case
        s["y"] = torch.empty((c["n"], _out(c["H"], c), _out(c["W"], c), c["cout"]), dtype=torch.bfloat16, device="cuda")
        nb = runtime.conv_workspace_bytes(c["n"], c["H"], c["W"], c["cin"], c["cout"], c["k"], c["stride"], c["k"] // 2)
        s["workspace"] = torch.empty(nb, dtype=torch.uint8, device="cuda") if nb else None
    elif case["kind"] == "stem":
        Hp, Wp = ((_out(v, {"k": 7, "stride": 2}) - 1) // 2 + 1 for v in (case["H"], case["W"]))
        s["y"] = torch.empty((case["n"], Hp, Wp, 64), dtype=torch.bfloat16, device="cuda")
    return s


# ---- one pass --------------------------------------------------------------

def run(s):
    c = s["case"]
    if c["kind"] == "plan":
        s["plan"].run(s["x"], None, s["logits"], s["records"])
        return {"logits": s["logits"], "records": s["records"]}
    if c["kind"] == "conv":
        w = s["l"]
        return runtime.conv(s["x"], w["packed"], c["cout"], c["k"], c["stride"], c["k"] // 2, w["scale"], w["shift"], s["res"],
                            c["act"], out=s["y"], workspace=s["workspace"])
    if c["kind"] == "stem":
        w = s["l"]
        return runtime.conv_maxpool(s["x"], w["packed"], 64, 7, 2, 3, w["scale"], w["shift"], 1, out=s["y"])
    if c["kind"] == "pair":
        a, b = s["l3"], s["l1"]
        return runtime.conv_pair(s["x"], a["packed"], a["scale"], a["shift"], s["res"], c["c3"], b["packed"], b["scale"],
                                 b["shift"], c["c1"])
    ptr = lambda t: None if t is None else ctypes.c_void_p(t.data_ptr())  # noqa: E731
    ws = s["workspace"]
    _lib.check(_lib.lib.dycl_op_compact(ptr(s["flags"]), ptr(s["orig"]), c["n"], *(ptr(t) for t in s["lists"]), ptr(s["counts"]),
                                        ptr(ws), ws.numel(), ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)))
    return [t for t in s["lists"] + [s["counts"]] if t is not None]


# ---- what a pass cannot do without -----------------------------------------

def work(case):
    kind = case["kind"]
    if kind == "compact":
        # flags (and ids) read, one index (and one id) written for each row
        return {"bytes": case["n"] * (13 if case["ids"] else 5), "flops": 0}
    if kind == "plan":
        B, wl = case["batch"], _network(case["net"])
        weights = sum((2 if t.dtype == "bf16" else 4) * t.value.size for t in wl.tensors.values())
        item = 4 if wl.in_dtype == "f32" else 2
        outer = B * (item * int(np.prod(wl.in_shape)) + 4 * wl.n_out + 16) + weights
        return {"bytes": outer, "flops": B * _network_flops(case["net"])}
    n, H, W = case["n"], case["H"], case["W"]
    if kind == "stem":
        Ho, Wo = (_out(v, {"k": 7, "stride": 2}) for v in (H, W))
        pooled = ((Ho - 1) // 2 + 1) * ((Wo - 1) // 2 + 1)
        return {"bytes": 2 * n * (H * W * 3 + pooled * 64) + 2 * 64 * 147, "flops": 2 * n * Ho * Wo * 64 * 147}
    if kind == "pair":
        cin, c3, c1, px = case["cin"], case["c3"], case["c1"], n * H * W
        return {"bytes": 2 * px * (cin + (2 if case["residual"] else 1) * c3 + c1) + 2 * c3 * (cin + c1),
                "flops": 2 * px * c3 * (cin + c1)}
    K, px = case["k"] ** 2 * case["cin"], n * _out(H, case) * _out(W, case)
    return {"bytes": 2 * (n * H * W * case["cin"] + (2 if case["residual"] else 1) * px * case["cout"] + K * case["cout"]),
            "flops": 2 * px * K * case["cout"]}


@functools.lru_cache(maxsize=None)
def _network_flops(name):
    """Operations of one sample of average depth: a stage counts with the share of samples that reach it (measured over a
    calibrated network's own input distribution: see the branch counts of the benchmark's batch)."""
    arch = _network(name).arch
    if name == "mlp_exit":
        return sum(2 * t["cin"] * t["cout"] for t in arch["layers"]) + sum(2 * h["cin"] * arch["n_classes"] for h in arch["heads"])
    size = (arch["input"][0] + 1) // 2
    flops, size = 2 * size * size * 64 * 147, (size + 1) // 2
    for share, blocks, head in zip((1.0, 0.71, 0.42, 0.20), arch["stages"], arch["heads"]):
        for b in blocks:
            for layer in ("proj", "c1", "c2", "c3"):
                c = b[layer]
                if c is not None:
                    out = -(-size // b["stride"]) if layer != "c1" else size
                    flops += share * 2 * out * out * c["k"] ** 2 * c["cin"] * c["cout"]
            size = -(-size // b["stride"])
        flops += share * 2 * head["cin"] * arch["n_classes"]
    return flops


# ---- how far another correct implementation may be off ----------------------

def tolerance(case):
    if case["kind"] == "compact":
        return "exact"
    if case["kind"] == "plan":
        if case["net"] == "mlp_exit":
            return {"rel": 2e-6, "max": 2e-5, "differ": 0.0}        # fp32 sums of at most 784 terms in another order: 2e-7
        # 50 bf16 layers: a rounding that falls the other way travels through all that follow
        return {"rel": 0.03, "max": 0.5, "differ": 0.01}
    # one rounding to bf16 at the end of an fp32 sum (the second layer of a pair reads the first's rounded output); against
    # 64 bits that is 1.7e-3 in the 2-norm, and half a unit in the last place of 8 bits at most
    return {"rel": 7e-3, "max": 3.2e-2}


# ---- the result in 64 bits ---------------------------------------------------

ACT = {0: lambda v: v, 1: torch.relu, 2: lambda v: F.gelu(v)}


def _conv64(x, layer, k, stride, res, act):
    """A convolution as one float64 product per tap, over the pixels that the tap reads."""
    n, H, W, cin = x.shape
    pad = k // 2
    Ho, Wo = (H + 2 * pad - k) // stride + 1, (W + 2 * pad - k) // stride + 1
    xp = F.pad(x, (0, 0, pad, pad, pad, pad)) if pad else x
    y = torch.zeros((n * Ho * Wo, layer["w"].shape[0]), dtype=torch.float64, device=x.device)
    for r in range(k):
        for c in range(k):
            tap = xp[:, r:r + stride * (Ho - 1) + 1:stride, c:c + stride * (Wo - 1) + 1:stride]
            y.addmm_(tap.reshape(-1, cin).double(), layer["w"][:, r, c].double().t().contiguous())
    y = y.mul_(layer["scale"].double()).add_(layer["shift"].double()).view(n, Ho, Wo, -1)
    return ACT[act](y if res is None else y.add_(res.double()))


def _mlp64(case, x):
    wl = _network(case["net"])
    W = {k: torch.from_numpy(np.asarray(t.value, np.float64)).cuda() for k, t in wl.tensors.items()}
    arch, h = wl.arch, x.double()
    logits = torch.zeros((x.shape[0], arch["n_classes"]), dtype=torch.float64, device=x.device)
    left = torch.ones(x.shape[0], dtype=torch.bool, device=x.device)
    for i, (layer, head) in enumerate(zip(arch["layers"], arch["heads"])):
        h = torch.relu(h @ W[layer["name"] + ".w"].t() + W[layer["name"] + ".b"])
        z = h @ W[head["name"] + ".w"].t() + W[head["name"] + ".b"]
        logits = torch.where(left[:, None], z, logits)
        sure = torch.softmax(z / W[head["name"] + ".T"], dim=1).amax(dim=1) >= arch["tau"]
        left = left & ~sure
    return logits


def exact(case, seed):
    s = _inputs(case, seed)
    kind = case["kind"]
    if kind == "compact":
        return None
    if kind == "plan":
        # a network that stores bf16 between its layers and branches on them has no result in 64 bits
        return {"logits": _mlp64(case, s["x"]), "records": None} if case["net"] == "mlp_exit" else None
    if kind == "pair":
        y3 = _conv64(s["x"], s["l3"], 1, 1, s["res"], 1)
        return y3, _conv64(y3.bfloat16(), s["l1"], 1, 1, None, 1)
    if kind == "stem":
        y = _conv64(s["x"], s["l"], 7, 2, None, 1).permute(0, 3, 1, 2)
        return F.max_pool2d(y, 3, 2, 1).permute(0, 2, 3, 1).contiguous()
    return _conv64(s["x"], s["l"], case["k"], case["stride"], s["res"], case["act"])
