"""What a program that serves or prepares a decoder with this library's weights has it do, as measurable cases.

A case is one pass through the public entry points, of one of four kinds:

  linear   one plain matmul call: a single projection
  blocks   the linear half of `layers` decoder blocks, each rms-norm + qkv, append of the new K/V rows to the layer's
           cache, attention output + residual, rms-norm + gate/up with the gated product, down + residual; `vocab`
           > 0 adds the vocabulary projection.  Attention is no part of the library: its result is an input
           (`context`).  `graph`: the pass is captured once and replayed, as a serving loop does with its fixed batch;
           else every call is made from Python, as for a prompt of any length
  plain    the four matmuls of `layers` blocks on bfloat16, which has no fused entry point
  pack     a weight matrix quantised, and dequantised again for inspection

`format` is the member of the number format's family, `group` the weights per scale and bias, M the rows of
activations (sequences of a decoded batch, or tokens of a prompt).
"""
import math

import torch

import paper_2403_20041_amd as e0m4

EPS = 1e-5
MOST = 640_000_000_000      # products of weights and rows in one pass, at most: the 14B layer's prompt of 2048
DEVICE = "cuda"


def blocks(name, M, hidden, qkv, ff, group=128, layers=1, graph=False, vocab=0, format="e0m4", kind="blocks"):
    return {"name": name, "kind": kind, "format": format, "M": M, "hidden": hidden, "qkv": qkv, "ff": ff, "group": group,
            "layers": layers, "graph": graph, "vocab": vocab}


def listed():
    return [
        # the smallest call: one projection of the smallest model for one token, launched by itself
        {"name": "projection one token", "kind": "linear", "format": "e0m4", "M": 1, "N": 2048, "K": 2048, "group": 128},
        # the headline workload: one decoding step of the 28-layer 6B model for a single user
        blocks("decode 6B b1", 1, 4096, 4608, 13696, layers=28, graph=True),
        # a few users on the 14B model with the finer group of 64 (six of its layers)
        blocks("decode 14B g64 b6", 6, 5120, 15360, 13696, group=64, layers=6, graph=True),
        # a full small batch on the 2B model with its vocabulary projection
        blocks("decode 2B b16", 16, 2048, 2560, 16384, layers=18, graph=True, vocab=256000),
        # 8-bit weights where 4 bits lose too much, three users (eight layers)
        blocks("decode 6B 8-bit b3", 3, 4096, 4608, 13696, layers=8, graph=True, format="e0m8"),
        # bfloat16 models, decoded for a handful of users
        blocks("decode 6B bf16 b5", 5, 4096, 4608, 13696, layers=4, graph=True, format="bf16", kind="plain"),
        # a chat turn: a prompt of a few dozen tokens
        blocks("prompt 45 6B", 45, 4096, 4608, 13696, layers=4),
        # a ragged prompt of ordinary length with the finest group
        blocks("prompt 317 2B g32", 317, 2048, 2560, 16384, group=32, layers=2),
        # the benchmark's prompts
        blocks("prompt 1024 6B", 1024, 4096, 4608, 13696, layers=2),
        blocks("prompt 2048 14B g64", 2048, 5120, 15360, 13696, group=64),
        # a bfloat16 prompt of odd length
        blocks("prompt 700 6B bf16", 700, 4096, 4608, 13696, format="bf16", kind="plain"),
        # preparing a model: its largest matrix
        {"name": "pack 27392 x 4096", "kind": "pack", "format": "e0m4", "N": 27392, "K": 4096, "group": 128},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["linear", "blocks", "blocks", "blocks", "plain", "pack"])
    if kind == "pack":
        fmt = rng.choice(["e0m4", "e0m4", "e0m3", "e0m8", "bf16"])
        group = rng.choice([64, 128] if fmt == "e0m8" else [32, 64, 128])
        return {"kind": kind, "format": fmt, "N": _log_int(rng, 1500, 28000), "K": 128 * _log_int(rng, 12, 100), "group": group}
    if kind == "linear":
        fmt = rng.choice(["e0m4", "e0m4", "e0m8", "bf16"])
        group = rng.choice([64, 128] if fmt == "e0m8" else [32, 64, 128])
        step = 128 if fmt == "e0m8" else max(64, group)
        N, K = 8 * _log_int(rng, 200, 3500), step * _log_int(rng, 1500 // step, 14000 // step)
        return {"kind": kind, "format": fmt, "M": min(_log_int(rng, 1, 2048), MOST // (N * K)), "N": N, "K": K, "group": group}
    group = rng.choice([64, 128])
    hidden = 128 * _log_int(rng, 12, 44)
    ff = 128 * int(hidden * rng.uniform(2.5, 4.5) / 128)
    qkv = hidden + 256 * rng.randint(1, 2 * hidden // 256)
    per_layer = hidden * (qkv + hidden + 3 * ff)
    M = min(_log_int(rng, 1, 2048), MOST // per_layer)
    fmt = "bf16" if kind == "plain" else rng.choice(["e0m4", "e0m4", "e0m8"])
    graph = M <= 16 or (M <= 64 and rng.random() < 0.5)
    layers = rng.randint(2, 8) if graph else (rng.randint(1, 2) if M * per_layer < 1.5e11 else 1)
    return {"kind": kind, "format": fmt, "M": M, "hidden": hidden, "qkv": qkv, "ff": ff, "group": group, "layers": layers,
            "graph": graph, "vocab": 8 * _log_int(rng, 4000, 19000) if graph and kind == "blocks" and rng.random() < 0.3 else 0}


class Inputs:
    """Seeded device-side inputs: weights ~ N(0, 0.02) with row scales in [0.5, 2], activations ~ N(0, 1) of which one
    channel in a hundred is an outlier (x 20), rms-norm weights around one."""

    def __init__(self, seed, dtype):
        self.gen = torch.Generator(device=DEVICE)
        self.gen.manual_seed(int(seed) + 1)
        self.dtype = dtype

    def weights(self, N, K):
        W = torch.randn((N, K), generator=self.gen, device=DEVICE, dtype=self.dtype)
        rows = torch.rand((N, 1), generator=self.gen, device=DEVICE, dtype=torch.float32) * 1.5 + 0.5
        return W.mul_((rows * 0.02).to(self.dtype))

    def activations(self, *shape):
        X = torch.randn(shape, generator=self.gen, device=DEVICE, dtype=torch.float32)
        K = shape[-1]
        X[..., torch.randperm(K, generator=self.gen, device=DEVICE)[:max(1, K // 100)]] *= 20.0
        return X.to(self.dtype)

    def norm_weight(self, K):
        return (1.0 + 0.1 * torch.randn(K, generator=self.gen, device=DEVICE, dtype=torch.float32)).to(self.dtype)


QUANTIZE = {"e0m4": e0m4.e0m4_quantize, "e0m3": e0m4.e0m3_quantize, "e0m8": e0m4.e0m8_quantize, "bf16": e0m4.e0m4_bf16_quantize}


def _dtype(case):
    return torch.bfloat16 if case["format"] == "bf16" else torch.float16


class Linear:
    """A quantised weight matrix as a program keeps it."""

    def __init__(self, inputs, fmt, N, K, group):
        self.fmt, self.N, self.K, self.group = fmt, N, K, group
        self.codes, self.scales, self.bias = QUANTIZE[fmt](inputs.weights(N, K), group)

    def __call__(self, X, out=None):
        if self.fmt == "bf16":
            return e0m4.e0m4_bf16_matmul(X, self.codes, self.N, self.K, self.group, out=out)
        if self.fmt == "e0m8":
            return e0m4.e0m8_matmul(X, self.codes, self.N, self.K, self.group, out=out)
        return e0m4.e0m4_matmul(X, self.codes, self.scales, self.bias, self.N, self.K, self.group, out=out)

    def fused(self, X, **operators):
        call = e0m4.e0m8_matmul_fused if self.fmt == "e0m8" else e0m4.e0m4_matmul_fused
        return call(X, self.codes, self.N, self.K, self.group, **operators)


class LinearPass:
    def __init__(self, case, seed):
        inputs = Inputs(seed, _dtype(case))
        self.weight = Linear(inputs, case["format"], case["N"], case["K"], case["group"])
        self.X = inputs.activations(case["M"], case["K"])

    def run(self):
        return self.weight(self.X)


class PackPass:
    def __init__(self, case, seed):
        self.fmt, self.N, self.K, self.group = case["format"], case["N"], case["K"], case["group"]
        self.W = Inputs(seed, _dtype(case)).weights(self.N, self.K)

    def run(self):
        codes, scales, bias = QUANTIZE[self.fmt](self.W, self.group)
        if self.fmt == "bf16":
            back = e0m4.e0m4_bf16_dequant(codes, self.N, self.K, self.group)
        elif self.fmt == "e0m8":
            back = e0m4.e0m8_dequant(codes, self.N, self.K, self.group)
        else:
            back = e0m4.e0m4_dequant(codes, scales, bias, self.N, self.K, self.group)
        return {"codes": codes, "scales": scales, "bias": bias, "weights": back}


class BlocksPass:
    def __init__(self, case, seed):
        inputs = Inputs(seed, torch.float16)
        M, H, Q, F, G, L = (case[k] for k in ("M", "hidden", "qkv", "ff", "group", "layers"))
        fmt = case["format"]
        self.H = H
        self.layers = [{
            "qkv": Linear(inputs, fmt, Q, H, G), "out": Linear(inputs, fmt, H, H, G),
            "gate_up": Linear(inputs, fmt, 2 * F, H, G), "down": Linear(inputs, fmt, H, F, G),
            "norm1": inputs.norm_weight(H), "norm2": inputs.norm_weight(H),
        } for _ in range(L)]
        self.vocab = Linear(inputs, fmt, case["vocab"], H, G) if case["vocab"] else None
        self.norm = inputs.norm_weight(H)
        self.x = inputs.activations(M, H)
        self.context = inputs.activations(L, M, H)
        positions = max(2048, M)
        self.cache = torch.zeros((L, positions, Q - H), dtype=torch.float16, device=DEVICE)
        self.position_ids = torch.randperm(positions, generator=inputs.gen, device=DEVICE)[:M].contiguous()
        self.graph = None
        if case["graph"]:
            side = torch.cuda.Stream()
            side.wait_stream(torch.cuda.current_stream())
            with torch.cuda.stream(side):
                self.step()                             # loads the kernels before the capture
            torch.cuda.current_stream().wait_stream(side)
            self.graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(self.graph):
                self.result = self.step()

    def step(self):
        h, new = self.x, []
        for layer, context, cache in zip(self.layers, self.context, self.cache):
            qkv = layer["qkv"].fused(h, rms_gamma=layer["norm1"], rms_eps=EPS)
            e0m4.e0m4_kv_append(cache, qkv[:, self.H:], self.position_ids)
            h = layer["out"].fused(context, residual=h)
            g = layer["gate_up"].fused(h, rms_gamma=layer["norm2"], rms_eps=EPS, epilogue=e0m4.E0M4_EPILOGUE_SWIGLU)
            h = layer["down"].fused(g, residual=h)
            new.append(qkv)
        out = {"hidden": h, "qkv": new, "cache": self.cache}
        if self.vocab is not None:
            out["logits"] = self.vocab.fused(h, rms_gamma=self.norm, rms_eps=EPS)
        return out

    def run(self):
        if self.graph is None:
            return self.step()
        self.graph.replay()
        return self.result


class PlainPass:
    def __init__(self, case, seed):
        inputs = Inputs(seed, torch.bfloat16)
        M, H, Q, F, G, L = (case[k] for k in ("M", "hidden", "qkv", "ff", "group", "layers"))
        self.layers = [[(Linear(inputs, "bf16", N, K, G), inputs.activations(M, K))
                        for N, K in ((Q, H), (H, H), (2 * F, H), (H, F))] for _ in range(L)]
        self.graph = None
        if case["graph"]:
            side = torch.cuda.Stream()
            side.wait_stream(torch.cuda.current_stream())
            with torch.cuda.stream(side):
                self.step()
            torch.cuda.current_stream().wait_stream(side)
            self.graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(self.graph):
                self.result = self.step()

    def step(self):
        return [[weight(X) for weight, X in layer] for layer in self.layers]

    def run(self):
        if self.graph is None:
            return self.step()
        self.graph.replay()
        return self.result


PASSES = {"linear": LinearPass, "blocks": BlocksPass, "plain": PlainPass, "pack": PackPass}


def prepare(case, seed):
    return PASSES[case["kind"]](case, seed)


def run(state):
    return state.run()


def _weight_bytes(case, N, K):
    return N * K * (8 if case["format"] == "e0m8" else 4) // 8 + 4 * N * (K // case["group"])


def work(case):
    if case["kind"] == "pack":
        N, K = case["N"], case["K"]
        # read W; write codes and parameters; read them back; write the weights
        return {"bytes": 4 * N * K + 2 * _weight_bytes(case, N, K), "flops": 6 * N * K}
    M = case["M"]
    if case["kind"] == "linear":
        N, K = case["N"], case["K"]
        return {"bytes": _weight_bytes(case, N, K) + 2 * M * (N + K), "flops": 2 * M * N * K}
    H, Q, F, L = (case[k] for k in ("hidden", "qkv", "ff", "layers"))
    shapes = [(Q, H), (H, H), (2 * F, H), (H, F)] * L
    if case["vocab"]:
        shapes.append((case["vocab"], H))
    weights = sum(_weight_bytes(case, N, K) for N, K in shapes)
    if case["kind"] == "plain":
        rows = sum(N + K for N, K in shapes)
    else:       # in: x, the attention results, norm weights; out: qkv, cache rows, the last hidden state, the logits
        rows = H + L * (H + Q + Q - H) + H + case["vocab"]
    return {"bytes": weights + 2 * M * rows, "flops": 2 * M * sum(N * K for N, K in shapes)}


def tolerance(case):
    """About four times what the path differs by from the same computation in float64 on the dequantised weights:
    2.2e-3 (largest 1.2e-2) for one bfloat16 matmul, 3.4e-4 (2e-3) for one fp16 matmul; a stack of blocks, whose residual
    stream is rounded to fp16 twice a layer, 4.8e-4 (2e-3) times the root of the layers."""
    if case["kind"] == "pack":
        return "exact"
    if case["format"] == "bf16":
        return {"rel": 9e-3, "max": 5e-2}
    if case["kind"] == "linear":
        return {"rel": 1.4e-3, "max": 8e-3}
    return {"rel": 2e-3 * math.sqrt(case["layers"]), "max": 8e-3 * math.sqrt(case["layers"])}
