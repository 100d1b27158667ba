"""Performance cases: what a program that serves 4-bit weights asks of this package.

Each case is one pass through the public entry points (``gemm``,
``MarlinLinear``, a captured HIP graph of a block's projections, the 2:4
sparse GEMM, loading a layer from fp16 weights, unpacking one).  The layers
are those of the package's tests and benchmark: the Llama-7B projections
(4096 x 4096, 4096 x 11008, 11008 x 4096) and the 70B-class ones
(8192 x 10240, 8192 x 8192, 8192 x 28672, 28672 x 8192), at batches from one
row (single-stream decode) to 4096 (prefill), plus drawn sizes in between.

Values: activations N(0, 1), codes uniform in 0..15, scales U[0.5, 1.5] /
(8 sqrt(K)) so that outputs are O(1); fp16 weights to be quantised are normal
with a per-channel spread and one entry in 1000 eight times larger.
"""
import math

import torch

import paper_2408_11743_amd as mk

LAYERS_7B = [(4096, 4096), (4096, 11008), (11008, 4096)]
LAYERS_70B = [(8192, 10240), (8192, 8192), (8192, 28672), (28672, 8192)]
MAX_M, MAX_WEIGHTS = 4096, 28672 * 8192


def _case(kind, layers, M, group=128, name=None):
    case = {"kind": kind, "layers": " ".join("%dx%d" % l for l in layers), "M": M, "group": group}
    if name:
        case["name"] = name
    return case


def listed():
    return [
        # one projection of a single-stream decode step, called from Python: launch latency and host time count
        _case("gemm", [(4096, 4096)], 1, name="attn_7b_m1"),
        # a small decode batch through the layer module, scales per output channel
        _case("linear", [(11008, 4096)], 8, group=-1, name="down_7b_channel_m8"),
        # single-stream decode as a serving loop runs it: the block's four projections in a captured graph
        _case("block", LAYERS_70B, 1, name="block_70b_graph_m1"),
        # decode batches: the 7B block at 16 sequences, the 70B one at 32 and 64
        _case("block", [(4096, 4096)] + LAYERS_7B, 16, name="block_7b_graph_m16"),
        _case("block", LAYERS_70B, 32, name="block_70b_graph_m32"),
        _case("block", LAYERS_70B, 64, name="block_70b_graph_m64"),
        # a ragged decode batch, and the largest one of the paper's sweep
        _case("linear", [(8192, 10240)], 100, name="qkv_70b_m100"),
        _case("gemm", [(8192, 28672)], 128, name="up_70b_m128"),
        # 2:4 sparse weights at a small decode batch
        _case("sparse", [(8192, 8192)], 8, name="sparse_8192_m8"),
        # prefill: a prompt of ragged length, and the largest batch that one launch takes
        _case("linear", [(4096, 11008)], 1000, name="prefill_7b_m1000"),
        _case("gemm", [(28672, 8192)], 4096, name="prefill_70b_m4096"),
        # loading a model: one fp16 layer quantised (ten clipping ratios) and packed
        _case("load", [(4096, 11008)], 0, name="load_up_7b"),
    ]


def _draw_layer(rng):
    if rng.random() < 0.5:
        return rng.choice(LAYERS_7B + LAYERS_70B)
    while True:  # any shape the layout allows, narrow and odd multiples among them
        K = 128 * round(2 ** rng.uniform(3, math.log2(28672 / 128)))
        N = 64 * round(2 ** rng.uniform(4, math.log2(28672 / 64)))
        if K * N <= MAX_WEIGHTS:
            return K, N


def draw(rng):
    kind = rng.choices(["gemm", "linear", "block", "sparse", "load", "unpack"], [30, 20, 18, 14, 10, 8])[0]
    layers = [_draw_layer(rng) for _ in range(rng.randint(2, 4) if kind == "block" else 1)]
    group = rng.choices([128, -1, 256, 512], [60, 20, 10, 10])[0]
    if any(K % group for K, _ in layers if group > 0):
        group = 128
    if kind in ("load", "unpack"):
        return _case(kind, layers, 0, group)
    # decode blocks are captured for batches up to 128; single calls take any batch
    M = round(2 ** rng.uniform(0, 7 if kind == "block" else 12))
    return _case(kind, layers, M, group)


def _layers(case):
    return [tuple(int(v) for v in l.split("x")) for l in case["layers"].split()]


def _rng(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _scale_rows(K, group):
    return 1 if group in (-1, K) else K // group


def _codes(g, K, N, sparse):
    q = torch.randint(0, 16, (K, N), dtype=torch.uint8, device="cuda", generator=g)
    if sparse:  # two rows kept of every four, uniform over the six patterns; pruned rows hold code 8
        r = torch.rand((K // 4, 4, N), device="cuda", generator=g)
        keep = torch.zeros((K // 4, 4, N), dtype=torch.bool, device="cuda")
        keep.scatter_(1, r.topk(2, dim=1).indices, True)
        q.masked_fill_(~keep.view(K, N), 8)
    return q


def _weights(case, seed):
    """Per layer: codes [K, N] and scales [G, N]."""
    g = _rng(seed)
    out = []
    for K, N in _layers(case):
        q = _codes(g, K, N, case["kind"] == "sparse")
        u = torch.rand((_scale_rows(K, case["group"]), N), device="cuda", generator=g) + 0.5
        out.append((q, (u / (8.0 * math.sqrt(K))).half()))
    return out


def _activations(case, seed):
    g = _rng(int(seed) + 1000003)
    return [torch.randn((case["M"], K), device="cuda", generator=g).half() for K, _ in _layers(case)]


def _fp16_weight(case, seed):
    """nn.Linear layout, [out_features, in_features]."""
    g = _rng(seed)
    (K, N), = _layers(case)
    sigma = (torch.rand((N, 1), device="cuda", generator=g) + 0.5) / math.sqrt(K)
    w = torch.randn((N, K), device="cuda", generator=g) * sigma
    outlier = torch.rand((N, K), device="cuda", generator=g) < 1e-3
    return torch.where(outlier, w * 8.0, w).half()


def prepare(case, seed):
    kind, group = case["kind"], case["group"]
    if kind == "load":
        return {"kind": kind, "weight": _fp16_weight(case, seed), "group": group}
    sparse = kind == "sparse"
    packed = [(*mk.pack(q, s, group=group, sparse=sparse), *q.shape) for q, s in _weights(case, seed)]
    if kind == "unpack":
        return {"kind": kind, "packed": packed[0], "group": group}
    A = _activations(case, seed)
    if kind == "linear":
        wp, sp, K, N = packed[0]
        # [sequences, tokens, features], as a model's hidden states come
        return {"kind": kind, "layer": mk.MarlinLinear(wp, sp, K, N, group), "x": A[0].unsqueeze(0)}
    if kind == "block":
        ws = mk.Workspace(A[0].device)
        C = [torch.empty((case["M"], p[3]), dtype=torch.float16, device="cuda") for p in packed]

        def step():
            for a, (wp, sp, K, N), c in zip(A, packed, C):
                mk.gemm(a, wp, sp, K, N, group, out=c, workspace=ws)

        step()  # the workspace grows to its size before the capture
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            step()
        return {"kind": kind, "graph": graph, "C": C, "keep": (A, packed, ws)}
    return {"kind": kind, "A": A[0], "packed": packed[0], "group": group, "sparse": sparse}


def run(state):
    kind = state["kind"]
    if kind == "block":
        state["graph"].replay()
        return state["C"]
    if kind == "linear":
        return state["layer"](state["x"])
    if kind == "load":
        layer = mk.MarlinLinear.from_float(state["weight"], group=state["group"])
        return layer.w_packed, layer.s_packed
    wp, sp, K, N = state["packed"]
    if kind == "unpack":
        return mk.unpack(wp, sp, K, N, group=state["group"])
    return mk.gemm(state["A"], wp, sp, K, N, group=state["group"], sparse=state["sparse"])


def work(case):
    M, kind = case["M"], case["kind"]
    total, flops = 0, 0
    for K, N in _layers(case):
        scales = 2 * _scale_rows(K, case["group"]) * N
        if kind == "load":  # fp16 in, codes and scales out; per ratio: scale, round, clamp, difference, square, sum
            total += 2 * K * N + K * N // 2 + scales
            flops += K * N * (len(mk.CLIP_RATIOS) * 7 + 6)
        elif kind == "unpack":  # 4-bit codes in, one byte each out
            total += K * N // 2 + K * N + 2 * scales
        else:
            total += (K * N // 8 * 3 if kind == "sparse" else K * N // 2) + scales + 2 * M * (K + N)
            flops += 2 * M * K * N // (2 if kind == "sparse" else 1)
    return {"bytes": total, "flops": flops}


def tolerance(case):
    if case["kind"] in ("load", "unpack"):
        return "exact"
    # Outputs are fp16 (2^-12 of the value on average: 2e-4 of the norm), and
    # the group scale may be applied to fp16 weights (as much again, per
    # weight): 2.1e-4 to 3.0e-4 measured against 64 bits over the listed cases.
    return {"rel": 1.2e-3, "max": 6e-3}


def exact(case, seed):
    kind = case["kind"]
    if kind == "load":
        return None
    if kind == "unpack":
        return _weights(case, seed)[0]
    out = []
    for A, (q, s) in zip(_activations(case, seed), _weights(case, seed)):
        K = q.shape[0]
        w = (q.double() - 8.0).view(s.shape[0], K // s.shape[0], -1) * s.double()[:, None, :]
        out.append(A.double() @ w.view(K, -1))
        del w
    if kind == "block":
        return out
    return out[0].unsqueeze(0) if kind == "linear" else out[0]
