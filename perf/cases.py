"""The calls this library is timed on: weight-only INT4 linears with outliers,
as a decoding or serving program makes them.

A case is one or more linears (K x N each) at M rows.  A program that decodes
captures its step in a HIP graph and replays it, so most cases are the captured
linears of one decoder layer, or of the same linear of several layers (weights
differ from layer to layer, as they do in a model); the two smallest are eager
calls, where the host's part of a call counts too.

Fields of a case:
  shapes   "KxN,KxN,...": the linears of one layer, in order
  layers   how many layers' worth of them, each with its own weights
  M        rows of X (sequences decoded together, or tokens of a prefill chunk)
  frac     share of the weights that are outliers
  cluster  True: half of the outliers lie in 2 % of the columns
  packing  "bucket" (the library's default) or "column" (by-column groups in 16
           buckets per tile, the paper's format)
  y        output type, "bf16" or "f32" (f32: a partial sum that a row-parallel
           layer reduces over GPUs)
  entry    "fused", "noalloc" (the allocation-free entry point) or "dense" (a
           weight without outliers)
  graph    True: captured once in prepare(), replayed by run(); False: eager calls
"""

import math

import numpy as np
import torch

import paper_2608_15531_amd as fq

GROUP = 128
LLAMA3_8B = "4096x6144,4096x4096,4096x28672,14336x4096"   # qkv, o, gate+up, down


def _case(name, shapes, M, layers=1, frac=0.01, cluster=False, packing="bucket", y="bf16",
          entry="fused", graph=True):
    return {"name": name, "shapes": shapes, "layers": layers, "M": M, "frac": frac,
            "cluster": cluster, "packing": packing, "y": y, "entry": entry, "graph": graph}


def listed():
    return [
        # one sequence being decoded: the four linears of a Llama-3-8B layer
        _case("layer8b_m1", LLAMA3_8B, 1),
        # a few sequences, weights packed in the paper's by-column format
        _case("layer8b_m4_bycolumn", LLAMA3_8B, 4, packing="column"),
        # a small serving batch, the most rows that one 16-row block takes
        _case("layer8b_m16", LLAMA3_8B, 16),
        # a middle batch that fills no block evenly
        _case("layer8b_m27", LLAMA3_8B, 27),
        # a large serving batch or a short prefill chunk, the most rows supported
        _case("layer8b_m128", LLAMA3_8B, 128),
        # the up projection of several layers at 64 rows, fp32 partial sums out
        _case("up8b_m64_f32", "4096x14336", 64, layers=3, y="f32"),
        # the largest matrix of a Llama-3-70B layer at batch 8
        _case("gate_up70b_m8", "8192x57344", 8),
        # the longest K: Llama-3-70B down projection at batch 16
        _case("down70b_m16", "28672x8192", 16),
        # smallest work: an eager call on one 8-way tensor-parallel shard of the
        # 70B qkv projection, through the allocation-free entry point
        _case("shard_m3_noalloc_eager", "8192x1280", 3, entry="noalloc", graph=False),
        # one eager call as a program without graphs makes it (the output is
        # allocated by the call)
        _case("o8b_m1_eager", "4096x4096", 1, graph=False),
        # weights quantised without outliers
        _case("up8b_m8_dense", "4096x14336", 8, layers=4, frac=0.0, entry="dense"),
        # many outliers, half of them in a few columns
        _case("up8b_m8_clustered5", "4096x14336", 8, layers=3, frac=0.05, cluster=True),
    ]


def draw(rng):
    """Any shape, row count, density, packing, output type and entry point of
    the same ranges; at most the largest listed case's weights and products."""
    def spread(lo, hi):
        return int(math.exp(rng.uniform(math.log(lo), math.log(hi + 0.999))))

    while True:
        K, N, M = 128 * spread(4, 224), 64 * spread(8, 896), spread(1, 128)
        if K * N <= 8192 * 57344 and K * N * max(1.0, M / 16) <= 1.7e9 and K * N >= 1 << 20:
            break
    entry = rng.choice(["fused", "fused", "fused", "fused", "noalloc", "dense"])
    frac = 0.0 if entry == "dense" else rng.choice([0.0, 0.005, 0.01, 0.01, 0.01, 0.02, 0.05])
    graph = rng.random() < 0.75
    c = _case("", "%dx%d" % (K, N), M, frac=frac, cluster=frac > 0 and rng.random() < 0.25,
              layers=max(1, min(4, (1 << 27) // (K * N))) if graph else 1,
              packing=rng.choice(["bucket", "bucket", "column"]),
              y=rng.choice(["bf16", "bf16", "f32"]), entry=entry, graph=graph)
    del c["name"]
    return c


def _linears(case):
    one = [tuple(int(v) for v in s.split("x")) for s in case["shapes"].split(",")]
    return one * case["layers"]


def _inputs(case, seed, i, K, N):
    """Linear i's X, codes [K][N] (uint8), scales and zero-points [K/128][N] and
    outliers (k, n, v), on the GPU: N(0, 1) activations, codes over the whole
    range, scales and zero-points as a symmetric-looking weight has them."""
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 1009 + i)
    dev, M, frac = "cuda", case["M"], case["frac"]
    X = torch.randn((M, K), generator=g, device=dev).to(torch.bfloat16)
    codes = torch.randint(0, 16, (K, N), generator=g, device=dev, dtype=torch.uint8)
    scales = (torch.rand((K // GROUP, N), generator=g, device=dev) * 0.015 + 0.005).to(torch.float16)
    zeros = torch.randint(6, 10, (K // GROUP, N), generator=g, device=dev, dtype=torch.uint8)
    if frac > 0:
        p = torch.full((N,), frac, device=dev)
        if case["cluster"]:
            n_c = max(1, round(0.02 * N))
            p.fill_(0.5 * frac * N / max(1, N - n_c))
            p[torch.randperm(N, generator=g, device=dev)[:n_c]] = min(1.0, 0.5 * frac * N / n_c)
        kn = (torch.rand((K, N), generator=g, device=dev) < p).nonzero()
        k, n = kn[:, 0], kn[:, 1]
        v = 0.5 * torch.randn((k.numel(),), generator=g, device=dev)
        v = torch.where(v.abs() < 0.1, torch.where(v < 0, -0.1, 0.1), v).to(torch.bfloat16)
        codes[k, n] = zeros[k // GROUP, n]   # a code at an outlier dequantises to zero
    else:
        k = n = torch.zeros(0, dtype=torch.int64, device=dev)
        v = torch.zeros(0, dtype=torch.bfloat16, device=dev)
    return X, codes, scales, zeros, k, n, v


def _nibbles(codes, axis):
    """Eight 4-bit codes along `axis` into one 32-bit word, the first lowest."""
    R, C = codes.shape
    c = codes.view(R // 8, 8, C) if axis == 0 else codes.view(R, C // 8, 8)
    out = None
    for j in range(8):
        word = (c[:, j, :] if axis == 0 else c[:, :, j]).to(torch.int32) << (4 * j)
        out = word if out is None else out | word
    return out.contiguous()


def _call(case, lin, ws):
    X, Wq, s, z, tc, Y = lin
    if case["entry"] == "dense":
        return fq.fq_w4a16_matmul(X, Wq, s, z, Y=Y, y_dtype=case["y"], ws=ws)
    if case["entry"] == "noalloc":
        return fq.fq_w4a16_outlier_matmul_noalloc(X, Wq, s, z, tc, Y, y_dtype=case["y"])
    return fq.fq_w4a16_outlier_matmul(X, Wq, s, z, tc, Y=Y, y_dtype=case["y"], ws=ws)


def prepare(case, seed):
    params = ({"buckets_per_tile": 16, "group_mode": fq.FQ_GROUP_BY_COLUMN}
              if case["packing"] == "column" else None)
    ydt = torch.float32 if case["y"] == "f32" else torch.bfloat16
    own_y = case["graph"] or case["entry"] == "noalloc"
    linears, need = [], 256
    for i, (K, N) in enumerate(_linears(case)):
        X, codes, scales, zeros, k, n, v = _inputs(case, seed, i, K, N)
        Wq, zw = _nibbles(codes, 0), _nibbles(zeros, 1)
        del codes
        tc = None
        if case["entry"] != "dense":
            host = fq.fq_pack_tile_coo(K, N, k.to(torch.int32).cpu().numpy(),
                                       n.to(torch.int32).cpu().numpy(),
                                       v.view(torch.int16).cpu().numpy().view(np.uint16), params)
            tc = fq.TileCOODevice(host, "cuda")
        Y = torch.empty((case["M"], N), dtype=ydt, device="cuda") if own_y else None
        linears.append((X, Wq, scales, zw, tc, Y))
        need = max(need, fq.fq_workspace_bytes(case["M"], K, N,
                                               fq.FQ_Y_F32 if case["y"] == "f32" else fq.FQ_Y_BF16))
    state = {"case": case, "linears": linears, "graph": None, "ws": None}
    if case["graph"]:
        state["ws"] = torch.zeros(need, dtype=torch.uint8, device="cuda")
        for lin in linears:
            _call(case, lin, state["ws"])
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            for lin in linears:
                _call(case, lin, state["ws"])
        state["graph"] = graph
    return state


def run(state):
    if state["graph"] is not None:
        state["graph"].replay()
        return [lin[5] for lin in state["linears"]]
    return [_call(state["case"], lin, None) for lin in state["linears"]]


def work(case):
    M, y = case["M"], 4 if case["y"] == "f32" else 2
    b = f = 0.0
    for K, N in _linears(case):
        nnz = K * N * case["frac"]
        # codes, scales, zero-points, four bytes an outlier (two indices, bf16), X, Y
        b += K * N / 2 + K * N / GROUP * 2.5 + 4 * nnz + 2 * M * K + y * M * N
        f += 2.0 * M * K * N + 2.0 * M * nnz
    return {"bytes": b, "flops": f}


def tolerance(case):
    # about four times what the path is off from exact(): bf16 outputs by their one
    # rounding (1.7e-3), fp32 outputs (1e-6) by fp32 sums of up to 28672 terms whose
    # partial sums exceed the result (the codes are offset by 128 + z)
    return {"rel": 5e-6} if case["y"] == "f32" else {"rel": 7e-3}


def exact(case, seed):
    """Y = X dequant(W_Q) + X W_O in 64 bits."""
    ys = []
    for i, (K, N) in enumerate(_linears(case)):
        X, codes, scales, zeros, k, n, v = _inputs(case, seed, i, K, N)
        Y = torch.zeros((case["M"], N), dtype=torch.float64, device="cuda")
        step = GROUP * max(1, (1 << 26) // (GROUP * N))   # rows of W held in fp64 at a time
        for k0 in range(0, K, step):
            k1 = min(K, k0 + step)
            g = torch.arange(k0, k1, device="cuda") // GROUP
            W = scales[g].double() * (codes[k0:k1].double() - zeros[g].double())
            here = (k >= k0) & (k < k1)
            W[k[here] - k0, n[here]] += v[here].double()
            Y += X[:, k0:k1].double() @ W
        ys.append(Y)
    return ys
