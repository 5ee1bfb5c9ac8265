"""The row-block kernel (more than 16 rows, long K) at the edges of its range.

Exact-arithmetic inputs: every fp32 sum is exact in any order, so the result
equals the fp64 oracle bit for bit on sampled columns (the first and last of
the 32-, 64- and 128-column blocks among them) and, on every column, the strip
kernel's, which a forced strip width selects.  Both kernels give the same bits
there, so every test asks fq_launch_kernel which one its calls run.
"""

import dataclasses

import numpy as np
import pytest
import torch

import oracle
from synth import bf16_bits_from_f32, make_exact_problem, make_problem

pytestmark = pytest.mark.gpu

# (M, K, N, outlier share, packing, row blocks, K ranges)
CASES = [
    (33, 1792, 16448, 0.02, None, 1, 1),        # 14 tiles, no split, N an odd multiple of 64
    (64, 7296, 8192, 0.01, None, 1, 4),         # 57 tiles split 4 ways: 14 and 15
    (97, 1920, 8320, 0.03, "column", 2, 1),     # 15 tiles (the K groups take 8 and 7)
    (128, 2176, 8256, 0.06, None, 2, 1),        # more than 64 groups in a tile, last block half empty
    (96, 14336, 2048, 0.0004, None, 2, 8),      # two row blocks and a split, most tiles empty
    (128, 4096, 6144, 0.01, None, 2, 2),        # two full row blocks and a split
    (17, 1792, 16512, 0.02, None, 1, 1),        # one 32-row block
    (32, 2048, 16448, 0.012, "column", 1, 1),   # one full 32-row block, up to 62 groups a tile
    (40, 16256, 4096, 0.01, None, 1, 8),        # 127 tiles split 8 ways: 15 and 16
    (48, 1792, 16448, 0.0, None, 1, 1),         # no outliers: the dense-only form
    (80, 14336, 2048, 0.0, None, 2, 8),         # the same, two row blocks and a split
]


@pytest.mark.parametrize("M,K,N,frac,packing,row_blocks,split", CASES,
                         ids=[f"rows{i}" for i in range(len(CASES))])
def test_rows_kernel_bit_exact(gpu_lib, M, K, N, frac, packing, row_blocks, split):
    fq = gpu_lib
    p = make_exact_problem(M, K, N, frac=frac, seed=M + N)
    X, Wq, s, z = fq.to_device(p)
    params = {"buckets_per_tile": 16, "group_mode": fq.FQ_GROUP_BY_COLUMN} if packing else None
    host = fq.fq_pack_tile_coo(K, N, p.k, p.n, p.v, params)
    tc = fq.TileCOODevice(host)
    c = fq.fq_launch_kernel(M, K, N, host)
    assert (c["kernel"], c["row_blocks"], c["split_k"]) == ("rows", row_blocks, split)
    full = host.sizes.max_tile_groups > 64 and host.sizes.n_groups >= 32 * host.sizes.n_tiles
    assert c["group_loads"] == (0 if frac == 0 else 2 if full else 1)
    assert fq.fq_launch_kernel(M, K, N, host, workspace_bytes=fq.NOALLOC_SCRATCH_BYTES) == c
    assert fq.fq_launch_kernel(M, K, N, host, flags=fq.FQ_STRIP_64)["kernel"] == "strip"
    if frac == 0:
        assert fq.fq_launch_kernel(M, K, N)["kernel"] == "rows"
    print(f"rows kernel M={M} K={K} N={N} outliers {frac}", flush=True)
    y = fq.fq_w4a16_outlier_matmul(X, Wq, s, z, tc, y_dtype="f32")
    again = fq.fq_w4a16_outlier_matmul(X, Wq, s, z, tc, y_dtype="f32")
    noalloc = torch.empty_like(y)
    fq.fq_w4a16_outlier_matmul_noalloc(X, Wq, s, z, tc, noalloc, y_dtype="f32")
    bf = fq.fq_w4a16_outlier_matmul(X, Wq, s, z, tc)
    strip = fq.fq_w4a16_outlier_matmul(X, Wq, s, z, tc, y_dtype="f32", flags=fq.FQ_STRIP_64)
    dense = fq.fq_w4a16_matmul(X, Wq, s, z, y_dtype="f32")
    dense_strip = fq.fq_w4a16_matmul(X, Wq, s, z, y_dtype="f32", flags=fq.FQ_STRIP_64)
    torch.cuda.synchronize()
    assert torch.equal(y, again) and torch.equal(y, noalloc)
    assert torch.equal(y, strip) and torch.equal(dense, dense_strip)
    assert torch.equal(bf, y.to(torch.bfloat16))
    cols = np.unique(np.concatenate([[0, 1, 31, 32, 63, 64, 127, 128, N - 65, N - 64, N - 33, N - 32, N - 1],
                                     np.random.default_rng(M).choice(N, 32, replace=False)]) % N)
    exact = oracle.matmul(p.X, p.Wq, p.scales, p.zeros, K, N, p.group, p.k, p.n, p.v, cols)
    assert np.array_equal(y.cpu().numpy()[:, cols], exact.astype(np.float32))


@pytest.mark.parametrize("M,groups,kernel", [(50, 64, "rows"), (50, 65, "rows"), (50, 129, "rows"),
                                             (50, 160, "rows"), (50, 161, "strip"),
                                             (32, 64, "rows"), (32, 65, "strip")])
def test_rows_kernel_one_full_tile(gpu_lib, M, groups, kernel):
    """Sparse tiles and one of `groups` groups: what one group load leaves is
    loaded inside the tile; past 160 groups, past 64 with 32-row blocks, the
    strip kernel runs."""
    fq = gpu_lib
    K, N = 1792, 16448
    p = make_exact_problem(M, K, N, frac=0.0, seed=groups)
    rng = np.random.Generator(np.random.PCG64(groups))
    pos = rng.choice(128 * 64, size=4 * groups - 1, replace=False)
    k = np.concatenate([3 * 128 + pos // 64, rng.choice(128, 9, replace=False) + 4 * 128]).astype(np.int32)
    n = np.concatenate([5 * 64 + pos % 64, np.full(9, 5 * 64 + 33)]).astype(np.int32)
    v = rng.integers(1, 33, size=k.size) / 8.0
    p = dataclasses.replace(p, k=k, n=n, v=bf16_bits_from_f32(v.astype(np.float32)))
    host = fq.fq_pack_tile_coo(K, N, p.k, p.n, p.v)
    assert host.sizes.max_tile_groups == groups
    assert fq.fq_launch_kernel(M, K, N, host)["kernel"] == kernel
    X, Wq, s, z = fq.to_device(p)
    print(f"rows kernel, one tile of {groups} groups", flush=True)
    y = fq.fq_w4a16_outlier_matmul(X, Wq, s, z, fq.TileCOODevice(host), y_dtype="f32")
    torch.cuda.synchronize()
    cols = np.concatenate([np.arange(5 * 64 - 2, 6 * 64 + 2), [0, N - 1]])
    exact = oracle.matmul(p.X, p.Wq, p.scales, p.zeros, K, N, p.group, p.k, p.n, p.v, cols)
    assert np.array_equal(y.cpu().numpy()[:, cols], exact.astype(np.float32))


def test_rows_kernel_graph_replays(gpu_lib):
    """Replays of a captured split-K launch leave the counters at zero and
    repeat the eager result, with eager calls on the same workspace between."""
    fq = gpu_lib
    M, K, N = 64, 7296, 8192
    p = make_exact_problem(M, K, N, frac=0.01, seed=3)
    X, Wq, s, z = fq.to_device(p)
    host = fq.fq_pack_tile_coo(K, N, p.k, p.n, p.v)
    tc = fq.TileCOODevice(host)
    c = fq.fq_launch_kernel(M, K, N, host)
    assert (c["kernel"], c["split_k"]) == ("rows", 4)
    ws = torch.zeros(fq.fq_workspace_bytes(M, K, N), dtype=torch.uint8, device="cuda")
    eager = fq.fq_w4a16_outlier_matmul(X, Wq, s, z, tc, y_dtype="f32", ws=ws)
    torch.cuda.synchronize()
    Y = torch.empty_like(eager)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        fq.fq_w4a16_outlier_matmul(X, Wq, s, z, tc, Y=Y, y_dtype="f32", ws=ws)
    for _ in range(4):
        Y.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(Y, eager)
        assert int(ws[:256 * 1024].count_nonzero()) == 0
        other = fq.fq_w4a16_outlier_matmul(X, Wq, s, z, tc, y_dtype="f32", ws=ws)
        torch.cuda.synchronize()
        assert torch.equal(other, eager)


def test_rows_kernel_small_workspace(gpu_lib):
    """A workspace without room for the row-block kernel's partial sums, but
    large enough for the strip kernel's launch, is served by the strip kernel."""
    fq = gpu_lib
    M, K, N = 64, 7296, 8192
    p = make_exact_problem(M, K, N, frac=0.01, seed=4)
    X, Wq, s, z = fq.to_device(p)
    host = fq.fq_pack_tile_coo(K, N, p.k, p.n, p.v)
    tc = fq.TileCOODevice(host)
    assert fq.fq_workspace_bytes(M, K, N) > 256 * 1024
    small = torch.zeros(256 * 1024, dtype=torch.uint8, device="cuda")   # 64-column strips need no split here
    assert fq.fq_launch_kernel(M, K, N, host)["kernel"] == "rows"
    assert fq.fq_launch_kernel(M, K, N, host, workspace_bytes=small.numel())["kernel"] == "strip"
    y = fq.fq_w4a16_outlier_matmul(X, Wq, s, z, tc, y_dtype="f32")
    y_small = fq.fq_w4a16_outlier_matmul(X, Wq, s, z, tc, y_dtype="f32", ws=small)
    torch.cuda.synchronize()
    assert torch.equal(y, y_small)


def test_rows_kernel_kept_workspace_grows(gpu_lib):
    """The workspace that an earlier small call left for a stream is enlarged
    for the row-block kernel: the same kernel, hence the same bits on inputs
    whose sums round, as with a workspace of the full size."""
    fq = gpu_lib
    M, K, N = 64, 7296, 8192
    stream = torch.cuda.Stream()
    p = make_problem(M, K, N, frac=0.01, seed=5)
    X, Wq, s, z = fq.to_device(p)
    host = fq.fq_pack_tile_coo(K, N, p.k, p.n, p.v)
    tc = fq.TileCOODevice(host)
    assert fq.fq_launch_kernel(M, K, N, host)["kernel"] == "rows"
    ws = torch.zeros(fq.fq_workspace_bytes(M, K, N), dtype=torch.uint8, device="cuda")
    full = fq.fq_w4a16_outlier_matmul(X, Wq, s, z, tc, y_dtype="f32", ws=ws)
    torch.cuda.synchronize()
    kept = torch.zeros(256 * 1024, dtype=torch.uint8, device="cuda")   # as a small call leaves it
    key = (X.device.index, int(stream.cuda_stream))
    before = fq._workspaces.get(key)   # streams come from a pool: put back what was there
    fq._workspaces[key] = kept
    try:
        torch.cuda.synchronize()
        y = fq.fq_w4a16_outlier_matmul(X, Wq, s, z, tc, y_dtype="f32", stream=stream)
        torch.cuda.synchronize()
        assert fq._workspaces[key].numel() >= fq.fq_workspace_bytes(M, K, N)
        assert torch.equal(y, full)
    finally:
        if before is None:
            del fq._workspaces[key]
        else:
            fq._workspaces[key] = before
