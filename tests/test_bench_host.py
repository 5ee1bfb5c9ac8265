"""Host-side pieces of bench.py that need no GPU: the dense bf16 weight the
bf16 GEMM comparator reads, bf16(dequant(W_Q) + W_O) (eq. 1 and eq. 3),
checked bit for bit against the oracle's dequantisation on the same
synthetic problem; the kernel names of the records; the length of the JSON line."""

import json

import numpy as np
import torch

import bench
import oracle
import paper_2608_15531_amd as fq
from synth import make_problem


def test_comparator_weight_matches_oracle():
    K, N = 512, 192
    p = make_problem(1, K, N, frac=0.02, seed=11)
    Wq = torch.from_numpy(p.Wq.view(np.int32).copy())
    s = torch.from_numpy(p.scales.view(np.int16).copy()).view(torch.float16)
    z = torch.from_numpy(p.zeros.view(np.int32).copy())
    w = bench.bf16_dequant_weight(torch, Wq, s, z, p.k, p.n, p.v, K, N)
    assert w.dtype == torch.bfloat16 and tuple(w.shape) == (K, N)
    ref = oracle.dequant(p.Wq, p.scales, p.zeros, K, N, 128)
    np.add.at(ref, (p.k, p.n), oracle.bf16_to_f64(p.v))
    want = oracle.bf16_rne_bits(ref)
    got = w.view(torch.int16).numpy().view(np.uint16)
    assert np.array_equal(got, want)
    # an outlier position holds exactly the outlier (its code is the zero-point)
    assert np.array_equal(got[p.k, p.n], p.v)


def _sizes(K, N, per_tile, fullest):
    s = fq.fq_tilecoo_sizes()
    s.n_groups, s.max_tile_groups = K // 128 * (N // 64) * per_tile, fullest
    return s


def test_kernel_names_follow_the_launch():
    assert bench.kernel_name(fq, 128, 4096, 28672) == "rows_kernel<2, true, 1>"
    # one tile beyond the row-block kernel's groups; partial sums beyond the scratch
    assert bench.kernel_name(fq, 128, 4096, 28672, sizes=_sizes(4096, 28672, 21, 161)).startswith("matmul_kernel<2, 1")
    assert bench.kernel_name(fq, 64, 28672, 28672).startswith("matmul_kernel<2, 1")
    # a second group load only where the instance exists
    full = _sizes(4096, 28672, 103, 124)
    assert bench.kernel_name(fq, 8, 4096, 28672, sizes=full).endswith("2>")
    for flags in (fq.FQ_SCHED_STREAM_K, fq.FQ_SPARSE_WAVES):
        assert bench.kernel_name(fq, 8, 4096, 28672, flags=flags, sizes=full).endswith("1>")
    assert bench.kernel_name(fq, 1, 4096, 28672, flags=fq.FQ_DENSE_VALU, sizes=full).endswith("1>")
    by_column = {"group_mode": fq.FQ_GROUP_BY_COLUMN, "buckets_per_tile": 16}
    assert bench.kernel_name(fq, 1, 4096, 28672, packing=by_column, sizes=full).endswith("1>")
    # FLOPs of the row-block kernel: 4 column waves x 224 column blocks x 2 row blocks, 32
    # tiles, 32 MFMAs of 32 x 32 x 16 and 4 of 16 x 16 x 32 each
    assert bench.mfma_flops(fq, 128, 4096, 28672) == 4 * 224 * 2 * 32 * (32 * 16384 + 4 * 8192) * 2


def test_json_line_is_short():
    """The line holds the contract's fields and every matmul's time, and stays
    below 3000 characters whatever the library kernels' names are."""
    details = [{"shape": name, "M": M, "K": K, "N": N, "kernel": "k" * 80, "bf16_gemm_kernel": "Cijk_" * 90,
                "fused_us": 12.345, "unfused_us": 23.456, "dense_only_us": 10.123, "bf16_gemm_us": 34.567}
               for name, K, N in bench.SHAPES for M in bench.MS]
    fields = {"metric": bench.METRIC, "value": 2700.12, "unit": "GB/s", "n_gpus": 1, "steps": 200,
              "warmup": 20, "ms_per_step": 0.18, "higher_is_better": True, "scaling": "weak",
              "vs_baseline": None, "dtype": "bf16", "data": "synthetic", "config": {"workload": "w" * 400},
              "roofline": {"kernel": "k" * 80, "launches": ["gate_up/M1"] * 8}}
    result = dict(fields, per_matmul=details, pack_s={"qkv": 0.1}, bf16_gemm_comparator="c" * 400,
                  layer_aggregate=[{"M": M, "bytes": 116000000, "fused_us": 41.234, "GBs": 2800.1,
                                    "pct_peak": 35.1, "pct_of_probe": 50.2} for M in bench.MS],
                  tilecoo_paper_format={"tilecoo": "t" * 90, "ms_per_step": 0.18, "value": 2800.1,
                                        "unit": "GB/s", "step_bytes": 1, "us_per_matmul": 1,
                                        "default_speedup": 1.01},
                  cpu_baseline={"value": 0.0055, "unit": "GB/s", "cores": 16, "kind": "oracle",
                                "cpu_model": "x", "sample": "s" * 300, "per_case": [{"case": "c" * 40}] * 8})
    line = bench.contract_line(result)
    assert all(line[k] == v for k, v in fields.items())
    assert set(line["fused_us"]) == {f"{n}/M{M}" for n, _, _ in bench.SHAPES for M in bench.MS}
    assert len(json.dumps(line)) < 3000
