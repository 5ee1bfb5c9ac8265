"""Tiles whose outlier groups fill the two group loads of a tile, end at their
edges, or go on past them (loaded four passes at once), beside an empty tile:
exact-arithmetic inputs, so the result equals the fp64 oracle bit for bit."""

import dataclasses

import numpy as np
import pytest
import torch

import oracle
from synth import bf16_bits_from_f32, make_exact_problem

pytestmark = pytest.mark.gpu


def _problem(M, groups, seed):
    """K = 256, N = 128: by-bucket groups of the four tiles as given (a tile's
    outliers fill all but its last group's last slot)."""
    p = make_exact_problem(M, 256, 128, frac=0.0, seed=seed)
    rng = np.random.Generator(np.random.PCG64(seed + 1))
    ks, ns = [], []
    for t, g in enumerate(groups):
        pos = rng.choice(128 * 64, size=max(0, 4 * g - 1), replace=False)
        ks.append((t % 2) * 128 + pos // 64)
        ns.append((t // 2) * 64 + pos % 64)
    k = np.concatenate(ks).astype(np.int32)
    n = np.concatenate(ns).astype(np.int32)
    v = rng.integers(1, 33, size=k.size) / 8.0 * np.where(rng.integers(0, 2, size=k.size) == 1, -1.0, 1.0)
    return dataclasses.replace(p, k=k, n=n, v=bf16_bits_from_f32(v.astype(np.float32)))


@pytest.mark.parametrize("groups", [65, 127, 128, 129, 384, 385, 2048])
@pytest.mark.parametrize("M", [1, 7, 16, 20])
def test_two_group_loads_bit_exact(gpu_lib, groups, M):
    fq = gpu_lib
    p = _problem(M, [groups, 0, 64, 65], seed=groups + M)
    host = fq.fq_pack_tile_coo(p.K, p.N, p.k, p.n, p.v)
    assert host.sizes.max_tile_groups == max(groups, 65)
    assert host.sizes.n_groups >= 32 * host.sizes.n_tiles   # the instance with two loads
    X, Wq, s, z = fq.to_device(p)
    tc = fq.TileCOODevice(host)
    print(f"two group loads: {groups} groups in the first tile, M={M}", flush=True)
    exact = oracle.matmul(p.X, p.Wq, p.scales, p.zeros, p.K, p.N, p.group, p.k, p.n, p.v)
    for flags in (0, fq.FQ_STRIP_32, fq.FQ_STRIP_64):
        for split_k in (0, 2):
            y = fq.fq_w4a16_outlier_matmul(X, Wq, s, z, tc, y_dtype="f32", flags=flags, split_k=split_k)
            torch.cuda.synchronize()
            assert np.array_equal(y.cpu().numpy(), exact.astype(np.float32)), (flags, split_k)
