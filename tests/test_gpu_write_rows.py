"""GPU: the cache write on both sides of the line between a wavefront per row and the bulk kernel (2560 rows
of a one-byte cache, 1536 of an fp16 one).  The bulk kernel's own edges need calls of many heads for that."""
import numpy as np
import pytest
import torch

import paper_2602_09323_amd as coopt
from gpu_utils import dev
from test_gpu_write import test_bulk_calls_with_every_slot_pattern as every_slot_pattern
from test_gpu_write import test_bulk_windows_equal_rows as windows_equal_rows

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kv_dtype", ["e4m3", "e5m2", "fp16"])
@pytest.mark.parametrize("d", [128, 64])
def test_windows(d, kv_dtype):
    windows_equal_rows(d, 32, kv_dtype)              # 40 tokens at a time: 1280 rows, 87 and more at once: 2784


@pytest.mark.parametrize("kv_dtype", ["e4m3", "fp16"])
@pytest.mark.parametrize("d", [128, 64])
def test_slot_patterns(oracle_mod, d, kv_dtype):
    every_slot_pattern(oracle_mod, d, 32, kv_dtype)


@pytest.mark.parametrize("kv_dtype,H_k,T", [("e4m3", 40, 64), ("e4m3", 40, 65), ("e4m3", 8, 320), ("e4m3", 8, 321),
                                            ("e5m2", 16, 161), ("fp16", 8, 192), ("fp16", 8, 193), ("fp16", 24, 64),
                                            ("fp16", 24, 65)])
def test_either_side_of_the_line(kv_dtype, H_k, T):
    """One call against the same tokens in calls that are all below it."""
    kv = {"e4m3": coopt.COOPT_KV_E4M3, "e5m2": coopt.COOPT_KV_E5M2, "fp16": coopt.COOPT_KV_FP16}[kv_dtype]
    d, NB, fp8 = 64, 2 * T // 16 + 4, kv_dtype != "fp16"
    shape = coopt.Shape(1, H_k, H_k, d, 16, NB, NB, kv, 1.0)
    rng = np.random.default_rng(T)
    slots = np.concatenate([np.arange(3, 3 + T // 2), T // 2 + 20 + rng.permutation(T)[:T - T // 2]])
    k, v, ds = (dev(x) for x in (rng.standard_normal((T, H_k, d)).astype(np.float16), rng.standard_normal((T, H_k, d)).astype(np.float16), slots))
    got = []
    for step in (T, 16):
        c = [torch.zeros(NB, H_k, 16 * d * (1 if fp8 else 2), dtype=torch.uint8, device="cuda") for _ in range(2)]
        c += [torch.zeros(NB, H_k, 16, device="cuda") for _ in range(2)] if fp8 else []
        for i in range(0, T, step):
            (coopt.kv_cache_write_fp8 if fp8 else coopt.kv_cache_write_fp16)(k[i:i + step], v[i:i + step], ds[i:i + step], *c, shape)
        torch.cuda.synchronize()
        got.append(c)
    assert all(torch.equal(a, b) for a, b in zip(*got))


@pytest.mark.parametrize("kv_dtype,d,H_k,T", [("e4m3", 128, 40, 3865), ("e4m3", 128, 40, 3866), ("e5m2", 64, 40, 12755),
                                              ("e5m2", 64, 40, 12756), ("fp16", 128, 40, 2929), ("fp16", 128, 40, 2930),
                                              ("fp16", 64, 24, 9766)])
def test_either_side_of_a_large_call(kv_dtype, d, H_k, T):
    """... 120 MB read and written (one byte a code, 64 dims: 200 MB): one call against calls of 32 tokens, a
    wavefront per row; runs of every alignment, single tokens, tokens that are filtered."""
    kv = {"e4m3": coopt.COOPT_KV_E4M3, "e5m2": coopt.COOPT_KV_E5M2, "fp16": coopt.COOPT_KV_FP16}[kv_dtype]
    NB, fp8 = T // 16 + 40, kv_dtype != "fp16"
    shape = coopt.Shape(1, H_k, H_k, d, 16, NB, NB, kv, 1.0)
    rng = np.random.default_rng(T)
    slots = np.concatenate([np.arange(5, 5 + T // 2), T // 2 + 8 + rng.permutation(T // 4),
                            3 * T // 4 + 27 + np.arange(T - T // 2 - T // 4)])
    slots[rng.permutation(T)[:T // 8]] = -1
    k, v = (torch.randn(T, H_k, d, device="cuda").half() for _ in range(2))
    ds, got = dev(slots), []
    for step in (T, 32):
        c = [torch.zeros(NB, H_k, 16 * d * (1 if fp8 else 2), dtype=torch.uint8, device="cuda") for _ in range(2)]
        c += [torch.zeros(NB, H_k, 16, device="cuda") for _ in range(2)] if fp8 else []
        for i in range(0, T, step):
            (coopt.kv_cache_write_fp8 if fp8 else coopt.kv_cache_write_fp16)(k[i:i + step], v[i:i + step], ds[i:i + step], *c, shape)
        torch.cuda.synchronize()
        got.append(c)
    assert all(torch.equal(a, b) for a, b in zip(*got))
