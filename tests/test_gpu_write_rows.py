"""GPU: the cache write on both sides of the line between a wavefront per row and the bulk kernel (2560 rows
of a one-byte cache, 1536 of an fp16 one), its large calls, and skip sets on either side of both."""
import numpy as np
import pytest
import torch

import paper_2602_09323_amd as coopt
from gpu_utils import dev

pytestmark = pytest.mark.gpu


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


@pytest.mark.parametrize("kv_dtype,d,H_k,T", [("e4m3", 128, 32, 422), ("e4m3", 64, 33, 425), ("e5m2", 128, 40, 259), ("fp16", 128, 24, 422),
                                              ("fp16", 64, 32, 423), ("e4m3", 128, 40, 3901), ("e5m2", 64, 40, 12802),
                                              ("fp16", 128, 40, 2963)])
def test_skip_set_of_a_bulk_call(kv_dtype, d, H_k, T):
    """One call, the last three of 120 or 200 MB and more, against calls of 32 tokens (a word of the bitmap each), a
    wavefront per row.  Tokens out of the set's reach lie around each skipped one: inside V quads, at the first and
    last tokens of windows, beside negative slots and lone tokens.  What is skipped keeps its bytes."""
    kv = {"e4m3": coopt.COOPT_KV_E4M3, "e5m2": coopt.COOPT_KV_E5M2, "fp16": coopt.COOPT_KV_FP16}[kv_dtype]
    NB, fp8 = T // 16 + 40, kv_dtype != "fp16"
    assert T >= 64 and T * H_k > (2560 if fp8 else 1536)
    shape = coopt.Shape(1, H_k, H_k, d, 16, NB, NB, kv, 1.0)
    rng = np.random.default_rng(T)
    slots = np.concatenate([np.arange(5, 5 + T // 2), T // 2 + 8 + rng.permutation(T // 4),
                            3 * T // 4 + 27 + np.arange(T - T // 2 - T // 4)])
    slots[rng.permutation(T)[:T // 16]] = -1
    skipped = rng.random(T) < 0.2
    window = {("fp16", 128): 13, ("fp16", 64): 29}.get((kv_dtype, d), 29 if d == 128 else 61)
    at = np.arange(T)
    skipped |= (at % (3 * window) == 0) | (at % (5 * window) == window - 1)
    skipped[[0, T - 1]] = True
    bits = np.packbits(np.pad(skipped, (0, -T % 32)), bitorder="little").view(np.uint32)
    k, v = (torch.randn(T, H_k, d, device="cuda").half() for _ in range(2))
    ds, db, got = dev(slots), dev(bits.view(np.int32)), []
    for step in (T, 32):
        c = [torch.full((NB, H_k, 16 * d * (1 if fp8 else 2)), 0xA5, dtype=torch.uint8, device="cuda") for _ in range(2)]
        c += [torch.full((NB, H_k, 16), -1.0, device="cuda") for _ in range(2)] if fp8 else [None, None]
        for i in range(0, T, step):
            coopt.kv_cache_write_skipset(k[i:i + step], v[i:i + step], ds[i:i + step], db[i // 32:(i + step + 31) // 32], *c, shape)
        torch.cuda.synchronize()
        got.append(c[:4 if fp8 else 2])
    assert all(torch.equal(a, b) for a, b in zip(*got))
    if fp8:
        kept = torch.ones(NB * 16, dtype=torch.bool)
        kept[torch.from_numpy(slots[(slots >= 0) & ~skipped])] = False
        for scale in got[0][2:]:
            assert torch.equal((scale.permute(0, 2, 1).reshape(NB * 16, H_k) == -1.0).cpu(), kept[:, None].expand(-1, H_k))
