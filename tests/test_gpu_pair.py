"""GPU parity: few pairs without a plan, where decode and the fused step are one launch of a workgroup
per (sequence, KV head) pair, or, for longer contexts, one of several workgroups per pair and the merge.
Against the oracle, at the edges of blocks, two-block groups and of the wavefronts and workgroups that
share a pair's groups; the step's cache bytes bit for bit; and the shapes at which one form takes over
from the other."""
import numpy as np
import pytest
import torch

import paper_2602_09323_amd as coopt
import workloads
from gpu_utils import alloc_dev_cache, assert_close, cache_to_dev, dev, dev_cache_to_host, hip_write, shape_of
from helpers import oracle_fill

pytestmark = pytest.mark.gpu

LENS = [0, 1, 2, 15, 16, 17, 31, 32, 33, 47, 64, 225, 255, 256, 257, 288, 511, 512]


def _workload(kv_dtype, H_q, H_k, d, lens=LENS, max_blocks=32):
    return workloads.make_custom("pair", seed=101, S=len(lens), H_q=H_q, H_k=H_k, d=d, B=16,
                                 NB=sum((t + 15) // 16 for t in lens) + 4, context_lens=lens,
                                 kv_dtype=kv_dtype, max_blocks=max_blocks)


def _oracle(oracle_mod, w, cache, kv_dtype, lens=None):
    return oracle_mod.paged_gqa_decode(w.q, *cache, w.block_tables, w.context_lens if lens is None else lens, H_q=w.H_q,
                                       H_k=w.H_k, d=w.d, B=w.B, softmax_scale=w.softmax_scale,
                                       fmt="e5m2" if kv_dtype == "e5m2" else "e4m3")


def _out(w):
    # (rows begin at a 2-byte boundary)
    return torch.full((w.S * w.H_q * w.d + 1,), -7.0, dtype=torch.float16, device="cuda")[1:].view(w.S, w.H_q, w.d)


@pytest.mark.parametrize("kv_dtype,H_q,H_k,d", [("e4m3", 40, 8, 128), ("e5m2", 32, 2, 64), ("fp16", 10, 2, 64),
                                                ("e4m3", 3, 3, 64), ("e5m2", 5, 1, 128)])
def test_decode(oracle_mod, kv_dtype, H_q, H_k, d):
    w = _workload(kv_dtype, H_q, H_k, d)
    cache = oracle_fill(oracle_mod, w)
    ref = _oracle(oracle_mod, w, cache, kv_dtype)
    shape, dcache = shape_of(w), cache_to_dev(cache)
    args = dev(w.q.view(np.uint16)), *dcache, dev(w.block_tables), dev(w.context_lens)
    ws = torch.empty(coopt.decode_workspace_bytes(shape), dtype=torch.uint8, device="cuda")
    ws.fill_(0x5A)
    outs = [_out(w) for _ in range(3)]
    coopt.paged_gqa_decode(*args, outs[0], ws, shape)
    coopt.paged_gqa_decode(*args, outs[1], None, shape)
    coopt.paged_gqa_decode_noalloc(*args, outs[2], shape)
    torch.cuda.synchronize()
    assert bool((ws == 0x5A).all())                            # one launch: no partials in memory
    assert_close(outs[0].cpu().numpy().astype(np.float64), ref, f"{kv_dtype} {H_q}/{H_k} x {d}")
    assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2])


@pytest.mark.parametrize("kv_dtype,H_q,H_k,d", [("e4m3", 40, 8, 128), ("e5m2", 32, 2, 64), ("fp16", 10, 2, 64),
                                                ("fp16", 5, 1, 128)])
def test_step(oracle_mod, kv_dtype, H_q, H_k, d):
    """Every third sequence's slot is negative: nothing is written and it attends to what is there."""
    lens = LENS if kv_dtype != "fp16" or d == 64 else [t for t in LENS if t <= 256]
    w = _workload(kv_dtype, H_q, H_k, d, lens, (max(lens) + 15) // 16)
    cache = oracle_fill(oracle_mod, w)
    ref = _oracle(oracle_mod, w, cache, kv_dtype)
    shape = shape_of(w)
    new = [int(np.sum(lens[:s + 1])) - 1 for s in range(w.S)]         # a sequence's last row; some row for an empty one
    new = np.maximum(new, 0)
    skipped = np.arange(w.S) % 3 == 1
    slots = np.where(skipped | (np.asarray(lens) == 0), -1, w.slots[new])
    dcache = alloc_dev_cache(w, fill_byte=0)
    before = [i for i in range(len(w.slots)) if i not in set(new[(slots >= 0)])]
    hip_write(w, dcache, idx=np.asarray(before))
    out = _out(w)
    ws = torch.full((coopt.decode_workspace_bytes(shape),), 0x5A, dtype=torch.uint8, device="cuda")
    coopt.paged_gqa_decode_step(dev(w.k_ctx[new].view(np.uint16)), dev(w.v_ctx[new].view(np.uint16)), dev(slots),
                                dev(w.q.view(np.uint16)), *dcache, dev(w.block_tables), dev(w.context_lens), out, ws, shape)
    torch.cuda.synchronize()
    assert bool((ws == 0x5A).all())
    assert_close(out.cpu().numpy().astype(np.float64), ref, f"step {kv_dtype} {H_q}/{H_k} x {d}")
    for name, got, want in zip(("k_cache", "v_cache", "k_scale", "v_scale"), dev_cache_to_host(w, dcache), cache):
        if want is not None:
            assert np.array_equal(got.reshape(-1).view(np.uint8), want.reshape(-1).view(np.uint8)), name


PART_LENS = [0, 1, 17, 33, 127, 128, 129, 256, 257, 545, 900, 1025]


@pytest.mark.parametrize("step", [False, True], ids=["decode", "step"])
@pytest.mark.parametrize("kv_dtype,H_q,H_k,d,lens,max_blocks", [
    ("e4m3", 40, 8, 128, [1789], 112),                   # 14 parts of four groups
    ("e4m3", 40, 8, 128, PART_LENS, 80),                 # 96 pairs: two parts of five turns
    ("e5m2", 32, 2, 64, PART_LENS, 130),                 # ten parts, two turns
    ("fp16", 10, 2, 64, PART_LENS, 66),
    ("fp16", 5, 1, 128, [3000, 1, 2999, 0, 1500], 188),
    ("e4m3", 16, 16, 64, PART_LENS[1:] * 2, 66),         # 352 pairs: more groups than the form takes
    ("e4m3", 16, 8, 64, [0, 1, 33, 150, 160, 17] * 10, 10),     # 480 pairs of 64 dims: one workgroup each, beyond the CUs
    ("fp16", 8, 8, 64, [129, 0, 255, 31] * 9, 16)])
def test_in_parts(oracle_mod, kv_dtype, H_q, H_k, d, lens, max_blocks, step):
    w = _workload(kv_dtype, H_q, H_k, d, lens, max_blocks)
    groups = len(lens) * H_k * ((max_blocks + 1) // 2)
    assert groups <= 5120 or H_k == 16
    cache = oracle_fill(oracle_mod, w)
    ref = _oracle(oracle_mod, w, cache, kv_dtype)
    shape, out = shape_of(w), _out(w)
    ws = torch.full((coopt.decode_workspace_bytes(shape) // 4,), float("nan"), device="cuda")     # what is read was written
    tail = dev(w.block_tables), dev(w.context_lens), out, ws, shape
    if not step:
        coopt.paged_gqa_decode(dev(w.q.view(np.uint16)), *cache_to_dev(cache), *tail)
    else:
        new = np.maximum(np.cumsum(lens) - 1, 0)
        slots = np.where(np.asarray(lens) == 0, -1, w.slots[new])
        dcache = alloc_dev_cache(w, fill_byte=0)
        hip_write(w, dcache, idx=np.asarray(sorted(set(range(len(w.slots))) - set(new[slots >= 0]))))
        coopt.paged_gqa_decode_step(dev(w.k_ctx[new].view(np.uint16)), dev(w.v_ctx[new].view(np.uint16)), dev(slots),
                                    dev(w.q.view(np.uint16)), *dcache, *tail)
        torch.cuda.synchronize()
        for name, got, want in zip(("k_cache", "v_cache", "k_scale", "v_scale"), dev_cache_to_host(w, dcache), cache):
            if want is not None:
                assert np.array_equal(got.reshape(-1).view(np.uint8), want.reshape(-1).view(np.uint8)), name
    torch.cuda.synchronize()
    assert_close(out.cpu().numpy().astype(np.float64), ref, f"parts {kv_dtype} {H_q}/{H_k} x {d}")


@pytest.mark.parametrize("S,H_q,H_k,d,max_blocks", [(33, 8, 8, 128, 6), (65, 8, 8, 64, 4), (40, 8, 8, 64, 18), (12, 8, 8, 128, 88),
                                                    (20, 8, 8, 128, 50)])
def test_beyond_the_line_of_parts(S, H_q, H_k, d, max_blocks):
    """More pairs, groups or turns than the form in parts is the faster for: what the default plan, passed as a
    plan, gives, bit for bit."""
    w = _workload("e4m3", H_q, H_k, d, [(37 * s) % (16 * max_blocks) + 1 for s in range(S)], max_blocks)
    shape, dcache = shape_of(w), alloc_dev_cache(w)
    hip_write(w, dcache)
    ws = torch.empty(coopt.decode_workspace_bytes(shape), dtype=torch.uint8, device="cuda")
    outs = [_out(w) for _ in range(2)]
    for out, plan in zip(outs, (None, coopt.default_decode_plan())):
        coopt.paged_gqa_decode(dev(w.q.view(np.uint16)), *dcache, dev(w.block_tables), dev(w.context_lens), out, ws, shape, plan=plan)
    torch.cuda.synchronize()
    assert torch.equal(*outs)


@pytest.mark.parametrize("lens,max_blocks", [([33, 65, 257, 20], 17), ([1025, 129, 33], 130)], ids=["whole", "parts"])
def test_infinite_key(oracle_mod, lens, max_blocks):
    """Every sequence's last key has an infinite element: no weight for the heads whose query is negative there,
    also where a wavefront sees no other token; no number for the others."""
    H_q, H_k, d = 10, 2, 64
    w = _workload("fp16", H_q, H_k, d, lens, max_blocks)
    cache = oracle_fill(oracle_mod, w)
    for s, t in enumerate(lens):                        # K blocks: [dim / 8][token][8]
        cache[0].reshape(w.NB, H_k, d // 8, 16, 8)[w.block_tables[s, (t - 1) // 16], :, 3, (t - 1) % 16, 2] = np.inf
    w.q[:, :, 26] = np.where(np.arange(H_q) % 2, 1, -1)
    with np.errstate(invalid="ignore"):
        ref = _oracle(oracle_mod, w, cache, "fp16")
    shape, out = shape_of(w), _out(w)
    ws = torch.full((coopt.decode_workspace_bytes(shape) // 4,), float("nan"), device="cuda")
    coopt.paged_gqa_decode(dev(w.q.view(np.uint16)), *cache_to_dev(cache), dev(w.block_tables), dev(w.context_lens), out, ws, shape)
    torch.cuda.synchronize()
    got = out.cpu().numpy().astype(np.float64)
    assert np.isnan(ref[:, 1::2]).all() and np.isnan(got[:, 1::2]).all()
    assert_close(got[:, ::2], ref[:, ::2], f"infinite keys, {max_blocks} blocks")


@pytest.mark.parametrize("S,H_q,H_k,d,max_blocks,one_launch", [(32, 8, 8, 128, 33, True), (33, 8, 8, 128, 33, False),
                                                               (2, 4, 2, 128, 33, True), (2, 4, 2, 128, 34, False),
                                                               (2, 4, 2, 64, 64, True), (2, 4, 2, 64, 65, False)])
def test_where_the_balanced_form_takes_over(oracle_mod, S, H_q, H_k, d, max_blocks, one_launch):
    """256 pairs, 140 000 bytes a pair: to either side of both."""
    lens = [(37 * s) % 150 + 1 for s in range(S)]
    w = _workload("e4m3", H_q, H_k, d, lens, max_blocks)
    cache = oracle_fill(oracle_mod, w)
    ref = _oracle(oracle_mod, w, cache, "e4m3")
    shape, out = shape_of(w), _out(w)
    ws = torch.full((coopt.decode_workspace_bytes(shape),), 0x5A, dtype=torch.uint8, device="cuda")
    coopt.paged_gqa_decode(dev(w.q.view(np.uint16)), *cache_to_dev(cache), dev(w.block_tables), dev(w.context_lens), out,
                           ws, shape)
    torch.cuda.synchronize()
    assert bool((ws == 0x5A).all()) == one_launch
    assert_close(out.cpu().numpy().astype(np.float64), ref, f"{S} x {H_k} pairs, {max_blocks} blocks")
