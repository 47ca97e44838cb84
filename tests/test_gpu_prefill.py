"""GPU parity: chunked prefill over the paged cache and the dequantising gather."""
import numpy as np
import pytest
import torch

import paper_2602_09323_amd as coopt
import workloads
from gpu_utils import alloc_dev_cache, assert_close, cache_to_dev, dev, hip_write, shape_of
from helpers import oracle_fill, v_logical, v_store_logical

pytestmark = pytest.mark.gpu


def _prefill_call(with_workspace, q, dcache, bt, dl, qs, rows, max_chunk, out, shape):
    """The plain entry point, or the one that takes a workspace for the launch's last round (the
    workspace poisoned with NaN: whatever the merge reads must have been written by this call).
    Returns the workspace size the shape asks for."""
    if not with_workspace:
        coopt.paged_gqa_prefill_chunk(q, *dcache, bt, dl, qs, rows, max_chunk, out, shape)
        return 0
    need = coopt.prefill_workspace_bytes(shape, max_chunk)
    ws = torch.full((need // 4,), float("nan"), dtype=torch.float32, device="cuda") if need else None
    coopt.paged_gqa_prefill_chunk_ws(q, *dcache, bt, dl, qs, rows, max_chunk, out, ws, shape)
    return need


def _hip_prefill(w, dcache, lens=None, query_start=None, max_chunk=None, with_workspace=False):
    shape = shape_of(w)
    qs = w.query_start if query_start is None else query_start
    n_rows = int(qs[-1])
    out = torch.full((n_rows, w.H_q, w.d), -7.0, dtype=torch.float16, device="cuda")
    _prefill_call(with_workspace, dev(w.q.view(np.uint16)), dcache, dev(w.block_tables),
                  dev(w.context_lens if lens is None else lens), dev(qs), n_rows,
                  w.new_per_seq if max_chunk is None else max_chunk, out, shape)
    torch.cuda.synchronize()
    return out.cpu().numpy().astype(np.float64)


def _oracle_prefill(oracle, w, cache, rows=None):
    return oracle.paged_gqa_prefill_chunk(w.q, *cache, w.block_tables, w.context_lens,
                                          w.query_start, H_q=w.H_q, H_k=w.H_k, d=w.d, B=w.B,
                                          softmax_scale=w.softmax_scale, rows=rows)


@pytest.mark.parametrize("kv_dtype", ["e4m3", "fp16"])
@pytest.mark.parametrize("ctx,C,H_q,H_k,d", [(40, 24, 10, 2, 128), (0, 33, 4, 2, 64), (100, 1, 5, 1, 128),
                                             (7, 130, 6, 3, 128), (256, 64, 40, 8, 128)])
def test_small_chunks(oracle_mod, kv_dtype, ctx, C, H_q, H_k, d):
    """A few workgroups only.  Through the entry point with a workspace such a launch is all "last
    round": every pair's stages are cut into up to eight runs (more runs than some of these
    streams have stages, so some parts are empty), one workgroup each, and merged."""
    w = workloads.make_custom("pf", seed=51, S=3, H_q=H_q, H_k=H_k, d=d, B=16, NB=96,
                              context_lens=[ctx + C] * 3, new_per_seq=C, kv_dtype=kv_dtype)
    cache = oracle_fill(oracle_mod, w)
    ref = _oracle_prefill(oracle_mod, w, cache)
    dcache = cache_to_dev(cache)
    assert_close(_hip_prefill(w, dcache), ref, f"prefill ctx={ctx} C={C} {kv_dtype}")
    assert coopt.prefill_workspace_bytes(shape_of(w), C) > 0
    assert_close(_hip_prefill(w, dcache, with_workspace=True), ref, f"prefill ctx={ctx} C={C} {kv_dtype}, workspace")


@pytest.mark.parametrize("kv_dtype", ["e4m3", "e5m2", "fp16"])
def test_one_sequence_spread_over_the_chip(oracle_mod, kv_dtype):
    """One sequence's chunk (8 KV heads: 8 pairs of 125 tiles = 64 workgroups) over a history of
    3000 tokens: with a workspace its stages are cut into four runs per 16 tiles."""
    C, hist = 400, 3000
    w = workloads.make_custom("pf_one", seed=57, S=1, H_q=40, H_k=8, d=128, B=16, NB=230,
                              context_lens=[hist + C], new_per_seq=C, kv_dtype=kv_dtype)
    cache = oracle_fill(oracle_mod, w)
    ref = oracle_mod.paged_gqa_prefill_chunk(w.q, *cache, w.block_tables, w.context_lens, w.query_start,
                                             H_q=w.H_q, H_k=w.H_k, d=w.d, B=w.B, softmax_scale=w.softmax_scale,
                                             fmt="e5m2" if kv_dtype == "e5m2" else "e4m3")
    shape = shape_of(w)
    # 125 tiles a pair = 8 workgroups: 64 in the launch, four parts of each fill the 256 CUs
    assert coopt.prefill_workspace_bytes(shape, C) == 8 * 125 * 4 * 16 * 130 * 4
    dcache = cache_to_dev(cache)
    assert_close(_hip_prefill(w, dcache), ref, f"one sequence {kv_dtype}")
    assert_close(_hip_prefill(w, dcache, with_workspace=True), ref, f"one sequence {kv_dtype}, workspace")


def test_chunk_written_on_device_then_attended(oracle_mod):
    w = workloads.make(4, shrink=16)
    cache = oracle_fill(oracle_mod, w)
    ref = _oracle_prefill(oracle_mod, w, cache)
    devc = alloc_dev_cache(w, fill_byte=0x7F)
    hip_write(w, devc, idx=w.history_index())
    hip_write(w, devc, idx=w.new_index())
    assert_close(_hip_prefill(w, devc), ref, "cfg4/16")


@pytest.mark.parametrize("with_workspace", [False, True])
@pytest.mark.parametrize("kv_dtype,chunks", [("e4m3", [512] * 8), ("fp16", [512, 500, 17, 512, 1, 300, 512, 496]),
                                             ("e5m2", [512, 40, 512, 512, 130, 512, 3, 512])])
def test_two_launch_split_every_row(oracle_mod, kv_dtype, chunks, with_workspace):
    """As many workgroups as the full configuration (64 pairs, up to 160 tiles each), so the entry
    point splits the work into its two launches, over a short history so that the oracle can check
    every row; the other cases have a different chunk length per sequence.  With a workspace one
    launch holds the whole streams and workgroups that stream half of a pair's stages each, and the
    other merges the halves (histories of 0 to 250 tokens: halves of one to five stages, and
    sequences whose last tiles do not exist)."""
    S, H_q, H_k, d = len(chunks), 40, 8, 128
    history = [48, 0, 100, 16, 33, 64, 7, 250]
    lens = [h + c for h, c in zip(history, chunks)]
    w = workloads.make_custom("split", seed=77, S=S, H_q=H_q, H_k=H_k, d=d, B=16, NB=512,
                              context_lens=lens, kv_dtype=kv_dtype)
    query_start = np.zeros(S + 1, dtype=np.int32)
    query_start[1:] = np.cumsum(chunks)
    rows = int(query_start[-1])
    q = np.random.default_rng(78).standard_normal((rows, H_q, d), dtype=np.float32).astype(np.float16)
    cache = oracle_fill(oracle_mod, w)
    ref = oracle_mod.paged_gqa_prefill_chunk(q, *cache, w.block_tables, w.context_lens, query_start, H_q=H_q,
                                             H_k=H_k, d=d, B=16, softmax_scale=w.softmax_scale,
                                             fmt="e5m2" if kv_dtype == "e5m2" else "e4m3")
    out = torch.full((rows, H_q, d), -7.0, dtype=torch.float16, device="cuda")
    need = _prefill_call(with_workspace, dev(q.view(np.uint16)), cache_to_dev(cache), dev(w.block_tables),
                         dev(w.context_lens), dev(query_start), rows, max(chunks), out, shape_of(w))
    torch.cuda.synchronize()
    assert not with_workspace or need > 0          # this shape does have a partly filled last round
    assert_close(out.cpu().numpy().astype(np.float64), ref, f"two launches {kv_dtype} {chunks}")


@pytest.mark.parametrize("with_workspace", [False, True])
@pytest.mark.parametrize("kv_dtype,max_blocks", [("e4m3", 32), ("e4m3", 400), ("fp16", 32)])
def test_order_of_tiles_and_workgroups(oracle_mod, kv_dtype, max_blocks, with_workspace):
    """48 pairs of up to 95 tiles: with a workspace 80 of them whole and 15 split, so the cut lies
    inside the fifth head (tile 80 = head 4, rows 64..79), and every sequence has its own number of
    tiles: none of the split ones, some, all.  The 32-block table keeps an XCD's streams within its
    L2 (workgroups turn by turn), the 400-block one does not (pair by pair); histories longer and
    shorter than a third of the chunk put the split workgroups behind, among or ahead of the rest."""
    chunks, history = [300, 299, 33, 1, 150, 290], [0, 210, 16, 130, 40, 3]
    S, H_q, H_k, d = len(chunks), 40, 8, 128
    w = workloads.make_custom("order", seed=91, S=S, H_q=H_q, H_k=H_k, d=d, B=16, NB=160, max_blocks=max_blocks,
                              context_lens=[h + c for h, c in zip(history, chunks)], kv_dtype=kv_dtype)
    query_start = np.zeros(S + 1, dtype=np.int32)
    query_start[1:] = np.cumsum(chunks)
    rows = int(query_start[-1])
    q = np.random.default_rng(92).standard_normal((rows, H_q, d), dtype=np.float32).astype(np.float16)
    cache = oracle_fill(oracle_mod, w)
    ref = oracle_mod.paged_gqa_prefill_chunk(q, *cache, w.block_tables, w.context_lens, query_start, H_q=H_q,
                                             H_k=H_k, d=d, B=16, softmax_scale=w.softmax_scale)
    out = torch.full((rows, H_q, d), -7.0, dtype=torch.float16, device="cuda")
    need = _prefill_call(with_workspace, dev(q.view(np.uint16)), cache_to_dev(cache), dev(w.block_tables),
                         dev(w.context_lens), dev(query_start), rows, max(chunks), out, shape_of(w))
    torch.cuda.synchronize()
    assert not with_workspace or need == S * H_k * 15 * 5 * 16 * 130 * 4
    assert_close(out.cpu().numpy().astype(np.float64), ref, f"order {kv_dtype} {max_blocks}")


@pytest.mark.parametrize("S,H_q,H_k,d,hist,C,parts", [(2, 40, 8, 128, 544, 400, 2), (1, 40, 40, 128, 1056, 333, 3),
                                                       (8, 40, 8, 64, 512, 16, 4), (1, 40, 8, 128, 1024, 16, 7)])
def test_infinite_value_rows(oracle_mod, S, H_q, H_k, d, hist, C, parts):
    """An uncompressed cache may hold an infinity.  Every query row sees the token at the history's
    end (in the last run of a split stream) with +inf in one dimension of its value row, and token 1
    (in the first run) with -inf in another: those two outputs are the infinities themselves through
    both entry points, whatever the number of runs the merge combines, and the other dimensions are
    what they are without them."""
    w = workloads.make_custom("inf", seed=58, S=S, H_q=H_q, H_k=H_k, d=d, B=16, NB=S * ((hist + C) // 16 + 2),
                              context_lens=[hist + C] * S, new_per_seq=C, kv_dtype="fp16")
    cache = oracle_fill(oracle_mod, w)
    ref = _oracle_prefill(oracle_mod, w, cache)
    v = v_logical(w, cache[1])
    for s in range(S):
        v[w.block_tables[s, (hist - 1) // 16], :, (hist - 1) % 16, 3] = np.inf
        v[w.block_tables[s, 0], :, 1, 7] = -np.inf
    v_store_logical(w, cache[1], v)
    tiles = H_q // H_k * ((C + 15) // 16)
    assert coopt.prefill_workspace_bytes(shape_of(w), C) == S * H_k * tiles * parts * 16 * (d + 2) * 4
    dcache = cache_to_dev(cache)
    for with_workspace in (False, True):
        got = _hip_prefill(w, dcache, with_workspace=with_workspace)
        assert (got[..., 3] == np.inf).all() and (got[..., 7] == -np.inf).all(), f"workspace: {with_workspace}"
        rest = np.delete(np.arange(d), (3, 7))
        assert_close(got[..., rest], ref[..., rest], f"infinite values, workspace: {with_workspace}")


def test_longer_chunk_than_announced(oracle_mod):
    """A sequence with more rows than `max_chunk_len` says: nothing is written beyond the workspace that
    was asked for, and the other sequence's rows are what they are without it."""
    chunks, announced = [64, 400], 64
    w = workloads.make_custom("over", seed=59, S=2, H_q=40, H_k=8, d=128, B=16, NB=64,
                              context_lens=[264, 600], kv_dtype="e4m3")
    query_start = np.array([0, 64, 464], dtype=np.int32)
    q = np.random.default_rng(60).standard_normal((464, 40, 128), dtype=np.float32).astype(np.float16)
    cache = oracle_fill(oracle_mod, w)
    ref = oracle_mod.paged_gqa_prefill_chunk(q, *cache, w.block_tables, w.context_lens, query_start, H_q=40, H_k=8,
                                             d=128, B=16, softmax_scale=w.softmax_scale)
    shape, out = shape_of(w), torch.full((464, 40, 128), -7.0, dtype=torch.float16, device="cuda")
    need = coopt.prefill_workspace_bytes(shape, announced)
    whole = coopt.prefill_workspace_bytes(shape, max(chunks))
    buf = torch.full((need + 4 * whole,), 0x5A, dtype=torch.uint8, device="cuda")      # the workspace, and what lies behind
    coopt.paged_gqa_prefill_chunk_ws(dev(q.view(np.uint16)), *cache_to_dev(cache), dev(w.block_tables),
                                     dev(w.context_lens), dev(query_start), 464, announced, out, buf[:need], shape)
    torch.cuda.synchronize()
    assert need > 0 and bool((buf[need:] == 0x5A).all())
    got = out.cpu().numpy().astype(np.float64)
    assert_close(got[:64], ref[:64], "the sequence as announced")
    written = (got[64:] != -7.0).any(axis=2)
    assert_close(got[64:][written], ref[64:][written], "what is written of the longer one")


@pytest.mark.parametrize("kv_dtype", ["e4m3", "e5m2"])
@pytest.mark.parametrize("S,C,limit,rest,parts", [(8, 352, 64, 46, 4), (3, 777, 160, 85, 5)])
def test_tiles_that_are_not_split_are_the_same_bits(S, C, limit, rest, parts, kv_dtype):
    """Fresh prompts for which the entry point without a workspace makes one launch of full workgroups
    and the one with a workspace splits the tiles from `limit` on.  The value rows grow along the prompt,
    so the normaliser of the v_scales -- taken over the rows of a workgroup -- tells which rows a tile
    was grouped with: tiles below `limit` have the same bits from both."""
    H_q, H_k, d = 40, 8, 128
    w = workloads.make_custom("bits", seed=61, S=S, H_q=H_q, H_k=H_k, d=d, B=16, NB=S * (C // 16 + 2),
                              context_lens=[C] * S, new_per_seq=C, kv_dtype=kv_dtype)
    grow = np.exp2((np.arange(len(w.slots)) % C) / 64.0).astype(np.float16)
    w.v_ctx = (w.v_ctx * grow[:, None, None]).astype(np.float16)
    dcache = alloc_dev_cache(w)
    hip_write(w, dcache)
    assert coopt.prefill_workspace_bytes(shape_of(w), C) == S * H_k * rest * parts * 16 * 130 * 4
    plain, split = (_hip_prefill(w, dcache, with_workspace=ws) for ws in (False, True))
    tiles_per_head = (C + 15) // 16
    tile = np.arange(H_q)[None, :] % (H_q // H_k) * tiles_per_head + (np.arange(S * C)[:, None] % C) // 16
    same = (plain == split).all(axis=2)                         # [row, head]
    assert same[tile < limit].all(), f"{int((~same[tile < limit]).sum())} rows differ"
    # (the others: two roundings to fp16, 2^-11 of the value each, and 2^-10 of the arithmetic's)
    assert np.abs(plain - split).max() <= 2e-3 * np.abs(plain).max()


def test_chunked_prefill_full_size(oracle_mod, record_property):
    """Full configuration in the launch shape the benchmark times.  The oracle computes every row
    of one whole sequence (512 rows x 40 heads over 8192 + 512 tokens: the stage pipeline 136
    stages deep, every tile, whole and split) and, of the other sequences, a sample of rows
    (first, last, tile edges, random).  About a minute and a half of oracle time on 16 cores."""
    w = workloads.make(4)
    print(f"full cfg4: tokens={w.total_tokens}", flush=True)
    cache = oracle_fill(oracle_mod, w)
    dcache = cache_to_dev(cache)
    got = _hip_prefill(w, dcache)
    got_ws = _hip_prefill(w, dcache, with_workspace=True)
    assert np.isfinite(got).all() and np.isfinite(got_ws).all()
    rng = np.random.default_rng(0)
    C = w.new_per_seq
    local = np.array([0, 1, 15, 16, 17, C // 2, C - 2, C - 1])
    rows = np.unique(np.concatenate([local, (w.S - 1) * C + local, rng.integers(0, w.S * C, 8)])).astype(np.int32)
    ref_rows = _oracle_prefill(oracle_mod, w, cache, rows=rows)
    print("full cfg4 sample max-abs %.2e" % assert_close(got[rows], ref_rows, "cfg4 sample", record_property), flush=True)
    whole = np.arange(5 * C, 6 * C, dtype=np.int32)                  # sequence 5, every row
    ref = _oracle_prefill(oracle_mod, w, cache, rows=whole)
    print("full cfg4 sequence 5, every row: max-abs %.2e" %
          assert_close(got[whole], ref, "cfg4 whole sequence", record_property), flush=True)
    # the entry point with a workspace (the last 32 tiles of every pair in two halves + a merge):
    # the same rows of the other tiles bit for bit, every checked row within the bar
    print("full cfg4 with workspace, sequence 5: max-abs %.2e" %
          assert_close(got_ws[whole], ref, "cfg4 whole sequence, workspace", record_property), flush=True)
    assert_close(got_ws[rows], ref_rows, "cfg4 sample, workspace")
    same = (got_ws == got).all(axis=2)                         # [row, head]
    tiles_per_head = C // 16
    tile = np.arange(w.H_q)[None, :] % (w.H_q // w.H_k) * tiles_per_head + (np.arange(w.S * C)[:, None] % C) // 16
    assert same[tile < 128].all(), "rows of whole streams differ between the two entry points"


def test_gather_cached_kv(oracle_mod):
    """Bit-exact: the device rounds code * scale to fp16 once, like the oracle's exact product."""
    for kv_dtype in ("e4m3", "fp16"):
        for d, H_k in ((128, 2), (64, 3)):
            w = workloads.make_custom("ga", seed=52 + d, S=2, H_q=2 * H_k, H_k=H_k, d=d, B=16, NB=24,
                                      context_lens=[150, 25], kv_dtype=kv_dtype)
            cache = oracle_fill(oracle_mod, w)
            dcache = cache_to_dev(cache)
            for seq, lo, hi in ((0, 3, 61), (0, 0, 150), (0, 16, 144), (0, 149, 150), (1, 7, 25), (1, 0, 16)):
                kref, vref = oracle_mod.gather_cached_kv(*cache, w.block_tables, seq, lo, hi, H_k=H_k, d=d, B=16)
                k_out = torch.full((hi - lo + 2, H_k, d), 7.0, dtype=torch.float16, device="cuda")
                v_out = torch.full_like(k_out, 7.0)
                coopt.gather_cached_kv(*dcache, dev(w.block_tables), seq, lo, hi, k_out[1:-1], v_out[1:-1], shape_of(w))
                torch.cuda.synchronize()
                for got, ref in ((k_out, kref), (v_out, vref)):
                    got = got.cpu().numpy()
                    assert np.all(got[0] == 7.0) and np.all(got[-1] == 7.0)      # nothing outside the range
                    want = ref.astype(np.float16)                                  # one rounding of the exact product
                    assert np.array_equal(got[1:-1].view(np.uint16), want.view(np.uint16)), (kv_dtype, d, seq, lo, hi)
