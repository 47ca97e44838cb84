"""GPU parity: chunked prefill where its launch takes another form than the one that the other tests reach --
ragged batches whose workgroups start in the order of their streams' lengths, workgroups of eight tiles,
split plans that run some or all sequences whole -- and factors that the kernel folds away."""
import numpy as np
import pytest
import torch

import paper_2602_09323_amd as coopt
import workloads
from gpu_utils import assert_close, cache_to_dev, dev, shape_of
from helpers import oracle_fill
from test_gpu_prefill import _prefill_call

pytestmark = pytest.mark.gpu


def _run(oracle_mod, kv_dtype, H_q, H_k, d, chunks, history, max_blocks=None, scale=None, offset=0):
    """Rows through both entry points against the oracle; returns the workspace's size."""
    S, lens = len(chunks), [h + c for h, c in zip(history, chunks)]
    w = workloads.make_custom("forms", seed=131, S=S, H_q=H_q, H_k=H_k, d=d, B=16, NB=sum((t + 15) // 16 for t in lens) + 4,
                              context_lens=lens, kv_dtype=kv_dtype, max_blocks=max_blocks)
    if scale is not None:
        w.softmax_scale = scale
    starts = np.zeros(S + 1, dtype=np.int32)
    starts[1:] = np.cumsum(chunks)
    rows = int(starts[-1])
    q = np.random.default_rng(132).standard_normal((rows, H_q, d), dtype=np.float32).astype(np.float16)
    cache = oracle_fill(oracle_mod, w)
    ref = oracle_mod.paged_gqa_prefill_chunk(q, *cache, w.block_tables, w.context_lens, starts, H_q=H_q, H_k=H_k, d=d, B=16,
                                             softmax_scale=w.softmax_scale, fmt="e5m2" if kv_dtype == "e5m2" else "e4m3")
    dcache, need = cache_to_dev(cache), 0
    held = torch.zeros(q.size + offset, dtype=torch.float16, device="cuda")       # (rows may begin at any 2-byte boundary)
    held[offset:] = dev(q.reshape(-1).view(np.uint16)).view(torch.float16)
    for with_workspace in (False, True):
        out = torch.full((rows * H_q * d + offset,), -7.0, dtype=torch.float16, device="cuda")[offset:].view(rows, H_q, d)
        need = _prefill_call(with_workspace, held[offset:].view(rows, H_q, d), dcache, dev(w.block_tables), dev(w.context_lens),
                             dev(starts), rows, max(chunks), out, shape_of(w))
        torch.cuda.synchronize()
        assert_close(out.cpu().numpy().astype(np.float64), ref, f"{kv_dtype} {H_q}/{H_k} x {d}, workspace {with_workspace}")
    return need


@pytest.mark.parametrize("kv_dtype,d", [("e4m3", 128), ("fp16", 64)])
def test_ragged_batch_by_length(oracle_mod, kv_dtype, d):
    """192 pairs of up to six workgroups, 53 % of the rows: more than four workgroups a CU, ranked."""
    chunks = [260 - 11 * (s % 23) for s in range(24)]
    chunks[5], chunks[17] = 1, 16
    history = [(37 * s) % 90 for s in range(24)]
    assert 4 * sum(chunks) <= 3 * 24 * max(chunks) and 192 * 6 >= 1024
    _run(oracle_mod, kv_dtype, 40, 8, d, chunks, history)


@pytest.mark.parametrize("kv_dtype,H_q,H_k,d", [("e4m3", 40, 8, 128), ("e5m2", 32, 8, 64), ("fp16", 16, 2, 128), ("fp16", 8, 2, 64)])
@pytest.mark.parametrize("history", [0, 100, 129, 700, 1500])
def test_eight_tiles(oracle_mod, kv_dtype, H_q, H_k, d, history):
    """Chunks of at most 16 rows: 4 to 8 tiles a pair, of which the last wavefront may have one."""
    _run(oracle_mod, kv_dtype, H_q, H_k, d, [16, 9, 1], [history, history + 31, max(history - 13, 0)])


@pytest.mark.parametrize("kv_dtype", ["e4m3", "fp16"])
def test_split_plan_runs_short_sequences_whole(oracle_mod, kv_dtype):
    """3 x 390 rows over 8 heads: quarters in three rounds, so sequences of up to 2304 tokens run whole and the
    longer one splits.  Then all of them short, by a table that says so."""
    chunks = [390, 390, 200]
    assert _run(oracle_mod, kv_dtype, 40, 8, 128, chunks, [0, 3000, 700]) > 0
    assert _run(oracle_mod, kv_dtype, 40, 8, 128, chunks, [0, 50, 100]) > 0


@pytest.mark.parametrize("kv_dtype", ["e4m3", "fp16"])
@pytest.mark.parametrize("scale", [-0.09, 0.0])
def test_softmax_scale_of_any_sign(oracle_mod, kv_dtype, scale):
    _run(oracle_mod, kv_dtype, 10, 2, 128, [130, 40], [300, 20], scale=scale)


@pytest.mark.parametrize("offset", [1, 4])
def test_rows_at_any_boundary(oracle_mod, offset):
    _run(oracle_mod, "e4m3", 10, 2, 64, [70, 33], [200, 0], offset=offset)
