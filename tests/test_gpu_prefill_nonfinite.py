"""GPU parity: chunked prefill over queries, keys and scales that are infinite or NaN.  A wavefront carries two
tiles of 16 rows whose sums share a matrix product: a row that is no number must be the oracle's rows that are
none and no other -- not the row of the same index in the other tile, nor rows in front of a bad key."""
import numpy as np
import pytest
import torch

import workloads
from gpu_utils import assert_close, cache_to_dev, dev, shape_of
from helpers import oracle_fill
from test_gpu_prefill import _prefill_call

pytestmark = pytest.mark.gpu


def _check(oracle_mod, w, cache, q, starts, chunks, bad_rows):
    """Both entry points against the oracle: the same rows NaN, `bad_rows` of them, the others within the bar."""
    with np.errstate(invalid="ignore"):
        ref = oracle_mod.paged_gqa_prefill_chunk(q, *cache, w.block_tables, w.context_lens, starts, H_q=w.H_q, H_k=w.H_k,
                                                 d=w.d, B=w.B, softmax_scale=w.softmax_scale,
                                                 fmt="e5m2" if w.kv_dtype == "e5m2" else "e4m3")
    bad = ~np.isfinite(ref).all(axis=2)
    assert not np.isfinite(ref[bad]).any() and bad_rows(bad), "the oracle's rows are not those that the test is about"
    for with_workspace in (False, True):
        out = torch.full(q.shape, -7.0, dtype=torch.float16, device="cuda")
        _prefill_call(with_workspace, dev(q.view(np.uint16)).view(torch.float16), cache_to_dev(cache), dev(w.block_tables),
                      dev(w.context_lens), dev(starts), len(q), max(chunks), out, shape_of(w))
        torch.cuda.synchronize()
        got = out.cpu().numpy().astype(np.float64)
        what = f"{w.kv_dtype} {w.H_q}/{w.H_k} x {w.d}, workspace {with_workspace}"
        assert np.isnan(got[bad]).all(), what
        assert_close(np.where(bad[..., None], 0.0, got), np.where(bad[..., None], 0.0, ref), what)


def _workload(kv_dtype, H_q, H_k, d, chunks, history):
    lens = [h + c for h, c in zip(history, chunks)]
    w = workloads.make_custom("nonfinite", seed=151, S=len(chunks), H_q=H_q, H_k=H_k, d=d, B=16,
                              NB=sum((t + 15) // 16 for t in lens) + 4, context_lens=lens, kv_dtype=kv_dtype)
    starts = np.zeros(len(chunks) + 1, dtype=np.int32)
    starts[1:] = np.cumsum(chunks)
    q = np.random.default_rng(152).standard_normal((int(starts[-1]), H_q, d), dtype=np.float32).astype(np.float16)
    return w, q, starts


SHAPES = [("e4m3", 10, 2, 128), ("e5m2", 4, 4, 64), ("fp16", 3, 3, 128), ("fp16", 10, 2, 64)]
# (a wave's tiles at neighbouring rows; eight tiles a pair; streams of whole stages, cut into runs)
CHUNKS = [([70, 33], [40, 0]), ([16, 9], [300, 700]), ([200], [3000])]


@pytest.mark.parametrize("chunks,history", CHUNKS)
@pytest.mark.parametrize("kv_dtype,H_q,H_k,d", SHAPES)
def test_query_rows(oracle_mod, kv_dtype, H_q, H_k, d, chunks, history):
    w, q, starts = _workload(kv_dtype, H_q, H_k, d, chunks, history)
    q[5, 1, 3], q[8, 0, d - 1] = np.nan, np.inf
    _check(oracle_mod, w, oracle_fill(oracle_mod, w), q, starts, chunks, lambda bad: bad.sum() == 2 and bad[5, 1] and bad[8, 0])


def _cache_row(w, position):
    """Block and offset of a token of the first sequence."""
    return int(w.block_tables[0, position // 16]), position % 16


@pytest.mark.parametrize("chunks,history", CHUNKS)
@pytest.mark.parametrize("kv_dtype,H_q,H_k,d", SHAPES)
def test_key_inside_the_chunk(oracle_mod, kv_dtype, H_q, H_k, d, chunks, history):
    """Rows in front of the key keep their values."""
    w, q, starts = _workload(kv_dtype, H_q, H_k, d, chunks, history)
    cache = oracle_fill(oracle_mod, w)
    block, at = _cache_row(w, history[0] + 11)
    if kv_dtype == "fp16":
        # K blocks: [dim / 8][token][8]
        cache[0].reshape(w.NB, H_k, d // 8, 16, 8).view(np.uint16)[block, 1, 2, at, 5] = 0x7e00
    else:
        cache[2][block, 1, at] = np.nan
    _check(oracle_mod, w, cache, q, starts, chunks,
           lambda bad: not bad[:11].any() and bad[11:chunks[0], H_q // H_k:2 * H_q // H_k].all())


@pytest.mark.parametrize("H_q,H_k,d", [(3, 3, 128), (10, 2, 64)])
@pytest.mark.parametrize("chunks,history,position", [([70, 33], [40, 0], 20), ([200], [3000], 100), ([200], [3000], 3050)])
def test_infinite_key(oracle_mod, H_q, H_k, d, chunks, history, position):
    """One infinite element: no weight where its product with the query is negative, else no number."""
    w, q, starts = _workload("fp16", H_q, H_k, d, chunks, history)
    cache = oracle_fill(oracle_mod, w)
    block, at = _cache_row(w, position)
    cache[0].reshape(w.NB, H_k, d // 8, 16, 8)[block, 0, 3, at, 2] = np.inf
    q[..., 26] = np.where(q[..., 26] == 0, 1, q[..., 26])                    # (0 * inf is none either)
    _check(oracle_mod, w, cache, q, starts, chunks,
           lambda bad: 0.2 < bad[max(position - history[0], 0):chunks[0], :H_q // H_k].mean() < 0.8)
