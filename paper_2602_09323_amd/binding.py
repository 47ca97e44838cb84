"""ctypes binding of the C ABI in ``include/coopt_attn.h``: same names, argument marshalling only.

Tensors are torch CUDA(HIP) tensors used purely as device memory; every step of the path runs in
the library's own kernels on the current torch stream.  If the shared library is missing the
binding raises: there is no fallback path.

The C side takes raw pointers and cannot see a buffer's size, type or residence, so the binding
checks what it can before anything is launched: every tensor is a contiguous device tensor, index
tensors have the integer width the kernels read (int64 slots, int32 tables / lengths / row
offsets), fp16 operands have 2-byte elements, and every buffer holds at least the bytes the shape
implies.  A violation raises ``CooptError``.
"""
from __future__ import annotations

import ctypes
import os
from typing import Optional

_HERE = os.path.dirname(os.path.abspath(__file__))
_LIB_PATH = os.path.join(_HERE, "libcoopt_attn.so")
_lib = None

COOPT_KV_FP16 = 0
COOPT_KV_E4M3 = 1
COOPT_KV_E5M2 = 2
COOPT_SCALE_TOKEN = 0
COOPT_SCALE_BLOCK = 1
COOPT_SCALE_STATIC = 2

EXPORTS = [
    "coopt_kv_cache_write_fp8", "coopt_kv_cache_write_fp16", "coopt_kv_cache_write_skipset",
    "coopt_kv_cache_write_fp8_scaled",
    "coopt_paged_gqa_decode", "coopt_paged_gqa_decode_step", "coopt_paged_gqa_decode_split",
    "coopt_paged_gqa_decode_merge", "coopt_decode_workspace_bytes", "coopt_default_decode_plan",
    "coopt_paged_gqa_decode_partitioned", "coopt_paged_gqa_reduce", "coopt_paged_gqa_prefill_chunk",
    "coopt_gather_cached_kv", "coopt_decode_schedule_bytes", "coopt_decode_schedule_prepare",
    "coopt_paged_gqa_decode_scheduled", "coopt_status_string",
    "coopt_paged_gqa_decode_noalloc", "coopt_decode_builtin_workspace_bytes",
    "coopt_paged_gqa_prefill_chunk_ws", "coopt_prefill_workspace_bytes",
]


class CooptError(RuntimeError):
    pass


class DecodePlan(ctypes.Structure):
    """Mirror of ``coopt_decode_plan``."""
    _fields_ = [("tokens_per_group", ctypes.c_int32), ("waves_per_group", ctypes.c_int32),
                ("pipeline_depth", ctypes.c_int32), ("grid_waves", ctypes.c_int32),
                ("softmax_reduction", ctypes.c_int32)]

    def as_dict(self) -> dict:
        return {name: int(getattr(self, name)) for name, _ in self._fields_}


class Shape(ctypes.Structure):
    """Mirror of ``coopt_shape``."""
    _fields_ = [("num_seqs", ctypes.c_int32), ("num_q_heads", ctypes.c_int32),
                ("num_kv_heads", ctypes.c_int32), ("head_dim", ctypes.c_int32),
                ("block_size", ctypes.c_int32), ("num_blocks", ctypes.c_int32),
                ("max_blocks_per_seq", ctypes.c_int32), ("kv_dtype", ctypes.c_int32),
                ("softmax_scale", ctypes.c_float)]


def lib_path() -> str:
    return _LIB_PATH


def load_library():
    """Load libcoopt_attn.so (built by ``paper_2602_09323_amd.build``); raises if absent."""
    global _lib
    if _lib is None:
        path = os.environ.get("COOPT_ATTN_LIB", _LIB_PATH)   # another build of the same library
        if not os.path.exists(path):
            raise CooptError(f"{path} is not built; run `python -m paper_2602_09323_amd.build`")
        lib = ctypes.CDLL(path)
        vp, i32, sz = ctypes.c_void_p, ctypes.c_int32, ctypes.c_size_t
        shp, plp = ctypes.POINTER(Shape), ctypes.POINTER(DecodePlan)
        lib.coopt_kv_cache_write_fp8.argtypes = [vp, vp, vp, i32, vp, vp, vp, vp, shp, vp]
        lib.coopt_kv_cache_write_fp8_scaled.argtypes = [vp, vp, vp, i32, vp, vp, vp, vp, i32, vp, vp, shp, vp]
        lib.coopt_kv_cache_write_fp16.argtypes = [vp, vp, vp, i32, vp, vp, shp, vp]
        lib.coopt_kv_cache_write_skipset.argtypes = [vp, vp, vp, vp, i32, vp, vp, vp, vp, shp, vp]
        lib.coopt_paged_gqa_decode.argtypes = [vp, vp, vp, vp, vp, vp, vp, vp, vp, sz, plp, shp, vp]
        lib.coopt_paged_gqa_decode_step.argtypes = [vp, vp, vp, vp, vp, vp, vp, vp, vp, vp, vp, vp, sz,
                                                    plp, shp, vp]
        lib.coopt_paged_gqa_decode_split.argtypes = [vp, vp, vp, vp, vp, vp, vp, vp, sz, plp, shp, vp]
        lib.coopt_paged_gqa_decode_merge.argtypes = [vp, vp, sz, vp, plp, shp, vp]
        lib.coopt_decode_workspace_bytes.argtypes = [shp, plp]
        lib.coopt_decode_workspace_bytes.restype = sz
        lib.coopt_default_decode_plan.argtypes = [plp]
        lib.coopt_default_decode_plan.restype = None
        lib.coopt_paged_gqa_decode_partitioned.argtypes = [vp, vp, vp, vp, vp, vp, vp, i32, vp, vp, vp,
                                                           i32, plp, shp, vp]
        lib.coopt_paged_gqa_reduce.argtypes = [vp, vp, vp, vp, i32, i32, vp, shp, vp]
        lib.coopt_paged_gqa_prefill_chunk.argtypes = [vp, vp, vp, vp, vp, vp, vp, vp, i32, i32, vp, shp, vp]
        lib.coopt_paged_gqa_prefill_chunk_ws.argtypes = [vp, vp, vp, vp, vp, vp, vp, vp, i32, i32, vp, vp, sz,
                                                         shp, vp]
        lib.coopt_prefill_workspace_bytes.argtypes = [shp, i32]
        lib.coopt_prefill_workspace_bytes.restype = sz
        lib.coopt_gather_cached_kv.argtypes = [vp, vp, vp, vp, vp, i32, i32, i32, vp, vp, shp, vp]
        lib.coopt_decode_schedule_bytes.argtypes = [shp, plp]
        lib.coopt_decode_schedule_bytes.restype = sz
        lib.coopt_decode_schedule_prepare.argtypes = [vp, vp, vp, vp, sz, plp, shp, vp]
        lib.coopt_paged_gqa_decode_scheduled.argtypes = [vp, vp, vp, vp, vp, vp, vp, vp, vp, vp, vp, sz,
                                                         vp, sz, plp, shp, vp]
        lib.coopt_paged_gqa_decode_noalloc.argtypes = [vp, vp, vp, vp, vp, vp, vp, vp, plp, shp, vp]
        lib.coopt_decode_builtin_workspace_bytes.argtypes = []
        lib.coopt_decode_builtin_workspace_bytes.restype = sz
        lib.coopt_status_string.argtypes = [ctypes.c_int]
        lib.coopt_status_string.restype = ctypes.c_char_p
        for name in EXPORTS:
            if name not in ("coopt_decode_workspace_bytes", "coopt_decode_schedule_bytes",
                            "coopt_prefill_workspace_bytes",
                            "coopt_status_string", "coopt_default_decode_plan",
                            "coopt_decode_builtin_workspace_bytes"):
                getattr(lib, name).restype = ctypes.c_int
        _lib = lib
    return _lib


def status_string(status: int) -> str:
    return load_library().coopt_status_string(int(status)).decode()


def _check(status: int, what: str) -> None:
    if status != 0:
        raise CooptError(f"{what}: status {status} ({status_string(status)})")


def _call(name: str, *args) -> None:
    """Enter the library: every argument has been checked and marshalled by now."""
    _check(getattr(load_library(), name)(*args), name)


# ---------------------------------------------------------------- argument checks (host, no launch)

# A decode step of a short batch takes the GPU some 10 us, and its dozen tensors are checked on the
# way.  The entry points of a serving loop go through csrc/binding_native.cpp, which makes the same
# checks and enters the library in native code (a fused step of one short sequence 14.2 us before, 10.1
# so, of which the library's two launches are 7.4); whatever it does not take as it is -- anything
# wrong above all -- comes back here, where the checks below say what it is.

_native = None


def _fast():
    """The native entry points once the library is loaded, None until then or where they are not built for
    this torch."""
    global _native
    if _native is None and isinstance(_lib, ctypes.CDLL):
        _native = _bind_native() or False
    return _native or None


def _bind_native():
    import importlib.util
    import warnings
    if importlib.util.find_spec("._binding", __package__) is None:
        return None
    c = _th()._C
    device, raw = getattr(c, "_cuda_getDevice", None), getattr(c, "_cuda_getCurrentRawStream", None)
    if device is None or raw is None:
        return None
    # (it reads torch's tensors by the layout of the headers that it was compiled with)
    try:
        _binding = importlib.import_module("._binding", __package__)
        why = f"it was built for torch {_binding.built_for}" if _binding.built_for != _torch.__version__ else None
    except (ImportError, AttributeError) as e:
        why = str(e)
    if why is not None:
        warnings.warn(f"the binding's native part is left out ({why}, this is torch {_torch.__version__}): every call goes "
                      "through ctypes; run `python -m paper_2602_09323_amd.build`", RuntimeWarning, stacklevel=4)
        return None
    names = ("kv_cache_write_fp8", "kv_cache_write_fp16", "paged_gqa_decode", "paged_gqa_decode_step",
             "decode_schedule_prepare", "paged_gqa_decode_scheduled", "paged_gqa_decode_partitioned",
             "paged_gqa_reduce", "paged_gqa_prefill_chunk_ws", "gather_cached_kv", "decode_workspace_bytes",
             "decode_schedule_bytes", "prefill_workspace_bytes")
    _binding.bind(tuple(ctypes.cast(getattr(_lib, "coopt_" + n), ctypes.c_void_p).value for n in names),
                  Shape, DecodePlan, device, raw)
    return _binding


def _entered(status: Optional[int], name: str) -> bool:
    """Whether a native entry point took the call (None: it did not); raises if the library refused."""
    if status:
        _check(status, name)
    return status is not None

def _nbytes(t) -> int:
    return t.numel() * t.element_size()


def _refuse(t, name: str, what: Optional[str], min_bytes: int, elem: Optional[int], dtype) -> None:
    """Raises what is wrong with an argument that ``_dev`` did not accept."""
    if what is not None:
        name = f"{what}: {name}"
    if t is None:
        raise CooptError(f"{name}: required tensor is None")
    if not getattr(t, "is_cuda", False):
        raise CooptError(f"{name}: not a device tensor")
    if not t.is_contiguous():
        raise CooptError(f"{name}: not contiguous")
    if dtype is not None and t.dtype != dtype:
        raise CooptError(f"{name}: dtype {t.dtype}, expected {dtype}")
    if elem is not None and t.element_size() != elem:
        raise CooptError(f"{name}: {t.element_size()}-byte elements, expected {elem}")
    raise CooptError(f"{name}: {_nbytes(t)} bytes, the shape needs {min_bytes}")


def _dev(t, name: str, what: Optional[str] = None, min_bytes: int = 0, elem: Optional[int] = None,
         dtype=None, optional: bool = False):
    """Pointer (an integer) of a contiguous device tensor of at least ``min_bytes`` bytes, with
    ``elem``-byte elements or exactly ``dtype`` where given.  None passes as NULL only if ``optional``.
    ``what`` and ``name`` name the entry point and the argument in what is raised."""
    if t is None and optional:
        return None
    if getattr(t, "is_cuda", False) and t.is_contiguous() and (dtype is None or t.dtype == dtype):
        size = t.element_size()
        if (elem is None or size == elem) and t.numel() * size >= min_bytes:
            return t.data_ptr()
    _refuse(t, name, what, min_bytes, elem, dtype)


def _sizes(shape: Shape):
    hk, d, S = shape.num_kv_heads, shape.head_dim, shape.num_seqs
    scaled = shape.kv_dtype != COOPT_KV_FP16
    slots = shape.num_blocks * hk * shape.block_size
    return {"cache": slots * d * (1 if scaled else 2),
            "scale": slots * 4,
            "q": S * shape.num_q_heads * d * 2,
            "tables": S * shape.max_blocks_per_seq * 4,
            "lens": S * 4,
            "row": hk * d * 2,
            "scaled": scaled}


def _cache_ptrs(k_cache, v_cache, k_scale, v_scale, z):
    unscaled = not z["scaled"]
    cache, scale = z["cache"], z["scale"]
    return (_dev(k_cache, "k_cache", None, cache), _dev(v_cache, "v_cache", None, cache),
            _dev(k_scale, "k_scale", None, scale, optional=unscaled),
            _dev(v_scale, "v_scale", None, scale, optional=unscaled))


_torch = None


def _th():
    """torch, imported at the first call (importing this module does not need it)."""
    global _torch
    if _torch is None:
        import torch
        _torch = torch
    return _torch


def _i32():
    return _th().int32


def _i64():
    return _th().int64


def _plan_ptr(plan: Optional[DecodePlan]):
    return None if plan is None else ctypes.byref(plan)


def _stream(stream=None):
    """The stream's handle (an integer): the given one's, or that of torch's current stream.  The
    handle alone is asked of torch where it offers that (0.3 us; building its Stream object: 2.7 us)."""
    if stream is not None:
        return stream.cuda_stream
    cuda = _th().cuda
    raw = getattr(_torch._C, "_cuda_getCurrentRawStream", None)
    return cuda.current_stream().cuda_stream if raw is None else raw(cuda.current_device())


def _new_rows(k, v, slot_mapping, z, what: str):
    """Pointers of new K/V rows [T][H_k][d] fp16 and their int64 slots; returns (pk, pv, ps, T)."""
    ps = _dev(slot_mapping, "slot_mapping", what, dtype=_i64())
    T = slot_mapping.numel()
    need = T * z["row"]
    return _dev(k, "k", what, need, 2), _dev(v, "v", what, need, 2), ps, T


# ---------------------------------------------------------------- plan

def default_decode_plan() -> DecodePlan:
    """The plan a call runs under when it is given none (``coopt_default_decode_plan``)."""
    p = DecodePlan()
    load_library().coopt_default_decode_plan(ctypes.byref(p))
    return p


def make_decode_plan(**fields) -> DecodePlan:
    """The default plan with the named fields of ``coopt_decode_plan`` replaced."""
    p = default_decode_plan()
    for k, val in fields.items():
        if k not in dict(DecodePlan._fields_):
            raise KeyError(k)
        setattr(p, k, int(val))
    return p


# ---------------------------------------------------------------- cache write

def kv_cache_write_fp8(k, v, slot_mapping, k_cache, v_cache, k_scale, v_scale, shape: Shape,
                       stream=None) -> None:
    fast = _fast()
    if fast is not None and _entered(fast.write_fp8(k, v, slot_mapping, k_cache, v_cache, k_scale, v_scale, shape, stream), "coopt_kv_cache_write_fp8"):
        return
    z = _sizes(shape)
    pk, pv, ps, T = _new_rows(k, v, slot_mapping, z, "kv_cache_write_fp8")
    _call("coopt_kv_cache_write_fp8",
          pk, pv, ps, T, *_cache_ptrs(k_cache, v_cache, k_scale, v_scale, z), ctypes.byref(shape),
        _stream(stream))


def kv_cache_write_fp8_scaled(k, v, slot_mapping, k_cache, v_cache, k_scale, v_scale, shape: Shape,
                              scale_mode: int, k_static=None, v_static=None, stream=None) -> None:
    """The write under another scale rule (COOPT_SCALE_*); k_static / v_static: device float32
    [H_k], required for COOPT_SCALE_STATIC only."""
    z = _sizes(shape)
    pk, pv, ps, T = _new_rows(k, v, slot_mapping, z, "kv_cache_write_fp8_scaled")
    static = int(scale_mode) == COOPT_SCALE_STATIC
    hk = shape.num_kv_heads * 4
    _call("coopt_kv_cache_write_fp8_scaled",
          pk, pv, ps, T, *_cache_ptrs(k_cache, v_cache, k_scale, v_scale, z), int(scale_mode),
          _dev(k_static, "k_static", elem=4, min_bytes=hk, optional=not static),
          _dev(v_static, "v_static", elem=4, min_bytes=hk, optional=not static),
          ctypes.byref(shape), _stream(stream))


def kv_cache_write_skipset(k, v, slot_mapping, skip_set, k_cache, v_cache, k_scale, v_scale,
                           shape: Shape, stream=None) -> None:
    """skip_set: device uint32 bitmap over the call's token indices, or None."""
    z = _sizes(shape)
    pk, pv, ps, T = _new_rows(k, v, slot_mapping, z, "kv_cache_write_skipset")
    pset = _dev(skip_set, "skip_set", min_bytes=(T + 31) // 32 * 4, elem=4, optional=True)
    _call("coopt_kv_cache_write_skipset",
          pk, pv, ps, pset, T, *_cache_ptrs(k_cache, v_cache, k_scale, v_scale, z),
        ctypes.byref(shape), _stream(stream))


def kv_cache_write_fp16(k, v, slot_mapping, k_cache, v_cache, shape: Shape, stream=None) -> None:
    fast = _fast()
    if fast is not None and _entered(fast.write_fp16(k, v, slot_mapping, k_cache, v_cache, shape, stream), "coopt_kv_cache_write_fp16"):
        return
    z = _sizes(shape)
    pk, pv, ps, T = _new_rows(k, v, slot_mapping, z, "kv_cache_write_fp16")
    pkc, pvc, _, _ = _cache_ptrs(k_cache, v_cache, None, None, z)
    _call("coopt_kv_cache_write_fp16",
          pk, pv, ps, T, pkc, pvc, ctypes.byref(shape), _stream(stream))


# ---------------------------------------------------------------- decode

def decode_workspace_bytes(shape: Shape, plan: Optional[DecodePlan] = None) -> int:
    return int(load_library().coopt_decode_workspace_bytes(ctypes.byref(shape), _plan_ptr(plan)))


def _decode_inputs(q, k_cache, v_cache, k_scale, v_scale, block_tables, context_lens, z, what: str):
    return (_dev(q, "q", what, elem=2, min_bytes=z["q"]),
            *_cache_ptrs(k_cache, v_cache, k_scale, v_scale, z),
            _dev(block_tables, "block_tables", what, dtype=_i32(), min_bytes=z["tables"]),
            _dev(context_lens, "context_lens", what, dtype=_i32(), min_bytes=z["lens"]))


def _workspace(workspace, shape: Shape, plan, what: str, optional: bool = False):
    if workspace is None and optional:
        return None, 0
    need = decode_workspace_bytes(shape, plan)
    return _dev(workspace, "workspace", what, need), _nbytes(workspace)


def paged_gqa_decode(q, k_cache, v_cache, k_scale, v_scale, block_tables, context_lens, out,
                     workspace, shape: Shape, plan: Optional[DecodePlan] = None, stream=None) -> None:
    fast = _fast()
    if fast is not None and _entered(fast.decode(q, k_cache, v_cache, k_scale, v_scale, block_tables, context_lens, out, workspace, shape, plan, stream), "coopt_paged_gqa_decode"):
        return
    what = "paged_gqa_decode"
    z = _sizes(shape)
    ins = _decode_inputs(q, k_cache, v_cache, k_scale, v_scale, block_tables, context_lens, z, what)
    pws, nws = _workspace(workspace, shape, plan, what, optional=True)
    _call("coopt_paged_gqa_decode",
          *ins, _dev(out, "out", what, elem=2, min_bytes=z["q"]), pws, nws,
        _plan_ptr(plan), ctypes.byref(shape), _stream(stream))


def decode_builtin_workspace_bytes() -> int:
    return int(load_library().coopt_decode_builtin_workspace_bytes())


def paged_gqa_decode_noalloc(q, k_cache, v_cache, k_scale, v_scale, block_tables, context_lens, out,
                             shape: Shape, plan: Optional[DecodePlan] = None, stream=None) -> None:
    """``paged_gqa_decode`` through the library's built-in workspace (no allocation anywhere)."""
    what = "paged_gqa_decode_noalloc"
    z = _sizes(shape)
    ins = _decode_inputs(q, k_cache, v_cache, k_scale, v_scale, block_tables, context_lens, z, what)
    _call("coopt_paged_gqa_decode_noalloc",
          *ins, _dev(out, "out", what, elem=2, min_bytes=z["q"]), _plan_ptr(plan),
          ctypes.byref(shape), _stream(stream))


def paged_gqa_decode_step(k, v, slot_mapping, q, k_cache, v_cache, k_scale, v_scale, block_tables,
                          context_lens, out, workspace, shape: Shape,
                          plan: Optional[DecodePlan] = None, stream=None) -> None:
    fast = _fast()
    if fast is not None and _entered(fast.step(k, v, slot_mapping, q, k_cache, v_cache, k_scale, v_scale, block_tables, context_lens, out, workspace,
                                              shape, plan, stream), "coopt_paged_gqa_decode_step"):
        return
    what = "paged_gqa_decode_step"
    z = _sizes(shape)
    pk, pv, ps, T = _new_rows(k, v, slot_mapping, z, what)
    if T < shape.num_seqs:
        raise CooptError(f"{what}: slot_mapping has {T} entries, the batch {shape.num_seqs} sequences")
    ins = _decode_inputs(q, k_cache, v_cache, k_scale, v_scale, block_tables, context_lens, z, what)
    pws, nws = _workspace(workspace, shape, plan, what)
    _call("coopt_paged_gqa_decode_step",
          pk, pv, ps, *ins, _dev(out, "out", what, elem=2, min_bytes=z["q"]), pws, nws,
        _plan_ptr(plan), ctypes.byref(shape), _stream(stream))


def paged_gqa_decode_split(q, k_cache, v_cache, k_scale, v_scale, block_tables, context_lens,
                           workspace, shape: Shape, plan: Optional[DecodePlan] = None,
                           stream=None) -> None:
    what = "paged_gqa_decode_split"
    z = _sizes(shape)
    ins = _decode_inputs(q, k_cache, v_cache, k_scale, v_scale, block_tables, context_lens, z, what)
    pws, nws = _workspace(workspace, shape, plan, what)
    _call("coopt_paged_gqa_decode_split",
          *ins, pws, nws, _plan_ptr(plan), ctypes.byref(shape), _stream(stream))


def paged_gqa_decode_merge(context_lens, workspace, out, shape: Shape,
                           plan: Optional[DecodePlan] = None, stream=None) -> None:
    what = "paged_gqa_decode_merge"
    z = _sizes(shape)
    pws, nws = _workspace(workspace, shape, plan, what)
    _call("coopt_paged_gqa_decode_merge",
          _dev(context_lens, "context_lens", what, dtype=_i32(), min_bytes=z["lens"]), pws, nws,
        _dev(out, "out", what, elem=2, min_bytes=z["q"]), _plan_ptr(plan), ctypes.byref(shape),
        _stream(stream))


def _partial_buffers(tmp_out, max_logits, exp_sums, max_parts: int, shape: Shape, what: str):
    rows = shape.num_seqs * shape.num_q_heads * int(max_parts)
    return (_dev(tmp_out, "tmp_out", what, elem=4, min_bytes=rows * shape.head_dim * 4),
            _dev(max_logits, "max_logits", what, elem=4, min_bytes=rows * 4),
            _dev(exp_sums, "exp_sums", what, elem=4, min_bytes=rows * 4))


def paged_gqa_decode_partitioned(q, k_cache, v_cache, k_scale, v_scale, block_tables,
                                 context_lens, partition_size: int, tmp_out, max_logits, exp_sums,
                                 max_parts: int, shape: Shape, plan: Optional[DecodePlan] = None,
                                 stream=None) -> None:
    fast = _fast()
    if fast is not None and _entered(fast.partitioned(q, k_cache, v_cache, k_scale, v_scale, block_tables, context_lens, partition_size,
                                                     tmp_out, max_logits, exp_sums, max_parts, shape, plan, stream), "coopt_paged_gqa_decode_partitioned"):
        return
    what = "paged_gqa_decode_partitioned"
    z = _sizes(shape)
    ins = _decode_inputs(q, k_cache, v_cache, k_scale, v_scale, block_tables, context_lens, z, what)
    _call("coopt_paged_gqa_decode_partitioned",
          *ins, int(partition_size), *_partial_buffers(tmp_out, max_logits, exp_sums, max_parts, shape, what),
        int(max_parts), _plan_ptr(plan), ctypes.byref(shape), _stream(stream))


def paged_gqa_reduce(tmp_out, max_logits, exp_sums, context_lens, partition_size: int,
                     max_parts: int, out, shape: Shape, stream=None) -> None:
    fast = _fast()
    if fast is not None and _entered(fast.reduce(tmp_out, max_logits, exp_sums, context_lens, partition_size, max_parts, out,
                                                shape, stream), "coopt_paged_gqa_reduce"):
        return
    what = "paged_gqa_reduce"
    z = _sizes(shape)
    _call("coopt_paged_gqa_reduce",
          *_partial_buffers(tmp_out, max_logits, exp_sums, max_parts, shape, what),
        _dev(context_lens, "context_lens", what, dtype=_i32(), min_bytes=z["lens"]),
        int(partition_size), int(max_parts), _dev(out, "out", what, elem=2, min_bytes=z["q"]),
        ctypes.byref(shape), _stream(stream))


def paged_gqa_prefill_chunk(q, k_cache, v_cache, k_scale, v_scale, block_tables, context_lens,
                            query_start, num_query_rows: int, max_chunk_len: int, out,
                            shape: Shape, stream=None) -> None:
    what = "paged_gqa_prefill_chunk"
    z = _sizes(shape)
    rows_bytes = int(num_query_rows) * shape.num_q_heads * shape.head_dim * 2
    _call("coopt_paged_gqa_prefill_chunk",
          _dev(q, "q", what, elem=2, min_bytes=rows_bytes),
        *_cache_ptrs(k_cache, v_cache, k_scale, v_scale, z),
        _dev(block_tables, "block_tables", what, dtype=_i32(), min_bytes=z["tables"]),
        _dev(context_lens, "context_lens", what, dtype=_i32(), min_bytes=z["lens"]),
        _dev(query_start, "query_start", what, dtype=_i32(), min_bytes=z["lens"] + 4),
        int(num_query_rows), int(max_chunk_len),
        _dev(out, "out", what, elem=2, min_bytes=rows_bytes), ctypes.byref(shape), _stream(stream))


def prefill_workspace_bytes(shape: Shape, max_chunk_len: int) -> int:
    return int(load_library().coopt_prefill_workspace_bytes(ctypes.byref(shape), int(max_chunk_len)))


def paged_gqa_prefill_chunk_ws(q, k_cache, v_cache, k_scale, v_scale, block_tables, context_lens,
                               query_start, num_query_rows: int, max_chunk_len: int, out, workspace,
                               shape: Shape, stream=None) -> None:
    """workspace: a device buffer of at least prefill_workspace_bytes(shape, max_chunk_len) bytes
    (None where that is 0)."""
    fast = _fast()
    if fast is not None and _entered(fast.prefill_ws(q, k_cache, v_cache, k_scale, v_scale, block_tables, context_lens, query_start,
                                                    num_query_rows, max_chunk_len, out, workspace, shape, stream), "coopt_paged_gqa_prefill_chunk_ws"):
        return
    what = "paged_gqa_prefill_chunk_ws"
    z = _sizes(shape)
    rows_bytes = int(num_query_rows) * shape.num_q_heads * shape.head_dim * 2
    need = prefill_workspace_bytes(shape, max_chunk_len)
    pws, nws = (None, 0) if workspace is None else (
        _dev(workspace, "workspace", what, need), _nbytes(workspace))
    _call("coopt_paged_gqa_prefill_chunk_ws",
          _dev(q, "q", what, elem=2, min_bytes=rows_bytes),
          *_cache_ptrs(k_cache, v_cache, k_scale, v_scale, z),
          _dev(block_tables, "block_tables", what, dtype=_i32(), min_bytes=z["tables"]),
          _dev(context_lens, "context_lens", what, dtype=_i32(), min_bytes=z["lens"]),
          _dev(query_start, "query_start", what, dtype=_i32(), min_bytes=z["lens"] + 4),
          int(num_query_rows), int(max_chunk_len),
          _dev(out, "out", what, elem=2, min_bytes=rows_bytes), pws, nws, ctypes.byref(shape),
          _stream(stream))


def decode_schedule_bytes(shape: Shape, plan: Optional[DecodePlan] = None) -> int:
    return int(load_library().coopt_decode_schedule_bytes(ctypes.byref(shape), _plan_ptr(plan)))


def decode_schedule_prepare(block_tables, context_lens, slot_mapping, schedule, shape: Shape,
                            plan: Optional[DecodePlan] = None, stream=None) -> None:
    """Write the decode schedule (``slot_mapping`` None: plain decode; else the fused step)."""
    fast = _fast()
    if fast is not None and _entered(fast.prepare(block_tables, context_lens, slot_mapping, schedule, shape, plan, stream), "coopt_decode_schedule_prepare"):
        return
    what = "decode_schedule_prepare"
    z = _sizes(shape)
    _call("coopt_decode_schedule_prepare",
          _dev(block_tables, "block_tables", what, dtype=_i32(), min_bytes=z["tables"]),
        _dev(context_lens, "context_lens", what, dtype=_i32(), min_bytes=z["lens"]),
        _dev(slot_mapping, "slot_mapping", what, dtype=_i64(), min_bytes=2 * z["lens"], optional=True),
        _dev(schedule, "schedule", what, min_bytes=decode_schedule_bytes(shape, plan)),
        _nbytes(schedule), _plan_ptr(plan), ctypes.byref(shape), _stream(stream))


def paged_gqa_decode_scheduled(k, v, slot_mapping, q, k_cache, v_cache, k_scale, v_scale, context_lens,
                               out, workspace, schedule, shape: Shape,
                               plan: Optional[DecodePlan] = None, stream=None) -> None:
    """Decode (k, v, slot_mapping None) or fused step from a prepared schedule; ``out`` None stops
    after the partial results."""
    fast = _fast()
    if fast is not None and _entered(fast.scheduled(k, v, slot_mapping, q, k_cache, v_cache, k_scale, v_scale, context_lens, out,
                                                   workspace, schedule, shape, plan, stream), "coopt_paged_gqa_decode_scheduled"):
        return
    what = "paged_gqa_decode_scheduled"
    z = _sizes(shape)
    if k is None and v is None and slot_mapping is None:
        pk = pv = ps = None
    else:
        pk, pv, ps, T = _new_rows(k, v, slot_mapping, z, what)
        if T < shape.num_seqs:
            raise CooptError(f"{what}: slot_mapping has {T} entries, the batch {shape.num_seqs} sequences")
    pws, nws = _workspace(workspace, shape, plan, what)
    _call("coopt_paged_gqa_decode_scheduled",
          pk, pv, ps, _dev(q, "q", what, elem=2, min_bytes=z["q"]),
        *_cache_ptrs(k_cache, v_cache, k_scale, v_scale, z),
        _dev(context_lens, "context_lens", what, dtype=_i32(), min_bytes=z["lens"]),
        _dev(out, "out", what, elem=2, min_bytes=z["q"], optional=True), pws, nws,
        _dev(schedule, "schedule", what, min_bytes=decode_schedule_bytes(shape, plan)),
        _nbytes(schedule), _plan_ptr(plan), ctypes.byref(shape), _stream(stream))


def gather_cached_kv(k_cache, v_cache, k_scale, v_scale, block_tables, seq: int, tok_begin: int,
                     tok_end: int, k_out, v_out, shape: Shape, stream=None) -> None:
    fast = _fast()
    if fast is not None and _entered(fast.gather(k_cache, v_cache, k_scale, v_scale, block_tables, seq, tok_begin, tok_end, k_out, v_out, shape,
                                                stream), "coopt_gather_cached_kv"):
        return
    what = "gather_cached_kv"
    z = _sizes(shape)
    rows = max(int(tok_end) - int(tok_begin), 0) * z["row"]
    _call("coopt_gather_cached_kv",
          *_cache_ptrs(k_cache, v_cache, k_scale, v_scale, z),
        _dev(block_tables, "block_tables", what, dtype=_i32(), min_bytes=z["tables"]), int(seq),
        int(tok_begin), int(tok_end), _dev(k_out, "k_out", what, elem=2, min_bytes=rows),
        _dev(v_out, "v_out", what, elem=2, min_bytes=rows), ctypes.byref(shape),
        _stream(stream))
