// The argument checks and marshalling of binding.py's hot entry points in native code.  A decode step's
// dozen tensors cost ctypes and Python 13 us a call, as much as the GPU takes for a short batch; here
// a call costs what its launches cost.
//
// Every function takes the arguments of the Python function of the same purpose, in its order, plan and
// stream included, and returns the library's status -- or None, having done nothing, for anything but
// the plain case: a tensor that is none, on the host, strided, too small or of another type, an object
// of another class, an exception on the way.  binding.py then takes its own path, which says what is
// wrong or handles it.  Nothing is kept between calls but the addresses that bind() was given.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/PythonTorchFunctionTLS.h>
#include <torch/csrc/autograd/python_variable.h>

#include "coopt_attn.h"

namespace {

typedef __int128 wide;          // sizes as Python computes them: no product of shape fields overflows

// What bind() was given: the library's functions, the classes of shapes and plans, and how torch is
// asked for the current stream.
struct {
    decltype(&coopt_kv_cache_write_fp8) write_fp8;
    decltype(&coopt_kv_cache_write_fp16) write_fp16;
    decltype(&coopt_paged_gqa_decode) decode;
    decltype(&coopt_paged_gqa_decode_step) step;
    decltype(&coopt_decode_schedule_prepare) prepare;
    decltype(&coopt_paged_gqa_decode_scheduled) scheduled;
    decltype(&coopt_paged_gqa_decode_partitioned) partitioned;
    decltype(&coopt_paged_gqa_reduce) reduce;
    decltype(&coopt_paged_gqa_prefill_chunk_ws) prefill_ws;
    decltype(&coopt_gather_cached_kv) gather;
    decltype(&coopt_decode_workspace_bytes) workspace_bytes;
    decltype(&coopt_decode_schedule_bytes) schedule_bytes;
    decltype(&coopt_prefill_workspace_bytes) prefill_bytes;
    PyObject *shape_class, *plan_class, *current_device, *raw_stream;
} lib = {};

// The call is not the plain case: back to Python.
struct Decline {};

// A ctypes structure's fields (the object outlives the call that holds it as an argument).
template <class T>
T fields_of(PyObject* o, PyObject* cls)
{
    if ((PyObject*)Py_TYPE(o) != cls) throw Decline();
    Py_buffer b;
    if (PyObject_GetBuffer(o, &b, PyBUF_SIMPLE) != 0) throw Decline();
    T out;
    const bool fits = b.len == (Py_ssize_t)sizeof(T);
    if (fits) memcpy(&out, b.buf, sizeof(T));
    PyBuffer_Release(&b);
    if (!fits) throw Decline();
    return out;
}

struct Plan {
    coopt_decode_plan fields;
    bool given;
    explicit Plan(PyObject* o) : given(o != Py_None)
    {
        if (given) fields = fields_of<coopt_decode_plan>(o, lib.plan_class);
    }
    const coopt_decode_plan* ptr() const { return given ? &fields : nullptr; }
};

struct Shape : coopt_shape {
    bool scaled;
    wide cache, scale, q, tables, lens, row;
    explicit Shape(PyObject* o) : coopt_shape(fields_of<coopt_shape>(o, lib.shape_class))
    {
        scaled = kv_dtype != COOPT_KV_FP16;
        const wide slots = (wide)num_blocks * num_kv_heads * block_size;
        cache = slots * head_dim * (scaled ? 1 : 2);
        scale = slots * 4;
        q = (wide)num_seqs * num_q_heads * head_dim * 2;
        tables = (wide)num_seqs * max_blocks_per_seq * 4;
        lens = (wide)num_seqs * 4;
        row = (wide)num_kv_heads * head_dim * 2;
    }
};

// Pointer of a contiguous device tensor of at least `bytes` bytes; elem: bytes of an element (0: any).
struct Tensor {
    void* at = nullptr;
    int64_t numel = 0, bytes = 0;
    Tensor(PyObject* o, wide need, int elem) { read(o, need, elem, nullptr); }
    Tensor(PyObject* o, wide need, c10::ScalarType type) { read(o, need, 0, &type); }
    void read(PyObject* o, wide need, int elem, const c10::ScalarType* type)
    {
        if (!THPVariable_CheckExact(o)) throw Decline();
        const at::Tensor& t = THPVariable_Unpack(o);
        if (!t.is_cuda() || !t.is_contiguous() || (type && t.scalar_type() != *type)) throw Decline();
        const int64_t size = (int64_t)t.element_size();
        numel = t.numel();
        bytes = numel * size;
        if ((elem && size != elem) || bytes < need) throw Decline();
        at = t.data_ptr();
    }
    template <class T>
    T* as() const { return (T*)at; }
};
// ... or NULL for None.
void* optional(PyObject* o, wide need, int elem) { return o == Py_None ? nullptr : Tensor(o, need, elem).at; }

struct Cache {
    void *k, *v;
    float *ks, *vs;
    Cache(PyObject* const* a, const Shape& sh) : k(Tensor(a[0], sh.cache, 0).at), v(Tensor(a[1], sh.cache, 0).at)
    {
        ks = (float*)(sh.scaled ? Tensor(a[2], sh.scale, 0).at : optional(a[2], sh.scale, 0));
        vs = (float*)(sh.scaled ? Tensor(a[3], sh.scale, 0).at : optional(a[3], sh.scale, 0));
    }
};

struct NewRows {
    Tensor slots;
    void *k, *v;
    NewRows(PyObject* const* a, const Shape& sh)      // k, v, slot_mapping
        : slots(a[2], 0, c10::kLong), k(Tensor(a[0], slots.numel * sh.row, 2).at), v(Tensor(a[1], slots.numel * sh.row, 2).at)
    {
        if (slots.numel > INT32_MAX) throw Decline();
    }
};

int32_t small_int(PyObject* o)
{
    if (!PyLong_CheckExact(o)) throw Decline();
    const long x = PyLong_AsLong(o);
    if (x == -1 && PyErr_Occurred()) throw Decline();
    if (x < INT32_MIN || x > INT32_MAX) throw Decline();
    return (int32_t)x;
}

// The given stream's handle, or that of torch's current stream.
void* stream_of(PyObject* o)
{
    PyObject* handle;
    if (o != Py_None) {
        handle = PyObject_GetAttrString(o, "cuda_stream");
    } else {
        PyObject* device = PyObject_CallNoArgs(lib.current_device);
        if (!device) throw Decline();
        handle = PyObject_CallOneArg(lib.raw_stream, device);
        Py_DECREF(device);
    }
    if (!handle) throw Decline();
    void* s = PyLong_AsVoidPtr(handle);
    Py_DECREF(handle);
    if (PyErr_Occurred()) throw Decline();
    return s;
}

// Runs `call` over N arguments: its status, or None where it declines.  No exception leaves.
template <int N, class F>
PyObject* guarded(Py_ssize_t n, F call)
{
    try {
        // (a torch function mode sees the questions that binding.py asks of the tensors)
        if (n == N && lib.step && !at::impl::torch_function_mode_enabled()) return PyLong_FromLong(call());
    } catch (...) {
        PyErr_Clear();
    }
    Py_RETURN_NONE;
}

// The library is entered without the interpreter lock, as ctypes does.
template <class F>
int unlocked(F enter)
{
    int status;
    Py_BEGIN_ALLOW_THREADS
    status = enter();
    Py_END_ALLOW_THREADS
    return status;
}

PyObject* write_fp8(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    return guarded<9>(n, [&] {
        const Shape sh(a[7]);
        const NewRows r(a, sh);
        const Cache c(a + 3, sh);
        void* s = stream_of(a[8]);
        return unlocked([&] {
            return lib.write_fp8(r.k, r.v, r.slots.as<int64_t>(), (int32_t)r.slots.numel, (uint8_t*)c.k, (uint8_t*)c.v, c.ks, c.vs, &sh, s);
        });
    });
}

PyObject* write_fp16(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    return guarded<7>(n, [&] {
        const Shape sh(a[5]);
        if (sh.scaled) throw Decline();
        const NewRows r(a, sh);
        const Tensor k(a[3], sh.cache, 0), v(a[4], sh.cache, 0);
        void* s = stream_of(a[6]);
        return unlocked([&] {
            return lib.write_fp16(r.k, r.v, r.slots.as<int64_t>(), (int32_t)r.slots.numel, k.at, v.at, &sh, s);
        });
    });
}

// q, cache, block tables and lengths, in this order
struct Inputs {
    Tensor q;
    Cache c;
    Tensor tables, lens;
    Inputs(PyObject* const* a, const Shape& sh)
        : q(a[0], sh.q, 2), c(a + 1, sh), tables(a[5], sh.tables, c10::kInt), lens(a[6], sh.lens, c10::kInt) {}
};

PyObject* decode(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    return guarded<12>(n, [&] {
        const Shape sh(a[9]);
        const Plan p(a[10]);
        const Inputs in(a, sh);
        const Tensor out(a[7], sh.q, 2);
        void* ws = nullptr;
        size_t ws_bytes = 0;
        if (a[8] != Py_None) {
            const Tensor w(a[8], (wide)lib.workspace_bytes(&sh, p.ptr()), 0);
            ws = w.at;
            ws_bytes = (size_t)w.bytes;
        }
        void* s = stream_of(a[11]);
        return unlocked([&] {
            return lib.decode(in.q.at, in.c.k, in.c.v, in.c.ks, in.c.vs, in.tables.as<int32_t>(), in.lens.as<int32_t>(),
                              out.at, ws, ws_bytes, p.ptr(), &sh, s);
        });
    });
}

PyObject* step(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    return guarded<15>(n, [&] {
        const Shape sh(a[12]);
        const Plan p(a[13]);
        const NewRows r(a, sh);
        if (r.slots.numel < sh.num_seqs) throw Decline();
        const Inputs in(a + 3, sh);
        const Tensor out(a[10], sh.q, 2), ws(a[11], (wide)lib.workspace_bytes(&sh, p.ptr()), 0);
        void* s = stream_of(a[14]);
        return unlocked([&] {
            return lib.step(r.k, r.v, r.slots.as<int64_t>(), in.q.at, in.c.k, in.c.v, in.c.ks, in.c.vs,
                            in.tables.as<int32_t>(), in.lens.as<int32_t>(), out.at, ws.at, (size_t)ws.bytes, p.ptr(), &sh, s);
        });
    });
}

PyObject* prepare(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    return guarded<7>(n, [&] {
        const Shape sh(a[4]);
        const Plan p(a[5]);
        const Tensor tables(a[0], sh.tables, c10::kInt), lens(a[1], sh.lens, c10::kInt);
        int64_t* slots = a[2] == Py_None ? nullptr : Tensor(a[2], 2 * sh.lens, c10::kLong).as<int64_t>();
        const Tensor sched(a[3], (wide)lib.schedule_bytes(&sh, p.ptr()), 0);
        void* s = stream_of(a[6]);
        return unlocked([&] {
            return lib.prepare(tables.as<int32_t>(), lens.as<int32_t>(), slots, sched.at, (size_t)sched.bytes, p.ptr(), &sh, s);
        });
    });
}

PyObject* scheduled(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    return guarded<15>(n, [&] {
        const Shape sh(a[12]);
        const Plan p(a[13]);
        void *k = nullptr, *v = nullptr;
        int64_t* slots = nullptr;
        if (a[0] != Py_None || a[1] != Py_None || a[2] != Py_None) {
            const NewRows r(a, sh);
            if (r.slots.numel < sh.num_seqs) throw Decline();
            k = r.k;
            v = r.v;
            slots = r.slots.as<int64_t>();
        }
        const Tensor q(a[3], sh.q, 2);
        const Cache c(a + 4, sh);
        const Tensor lens(a[8], sh.lens, c10::kInt);
        void* out = optional(a[9], sh.q, 2);
        const Tensor ws(a[10], (wide)lib.workspace_bytes(&sh, p.ptr()), 0);
        const Tensor sched(a[11], (wide)lib.schedule_bytes(&sh, p.ptr()), 0);
        void* s = stream_of(a[14]);
        return unlocked([&] {
            return lib.scheduled(k, v, slots, q.at, c.k, c.v, c.ks, c.vs, lens.as<int32_t>(), out, ws.at,
                                 (size_t)ws.bytes, sched.at, (size_t)sched.bytes, p.ptr(), &sh, s);
        });
    });
}

struct Partials {
    Tensor tmp, max, sum;
    Partials(PyObject* const* a, int32_t parts, const Shape& sh)
        : tmp(a[0], rows(parts, sh) * sh.head_dim * 4, 4), max(a[1], rows(parts, sh) * 4, 4), sum(a[2], rows(parts, sh) * 4, 4) {}
    static wide rows(int32_t parts, const Shape& sh) { return (wide)sh.num_seqs * sh.num_q_heads * parts; }
};

PyObject* partitioned(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    return guarded<15>(n, [&] {
        const Shape sh(a[12]);
        const Plan p(a[13]);
        const Inputs in(a, sh);
        const int32_t size = small_int(a[7]), parts = small_int(a[11]);
        const Partials t(a + 8, parts, sh);
        void* s = stream_of(a[14]);
        return unlocked([&] {
            return lib.partitioned(in.q.at, in.c.k, in.c.v, in.c.ks, in.c.vs, in.tables.as<int32_t>(), in.lens.as<int32_t>(),
                                   size, t.tmp.as<float>(), t.max.as<float>(), t.sum.as<float>(), parts, p.ptr(), &sh, s);
        });
    });
}

PyObject* reduce(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    return guarded<9>(n, [&] {
        const Shape sh(a[7]);
        const int32_t size = small_int(a[4]), parts = small_int(a[5]);
        const Partials t(a, parts, sh);
        const Tensor lens(a[3], sh.lens, c10::kInt), out(a[6], sh.q, 2);
        void* s = stream_of(a[8]);
        return unlocked([&] {
            return lib.reduce(t.tmp.as<float>(), t.max.as<float>(), t.sum.as<float>(), lens.as<int32_t>(), size, parts, out.at, &sh, s);
        });
    });
}

PyObject* prefill_ws(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    return guarded<14>(n, [&] {
        const Shape sh(a[12]);
        const int32_t rows = small_int(a[8]), longest = small_int(a[9]);
        const wide rows_bytes = (wide)rows * sh.num_q_heads * sh.head_dim * 2;
        const Tensor q(a[0], rows_bytes, 2);
        const Cache c(a + 1, sh);
        const Tensor tables(a[5], sh.tables, c10::kInt), lens(a[6], sh.lens, c10::kInt), starts(a[7], sh.lens + 4, c10::kInt);
        const Tensor out(a[10], rows_bytes, 2);
        void* ws = nullptr;
        size_t ws_bytes = 0;
        if (a[11] != Py_None) {
            const Tensor w(a[11], (wide)lib.prefill_bytes(&sh, longest), 0);
            ws = w.at;
            ws_bytes = (size_t)w.bytes;
        }
        void* s = stream_of(a[13]);
        return unlocked([&] {
            return lib.prefill_ws(q.at, c.k, c.v, c.ks, c.vs, tables.as<int32_t>(), lens.as<int32_t>(), starts.as<int32_t>(),
                                  rows, longest, out.at, ws, ws_bytes, &sh, s);
        });
    });
}

PyObject* gather(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    return guarded<12>(n, [&] {
        const Shape sh(a[10]);
        const int32_t seq = small_int(a[5]), begin = small_int(a[6]), end = small_int(a[7]);
        const wide rows = (end > begin ? (wide)end - begin : 0) * sh.row;
        const Cache c(a, sh);
        const Tensor tables(a[4], sh.tables, c10::kInt), k(a[8], rows, 2), v(a[9], rows, 2);
        void* s = stream_of(a[11]);
        return unlocked([&] {
            return lib.gather(c.k, c.v, c.ks, c.vs, tables.as<int32_t>(), seq, begin, end, k.at, v.at, &sh, s);
        });
    });
}

// bind(addresses of the library's functions in the order of `lib`, Shape, DecodePlan, current device, raw stream)
PyObject* bind(PyObject*, PyObject* args)
{
    unsigned long long f[13];
    PyObject* o[4];
    if (!PyArg_ParseTuple(args, "(KKKKKKKKKKKKK)OOOO", f, f + 1, f + 2, f + 3, f + 4, f + 5, f + 6, f + 7, f + 8, f + 9,
                          f + 10, f + 11, f + 12, o, o + 1, o + 2, o + 3))
        return nullptr;
    void* const at[] = {&lib.write_fp8, &lib.write_fp16, &lib.decode, &lib.step, &lib.prepare, &lib.scheduled, &lib.partitioned,
                        &lib.reduce, &lib.prefill_ws, &lib.gather, &lib.workspace_bytes, &lib.schedule_bytes, &lib.prefill_bytes};
    for (int i = 0; i < 13; ++i) {
        const uintptr_t p = (uintptr_t)f[i];
        memcpy(at[i], &p, sizeof p);
    }
    PyObject** const kept[] = {&lib.shape_class, &lib.plan_class, &lib.current_device, &lib.raw_stream};
    for (int i = 0; i < 4; ++i) {
        Py_INCREF(o[i]);
        Py_XDECREF(*kept[i]);
        *kept[i] = o[i];
    }
    Py_RETURN_NONE;
}

#define FAST(name) {#name, (PyCFunction)(void*)name, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {FAST(write_fp8), FAST(write_fp16), FAST(decode), FAST(step), FAST(prepare), FAST(scheduled),
                         FAST(partitioned), FAST(reduce), FAST(prefill_ws), FAST(gather),
                         {"bind", bind, METH_VARARGS, nullptr}, {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_binding", nullptr, -1, methods};

}  // namespace

// built_for: the torch whose headers these are.
PyMODINIT_FUNC PyInit__binding()
{
    PyObject* m = PyModule_Create(&module);
    if (m && PyModule_AddStringConstant(m, "built_for", COOPT_TORCH_VERSION) != 0) Py_CLEAR(m);
    return m;
}
