// vpp_torch.cpp -- the Python wrapper's calls, made from C++.
//
// A run is 20 to 25 pointers, strides and sizes out of five tensors. Read and
// checked in Python and passed through ctypes they take 12 us a call, more than
// the kernel of a small chunk; read here, about 1 us and the launch. A Caller
// holds what a plan fixes (heads, dims, device, rows) and takes the plain case
// only: tensors that are exactly torch's own type, on the plan's device, of the
// dtype, shape and layout the entry point needs, launched on the current stream.
// For anything else it returns NOT_HANDLED before any device work, and the Python
// wrapper does the call its general way, errors included.
#include <Python.h>

#include <c10/hip/HIPFunctions.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include "vpp_chunk_attn.h"

namespace {

constexpr long NOT_HANDLED = -1;

// The C ABI, bound once by address from the library the ctypes binding loaded.
struct Api {
    decltype(&vpp_chunk_attn_run) run = nullptr;
    decltype(&vpp_chunk_attn_run_noalloc) run_noalloc = nullptr;
    decltype(&vpp_chunk_attn_run_mla) run_mla = nullptr;
    decltype(&vpp_chunk_attn_run_paged) run_paged = nullptr;
    decltype(&vpp_kv_append_paged) append = nullptr;
} api;

// A tensor argument: torch's own class, a plain strided GPU tensor of the given
// device (no functorch wrapper, no fake, lazy, conjugated or functional tensor).
const at::Tensor* plain(PyObject* o, int device, at::ScalarType dtype, int64_t ndim) {
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor& t = THPVariable_Unpack(o);
    static const uint64_t allowed =
        c10::DispatchKeySet({c10::DispatchKey::CUDA, c10::DispatchKey::AutogradCUDA, c10::DispatchKey::AutocastCUDA,
                               c10::DispatchKey::ADInplaceOrView})
            .raw_repr();
    if (!t.defined() || (t.key_set().raw_repr() & ~allowed) != 0) return nullptr;
    if (!t.is_cuda() || t.get_device() != device || t.layout() != at::kStrided) return nullptr;
    if (t.scalar_type() != dtype || t.dim() != ndim || t.stride(ndim - 1) != 1) return nullptr;
    return &t;
}

struct Caller {
    PyObject_HEAD
    vpp_chunk_attn_plan_t plan;
    int64_t hq, hkv, dqk, dv;
    int device;
    int64_t tokens, max_row;     // rows of q, cache rows the chunk reads
    int64_t segments, seg_rows;  // segments, most cache rows of one (paged)
};

// Pointer and strides of a tensor, read while the interpreter lock is held.
struct View {
    void* p = nullptr;
    int64_t s0 = 0, s1 = 0, s2 = 0;
    explicit View(const at::Tensor* t) : p(t->data_ptr()), s0(t->stride(0)) {
        if (t->dim() > 1) s1 = t->stride(1);
        if (t->dim() > 2) s2 = t->stride(2);
    }
    View() = default;
};

// q, out and lse as every run takes them; false: not the plain case.
struct IO {
    View q, out, lse;
};
bool get_io(const Caller* c, PyObject* q, PyObject* out, PyObject* lse, IO& io) {
    if (!c->plan) return false;
    const at::Tensor* tq = plain(q, c->device, at::kBFloat16, 3);
    const at::Tensor* to = plain(out, c->device, at::kBFloat16, 3);
    if (!tq || !to) return false;
    if (tq->size(0) < c->tokens || tq->size(1) != c->hq || tq->size(2) != c->dqk) return false;
    if (to->size(0) < c->tokens || to->size(1) != c->hq || to->size(2) != c->dv) return false;
    io.q = View(tq);
    io.out = View(to);
    if (lse != Py_None) {
        const at::Tensor* t = plain(lse, c->device, at::kFloat, 2);
        if (!t || t->size(0) != c->hq || t->size(1) < c->tokens) return false;
        io.lse = View(t);
    }
    return true;
}
const at::Tensor* cache(const Caller* c, PyObject* o, int64_t heads, int64_t dim) {
    const at::Tensor* t = plain(o, c->device, at::kBFloat16, 3);
    return t && t->size(1) == heads && t->size(2) == dim && t->size(0) >= c->max_row ? t : nullptr;
}

void* stream_of(int device) { return (void*)c10::hip::getCurrentHIPStream((c10::DeviceIndex)device).stream(); }

PyObject* not_handled() { return PyLong_FromLong(NOT_HANDLED); }

// Runs `prepare`, which checks the arguments and returns false for what it does not
// take (so does an exception of torch's accessors), then `call` without the
// interpreter lock, as ctypes does.
template <typename P, typename F>
PyObject* checked_call(P&& prepare, F&& call) {
    try {
        if (!prepare()) return not_handled();
    } catch (...) {
        return not_handled();
    }
    vpp_status_t st;
    Py_BEGIN_ALLOW_THREADS
    st = call();
    Py_END_ALLOW_THREADS
    return PyLong_FromLong((long)st);
}

#define Q_ARGS io.q.p, io.q.s0, io.q.s1
#define OUT_ARGS io.out.p, io.out.s0, io.out.s1, (float*)io.lse.p, io.lse.s0

PyObject* call_run(PyObject* self, PyObject* const* a, Py_ssize_t n) {
    const Caller* c = (Caller*)self;
    IO io;
    View k, v, ws;
    int64_t ws_bytes = 0;
    void* stream = nullptr;
    return checked_call(
        [&] {
            if (n != 6 || !get_io(c, a[0], a[3], a[4], io)) return false;
            const at::Tensor *tk = cache(c, a[1], c->hkv, c->dqk), *tv = cache(c, a[2], c->hkv, c->dv);
            const at::Tensor* tw = plain(a[5], c->device, at::kByte, 1);
            if (!tk || !tv || !tw) return false;
            k = View(tk), v = View(tv), ws = View(tw);
            ws_bytes = tw->numel();
            stream = stream_of(c->device);
            return true;
        },
        [&] {
            return api.run(c->plan, Q_ARGS, k.p, k.s0, k.s1, v.p, v.s0, v.s1, OUT_ARGS, ws.p, (size_t)ws_bytes, stream);
        });
}

PyObject* call_run_noalloc(PyObject* self, PyObject* const* a, Py_ssize_t n) {
    const Caller* c = (Caller*)self;
    IO io;
    View k, v;
    void* stream = nullptr;
    return checked_call(
        [&] {
            if (n != 5 || !get_io(c, a[0], a[3], a[4], io)) return false;
            const at::Tensor *tk = cache(c, a[1], c->hkv, c->dqk), *tv = cache(c, a[2], c->hkv, c->dv);
            if (!tk || !tv) return false;
            // the library takes the scratch of the current device: the general path makes
            // the tensors' device current
            if ((int)c10::hip::current_device() != c->device) return false;
            k = View(tk), v = View(tv);
            stream = stream_of(c->device);
            return true;
        },
        [&] { return api.run_noalloc(c->plan, Q_ARGS, k.p, k.s0, k.s1, v.p, v.s0, v.s1, OUT_ARGS, stream); });
}

PyObject* call_run_mla(PyObject* self, PyObject* const* a, Py_ssize_t n) {
    const Caller* c = (Caller*)self;
    IO io;
    View kn, kr, v, ws;
    int64_t ws_bytes = 0;
    void* stream = nullptr;
    return checked_call(
        [&] {
            if (n != 7 || c->dqk != 192 || c->dv != 128 || !get_io(c, a[0], a[4], a[5], io)) return false;
            const at::Tensor *tn = cache(c, a[1], c->hkv, 128), *tv = cache(c, a[3], c->hkv, c->dv);
            const at::Tensor* tr = plain(a[2], c->device, at::kBFloat16, 2);
            const at::Tensor* tw = plain(a[6], c->device, at::kByte, 1);
            if (!tn || !tv || !tr || !tw || tr->size(1) != 64 || tr->size(0) < c->max_row) return false;
            kn = View(tn), kr = View(tr), v = View(tv), ws = View(tw);
            ws_bytes = tw->numel();
            stream = stream_of(c->device);
            return true;
        },
        [&] {
            return api.run_mla(c->plan, Q_ARGS, kn.p, kn.s0, kn.s1, kr.p, kr.s0, v.p, v.s0, v.s1, OUT_ARGS, ws.p,
                               (size_t)ws_bytes, stream);
        });
}

PyObject* call_run_paged(PyObject* self, PyObject* const* a, Py_ssize_t n) {
    const Caller* c = (Caller*)self;
    IO io;
    View k, v, bt, ws;
    int64_t ws_bytes = 0, pages = 0, page = 0;
    void* stream = nullptr;
    return checked_call(
        [&] {
            if (n != 7 || !get_io(c, a[0], a[4], a[5], io)) return false;
            const at::Tensor *tk = plain(a[1], c->device, at::kBFloat16, 4), *tv = plain(a[2], c->device, at::kBFloat16, 4);
            const at::Tensor* tb = plain(a[3], c->device, at::kInt, 2);
            const at::Tensor* tw = plain(a[6], c->device, at::kByte, 1);
            if (!tk || !tv || !tb || !tw) return false;
            if (tk->size(2) != c->hkv || tk->size(3) != c->dqk || tv->size(2) != c->hkv || tv->size(3) != c->dv) return false;
            pages = tk->size(0), page = tk->size(1);
            if (tv->size(0) != pages || tv->size(1) != page || pages > INT32_MAX || page > INT32_MAX) return false;
            if (tb->size(0) < c->segments || c->seg_rows > tb->size(1) * page) return false;
            k = View(tk), v = View(tv), bt = View(tb), ws = View(tw);
            ws_bytes = tw->numel();
            stream = stream_of(c->device);
            return true;
        },
        [&] {
            return api.run_paged(c->plan, Q_ARGS, k.p, k.s0, k.s1, k.s2, v.p, v.s0, v.s1, v.s2, (int32_t)page,
                                 (int32_t)pages, (const int32_t*)bt.p, bt.s0, OUT_ARGS, ws.p, (size_t)ws_bytes, stream);
        });
}

// append(k_new, v_new, k_pages, v_pages, slot_mapping) on the current stream
PyObject* call_append(PyObject*, PyObject* const* a, Py_ssize_t n) {
    View kn, vn, k, v, slots;
    int64_t tokens = 0, heads = 0, dqk = 0, dv = 0, pages = 0, page = 0;
    void* stream = nullptr;
    return checked_call(
        [&] {
            if (n != 5 || !THPVariable_CheckExact(a[0])) return false;
            const at::Tensor& t0 = THPVariable_Unpack(a[0]);
            if (!t0.defined() || !t0.is_cuda()) return false;
            const int dev = (int)t0.get_device();
            const at::Tensor *tkn = plain(a[0], dev, at::kBFloat16, 3), *tvn = plain(a[1], dev, at::kBFloat16, 3);
            const at::Tensor *tk = plain(a[2], dev, at::kBFloat16, 4), *tv = plain(a[3], dev, at::kBFloat16, 4);
            const at::Tensor* ts = plain(a[4], dev, at::kLong, 1);
            if (!tkn || !tvn || !tk || !tv || !ts) return false;
            tokens = tkn->size(0), heads = tkn->size(1), dqk = tkn->size(2), dv = tvn->size(2);
            pages = tk->size(0), page = tk->size(1);
            if (tvn->size(0) != tokens || tvn->size(1) != heads || ts->size(0) != tokens) return false;
            if (tk->size(2) != heads || tk->size(3) != dqk || tv->size(2) != heads || tv->size(3) != dv) return false;
            if (tv->size(0) != pages || tv->size(1) != page) return false;
            for (const int64_t x : {tokens, heads, dqk, dv, pages, page})
                if (x > INT32_MAX) return false;
            kn = View(tkn), vn = View(tvn), k = View(tk), v = View(tv), slots = View(ts);
            stream = stream_of(dev);
            return true;
        },
        [&] {
            return api.append(kn.p, kn.s0, kn.s1, vn.p, vn.s0, vn.s1, k.p, k.s0, k.s1, k.s2, v.p, v.s0, v.s1, v.s2,
                              (int32_t)tokens, (int32_t)heads, (int32_t)dqk, (int32_t)dv, (int32_t)page, (int32_t)pages,
                              (const int64_t*)slots.p, stream);
        });
}

PyObject* call_set_plan(PyObject* self, PyObject* args) {
    Caller* c = (Caller*)self;
    unsigned long long plan;
    long long tokens, max_row, segments, seg_rows;
    if (!PyArg_ParseTuple(args, "KLLLL", &plan, &tokens, &max_row, &segments, &seg_rows)) return nullptr;
    c->plan = (vpp_chunk_attn_plan_t)(uintptr_t)plan;
    c->tokens = tokens;
    c->max_row = max_row;
    c->segments = segments;
    c->seg_rows = seg_rows;
    Py_RETURN_NONE;
}

int caller_init(PyObject* self, PyObject* args, PyObject*) {
    Caller* c = (Caller*)self;
    long long hq, hkv, dqk, dv;
    if (!PyArg_ParseTuple(args, "LLLLi", &hq, &hkv, &dqk, &dv, &c->device)) return -1;
    c->hq = hq;
    c->hkv = hkv;
    c->dqk = dqk;
    c->dv = dv;
    c->plan = nullptr;
    return 0;
}

PyMethodDef caller_methods[] = {
    {"set_plan", call_set_plan, METH_VARARGS, "set_plan(handle or 0, tokens, max_row, segments, seg_rows)"},
    {"run", (PyCFunction)(void (*)(void))call_run, METH_FASTCALL, "run(q, k, v, out, lse, workspace) -> status or -1"},
    {"run_noalloc", (PyCFunction)(void (*)(void))call_run_noalloc, METH_FASTCALL, "run_noalloc(q, k, v, out, lse)"},
    {"run_mla", (PyCFunction)(void (*)(void))call_run_mla, METH_FASTCALL, "run_mla(q, k_nope, k_rope, v, out, lse, workspace)"},
    {"run_paged", (PyCFunction)(void (*)(void))call_run_paged, METH_FASTCALL,
     "run_paged(q, k_pages, v_pages, block_table, out, lse, workspace)"},
    {nullptr, nullptr, 0, nullptr}};

PyTypeObject CallerType = {PyVarObject_HEAD_INIT(nullptr, 0)};

PyObject* bind(PyObject*, PyObject* args) {
    unsigned long long p[5];
    if (!PyArg_ParseTuple(args, "KKKKK", &p[0], &p[1], &p[2], &p[3], &p[4])) return nullptr;
    api.run = (decltype(api.run))(uintptr_t)p[0];
    api.run_noalloc = (decltype(api.run_noalloc))(uintptr_t)p[1];
    api.run_mla = (decltype(api.run_mla))(uintptr_t)p[2];
    api.run_paged = (decltype(api.run_paged))(uintptr_t)p[3];
    api.append = (decltype(api.append))(uintptr_t)p[4];
    Py_RETURN_NONE;
}

PyMethodDef module_methods[] = {
    {"bind", bind, METH_VARARGS, "bind(run, run_noalloc, run_mla, run_paged, append): addresses of the C entry points"},
    {"append", (PyCFunction)(void (*)(void))call_append, METH_FASTCALL,
     "append(k_new, v_new, k_pages, v_pages, slot_mapping) -> status or -1"},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module_def = {PyModuleDef_HEAD_INIT, "vpp_torch", "Calls of the attention library on torch tensors.", -1,
                          module_methods};

}  // namespace

PyMODINIT_FUNC PyInit_vpp_torch(void) {
    CallerType.tp_name = "vpp_torch.Caller";
    CallerType.tp_basicsize = sizeof(Caller);
    CallerType.tp_flags = Py_TPFLAGS_DEFAULT;
    CallerType.tp_doc = "Caller(num_q_heads, num_kv_heads, head_dim_qk, head_dim_v, device index)";
    CallerType.tp_methods = caller_methods;
    CallerType.tp_init = caller_init;
    CallerType.tp_new = PyType_GenericNew;
    if (PyType_Ready(&CallerType) < 0) return nullptr;
    PyObject* m = PyModule_Create(&module_def);
    if (!m) return nullptr;
    Py_INCREF(&CallerType);
    if (PyModule_AddObject(m, "Caller", (PyObject*)&CallerType) < 0) return nullptr;
    return m;
}
