// Argument marshalling of the Python binding (api.py) in native code: the checks a call makes on its tensors and the call into
// libmetro.so, without the dozen attribute look-ups and conversions per tensor that they cost in Python.
//
// Every function takes the address of a libmetro function and the arguments of the api.py call, all outputs allocated, and
// returns the library's status -- or kUnusual, with nothing enqueued, for anything that is not the plain case (a subclass of
// Tensor, another dtype, device or layout, a missing buffer, an integer out of range).  api.py then takes the same call
// through its Python checks, which decide and word what is refused.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <torch/csrc/autograd/python_variable.h>

#include <algorithm>
#include <cstdint>

#include "metro.h"

namespace {

constexpr long kUnusual = 1;                            // no status of the library is positive
static_assert(METRO_OK == 0, "statuses are zero or negative");

// An address that has passed the checks; converts to the pointer type that a prototype asks for.
struct Ptr {
    void* p = nullptr;
    template <typename T>
    operator T*() const { return static_cast<T*>(p); }
};

struct Args {
    PyObject* const* v;
    Py_ssize_t n, at = 0;
    bool ok = true;

    PyObject* next() {
        if (at < n) return v[at++];
        ok = false;
        return nullptr;
    }
    void* address() {
        PyObject* o = next();
        if (!o || !PyLong_CheckExact(o)) return ok = false, nullptr;
        void* p = PyLong_AsVoidPtr(o);
        if (PyErr_Occurred()) return PyErr_Clear(), ok = false, nullptr;
        return p;
    }
    int integer() {
        PyObject* o = next();
        if (!o || !PyLong_CheckExact(o)) return ok = false, 0;
        int over = 0;
        const long x = PyLong_AsLongAndOverflow(o, &over);
        if (over || x < INT32_MIN || x > INT32_MAX) return ok = false, 0;
        return (int)x;
    }
    // A plain tensor with memory of its own on the device.
    const at::Tensor* tensor() { return as_tensor(next()); }
    const at::Tensor* as_tensor(PyObject* o) {
        static const at::Tensor none;
        if (!o || !THPVariable_CheckExact(o)) return ok = false, &none;
        const at::Tensor& t = THPVariable_Unpack(o);
        if (!t.defined() || !t.is_cuda() || t.layout() != at::kStrided || !t.has_storage()) return ok = false, &none;
        return &t;
    }
    const at::Tensor* field(PyObject* dict, const char* name) {
        return as_tensor(dict && PyDict_CheckExact(dict) ? PyDict_GetItemString(dict, name) : nullptr);
    }
    // Pointer of a contiguous tensor of one dtype: of an input, and of a buffer that is written (which may be a lazy clone:
    // its mutable pointer gives it memory of its own first).
    Ptr in(const at::Tensor* t, at::ScalarType type = at::kInt) {
        if (!ok || t->scalar_type() != type || !t->is_contiguous()) return ok = false, Ptr{};
        return Ptr{const_cast<void*>(t->const_data_ptr())};
    }
    Ptr out(const at::Tensor* t, at::ScalarType type = at::kInt) {
        if (!ok || t->scalar_type() != type || !t->is_contiguous()) return ok = false, Ptr{};
        return Ptr{t->mutable_data_ptr()};
    }
};

PyObject *get_device, *get_raw_stream;                  // of torch._C; held for the life of the process

// The current stream of the current device, as torch.cuda.current_stream() gives it.
void* current_stream(Args& a) {
    if (!a.ok) return nullptr;
    PyObject* device = PyObject_CallNoArgs(get_device);
    PyObject* raw = device ? PyObject_CallOneArg(get_raw_stream, device) : nullptr;
    void* p = raw ? PyLong_AsVoidPtr(raw) : nullptr;
    Py_XDECREF(device);
    Py_XDECREF(raw);
    if (PyErr_Occurred()) return PyErr_Clear(), a.ok = false, nullptr;
    return p;
}

int32_t dtype_code(Args& a, const at::Tensor* t) {      // METRO_DTYPE_*
    if (a.ok && t->scalar_type() == at::kBFloat16) return METRO_DTYPE_BF16;
    if (a.ok && t->scalar_type() == at::kFloat) return METRO_DTYPE_F32;
    a.ok = false;
    return METRO_DTYPE_F32;
}

bool fits(int64_t v) { return v >= 0 && v <= INT32_MAX; }

PyObject* answer(long status) { return PyLong_FromLong(status); }
// fn: address of a library function, called as its prototype F in metro.h, without the interpreter lock, as through ctypes.
template <typename F, typename... A>
PyObject* call(void* fn, A... args) {
    int status;
    Py_BEGIN_ALLOW_THREADS
    status = reinterpret_cast<F>(fn)(args...);
    Py_END_ALLOW_THREADS
    return answer(status);
}
PyObject* unusual() {
    if (PyErr_Occurred()) PyErr_Clear();
    return answer(kUnusual);
}

// route(fn, metro, topk_ids, slot_to_expert, N, G, spr, out)
PyObject* route(PyObject*, PyObject* const* v, Py_ssize_t n) {
    Args a{v, n};
    void* fn = a.address();
    const int metro = a.integer();
    const at::Tensor *ids = a.tensor(), *s2e = a.tensor();
    const int N = a.integer(), G = a.integer(), spr = a.integer();
    PyObject* out = a.next();
    if (!a.ok || (ids->dim() != 2 && ids->dim() != 3) || (s2e->dim() != 1 && s2e->dim() != 2)) return unusual();
    const int64_t L = ids->dim() == 3 ? ids->size(0) : 1, T = ids->size(-2), k = ids->size(-1);
    if (!fits(L) || !fits(T) || !fits(k) || (s2e->dim() == 2 ? s2e->size(0) : 1) != L || s2e->size(-1) != (int64_t)G * spr)
        return unusual();
    const Ptr pi = a.in(ids), ps = a.in(s2e), slot = a.out(a.field(out, "pair_slot")), active = a.out(a.field(out, "rank_active")),
         bitmap = a.out(a.field(out, "rank_bitmap"), at::kLong), err = a.out(a.field(out, "err_flag"));
    const Ptr expert = metro ? a.out(a.field(out, "expert_slot")) : Ptr{};
    void* stream = current_stream(a);
    if (!a.ok) return unusual();
    if (metro)
        return call<decltype(&metro_route)>(fn, pi, ps, (int)L, (int)T, (int)k, N, G, spr, slot, expert, active, bitmap, err, stream);
    return call<decltype(&metro_route_token_balanced)>(fn, pi, ps, (int)L, (int)T, (int)k, N, G, spr, slot, active, bitmap, err, stream);
}

// route_permute(fn, metro, topk_ids, slot_to_expert, N, G, spr, rank, out, lists)
PyObject* route_permute(PyObject*, PyObject* const* v, Py_ssize_t n) {
    Args a{v, n};
    void* fn = a.address();
    const int metro = a.integer();
    const at::Tensor *ids = a.tensor(), *s2e = a.tensor();
    const int N = a.integer(), G = a.integer(), spr = a.integer(), rank = a.integer();
    PyObject *out = a.next(), *lists = a.next();
    if (!a.ok || ids->dim() != 2 || s2e->dim() != 1 || s2e->numel() != (int64_t)G * spr) return unusual();
    const int64_t T = ids->size(0), k = ids->size(1);
    if (!fits(T) || !fits(k)) return unusual();
    const Ptr pi = a.in(ids), ps = a.in(s2e), slot = a.out(a.field(out, "pair_slot")), active = a.out(a.field(out, "rank_active")),
         bitmap = a.out(a.field(out, "rank_bitmap"), at::kLong), err = a.out(a.field(out, "err_flag")),
         offsets = a.out(a.field(lists, "group_offsets")), perm = a.out(a.field(lists, "perm_pair")),
         row = a.out(a.field(lists, "pair_row")), pairs = a.out(a.field(lists, "n_pairs"));
    const Ptr expert = metro ? a.out(a.field(out, "expert_slot")) : Ptr{};
    void* stream = current_stream(a);
    if (!a.ok) return unusual();
    if (metro)
        return call<decltype(&metro_route_permute)>(fn, pi, ps, (int)T, (int)k, N, G, spr, rank, slot, expert, active, bitmap, err, offsets, perm, row, pairs, stream);
    return call<decltype(&metro_route_token_balanced_permute)>(fn, pi, ps, (int)T, (int)k, N, G, spr, rank, slot, active, bitmap, err, offsets, perm, row, pairs, stream);
}

// Weights [slots, rows, K]: K contiguous, rows `ld` elements apart, slots rows * ld apart.
Ptr weights(Args& a, const at::Tensor* t, at::ScalarType type, int64_t slots, int64_t rows, int64_t K, int& ld) {
    if (!a.ok || t->scalar_type() != type || t->dim() != 3 || t->size(0) != slots || t->size(1) != rows || t->size(2) != K)
        return a.ok = false, Ptr{};
    const int64_t pitch = rows > 1 ? t->stride(1) : std::max(K, t->stride(1));
    if (t->stride(2) != 1 || pitch < K || !fits(pitch) || (slots > 1 && t->stride(0) != rows * pitch)) return a.ok = false, Ptr{};
    ld = (int)pitch;
    return Ptr{const_cast<void*>(t->const_data_ptr())};
}

// ffn(fn, x, perm_pair, group_offsets, k, w13, w2, y_perm, ws)
PyObject* ffn(PyObject*, PyObject* const* v, Py_ssize_t n) {
    Args a{v, n};
    void* fn = a.address();
    const at::Tensor *x = a.tensor(), *perm = a.tensor(), *offsets = a.tensor();
    const int k = a.integer();
    const at::Tensor *w13 = a.tensor(), *w2 = a.tensor(), *y = a.tensor(), *ws = a.tensor();
    if (!a.ok || x->dim() != 2 || w13->dim() != 3) return unusual();
    const int64_t T = x->size(0), H = x->size(1), spr = w13->size(0), I = w13->size(1) / 2;
    if (!fits(T) || !fits(H) || !fits(spr) || !fits(I) || perm->numel() < T * k || offsets->numel() != spr + 1) return unusual();
    const int code = dtype_code(a, x);
    int ld13 = 0, ld2 = 0;
    const Ptr p13 = weights(a, w13, x->scalar_type(), spr, 2 * I, H, ld13), p2 = weights(a, w2, x->scalar_type(), spr, H, I, ld2);
    const Ptr px = a.in(x, x->scalar_type()), pp = a.in(perm), po = a.in(offsets), py = a.out(y, x->scalar_type()),
         pws = a.out(ws, at::kByte);
    void* stream = current_stream(a);
    if (!a.ok) return unusual();
    return call<decltype(&moe_grouped_ffn)>(fn, px, pp, po, (int)T, k, (int)spr, (int)H, (int)I, code, p13, ld13, p2, ld2, py, pws, (size_t)ws->numel(), stream);
}

// unpermute(fn, y_perm, pair_row, topk_w, out)
PyObject* unpermute(PyObject*, PyObject* const* v, Py_ssize_t n) {
    Args a{v, n};
    void* fn = a.address();
    const at::Tensor *y = a.tensor(), *row = a.tensor(), *w = a.tensor(), *out = a.tensor();
    if (!a.ok || row->dim() != 2 || y->dim() < 2) return unusual();
    const int64_t T = row->size(0), k = row->size(1), H = y->size(1);
    if (!fits(T) || !fits(k) || !fits(H)) return unusual();
    const int code = dtype_code(a, y);
    const Ptr py = a.in(y, y->scalar_type()), pr = a.in(row), pw = a.in(w, at::kFloat), po = a.out(out, y->scalar_type());
    void* stream = current_stream(a);
    if (!a.ok) return unusual();
    return call<decltype(&moe_unpermute)>(fn, py, pr, pw, (int)T, (int)k, (int)H, code, po, stream);
}

// gate_topk(fn, x, w_gate, k, out, ws, n_valid or None)
PyObject* gate_topk(PyObject*, PyObject* const* v, Py_ssize_t n) {
    Args a{v, n};
    void* fn = a.address();
    const at::Tensor *x = a.tensor(), *w = a.tensor();
    const int k = a.integer();
    PyObject* out = a.next();
    const at::Tensor* ws = a.tensor();
    PyObject* valid = a.next();
    const at::Tensor* nv = valid && valid != Py_None ? a.as_tensor(valid) : nullptr;
    if (!a.ok || x->dim() != 2 || w->dim() != 2 || w->size(1) != x->size(1) || w->stride(1) != 1 ||
        w->scalar_type() != x->scalar_type())
        return unusual();
    const int64_t T = x->size(0), H = x->size(1), N = w->size(0), ldw = N > 1 ? w->stride(0) : H;
    if (!fits(T) || !fits(H) || !fits(N) || !fits(ldw)) return unusual();
    const int code = dtype_code(a, x);
    const Ptr px = a.in(x, x->scalar_type()), ids = a.out(a.field(out, "topk_ids")),
         tw = a.out(a.field(out, "topk_w"), at::kFloat), cnt = a.out(a.field(out, "expert_count")),
         pws = a.out(ws, at::kByte), pnv = nv ? a.in(nv) : Ptr{};
    void* stream = current_stream(a);
    if (!a.ok) return unusual();
    return call<decltype(&moe_gate_topk)>(fn, px, Ptr{const_cast<void*>(w->const_data_ptr())}, (int)ldw, (int)T, (int)H, (int)N, k, code, pnv, ids, tw, cnt, pws, (size_t)ws->numel(), stream);
}

template <PyObject* (*F)(PyObject*, PyObject* const*, Py_ssize_t)>
PyObject* guarded(PyObject* self, PyObject* const* v, Py_ssize_t n) {
    try {
        return F(self, v, n);
    } catch (...) {                                     // a C++ exception of a tensor accessor: the Python checks word it
        return unusual();
    }
}

#define METRO_CALL(f) {#f, (PyCFunction)(void (*)(void))guarded<f>, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {METRO_CALL(route),     METRO_CALL(route_permute), METRO_CALL(ffn),
                         METRO_CALL(unpermute), METRO_CALL(gate_topk),     {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_call", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__call(void) {
    PyObject* torch_c = PyImport_ImportModule("torch._C");
    if (!torch_c) return nullptr;
    get_device = PyObject_GetAttrString(torch_c, "_cuda_getDevice");
    get_raw_stream = PyObject_GetAttrString(torch_c, "_cuda_getCurrentRawStream");
    Py_DECREF(torch_c);
    return get_device && get_raw_stream ? PyModule_Create(&module) : nullptr;
}
