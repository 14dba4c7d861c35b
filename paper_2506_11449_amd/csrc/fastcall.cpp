// The short way from Python to the C ABI, for the calls of a training step.  Each function here does for one entry point what
// binding.py does for all of them -- dtype, shape, layout and device of every tensor, the outputs that are not given, the workspace's
// size, the call -- and only for the plain kind of call: exact tensors, the workspace large enough.  To any other (a block to be grown,
// a subclass of Tensor, a tensor without storage, anything that a check refuses) it answers None with nothing done, and binding.py
// goes the long way, which grows or raises.  Otherwise the answer is what the function of that name in binding.py returns.
//
// Why: small layers wait for the host.  A launch takes it 3 us or a little more, and checks and ctypes in Python added as much again:
// a call of a 64 x 64 layer with 16 tokens took 4.8 (selection), 5.4 (product) and 7.1 us (backward pass), here 3.0, 3.5 and 3.6;
// the layer's step 19.8 -> 14.0 us, a heuristic update of 3072 candidates, whose outputs are allocated, 15.0 -> 13.1 us.
#include <Python.h>

#include <ATen/ops/empty.h>
#include <torch/csrc/autograd/python_variable.h>

#include <algorithm>
#include <cstring>
#include <exception>
#include <unordered_map>

#include "../../include/dynadiag.h"

namespace {

// The entry points of the library that binding.py has loaded, in the order of bind()'s addresses.
struct Entries {
    decltype(&dd_workspace_bytes) workspace_bytes;
    decltype(&dd_fwd) fwd;
    decltype(&dd_bwd_input) bwd_input;
    decltype(&dd_bwd) bwd;
    decltype(&dd_bwd_weight) bwd_weight;
    decltype(&dd_select_diagonals) select_diagonals;
    decltype(&dd_select_prepare) select_prepare;
    decltype(&dd_diag_magnitude) diag_magnitude;
    decltype(&dd_diagheur_update) diagheur_update;
} lib;

struct LayerKey {
    int op;
    dd_layer l;
    bool operator==(const LayerKey &o) const
    {
        return op == o.op && l.tokens == o.l.tokens && l.in_features == o.l.in_features && l.out_features == o.l.out_features && l.K == o.l.K &&
               l.dtype == o.l.dtype && l.algo == o.l.algo;
    }
};
struct LayerHash {
    size_t operator()(const LayerKey &k) const
    {
        uint64_t h = uint64_t(k.l.tokens);
        for (const int v : {k.op, k.l.in_features, k.l.out_features, k.l.K, k.l.dtype, k.l.algo}) h = h * 0x9e3779b97f4a7c15ull + uint32_t(v) + (h >> 31);
        return size_t(h ^ (h >> 32));
    }
};

// Scratch of an entry point, a function of its sizes alone: asked for once per layer.  Called with Python's lock held, like all here.
size_t scratch(int op, const dd_layer &l)
{
    static std::unordered_map<LayerKey, size_t, LayerHash> known;
    const LayerKey key = {op, l};
    const auto hit = known.find(key);
    if (hit != known.end()) return hit->second;
    if (known.size() >= 4096) known.clear();
    return known[key] = lib.workspace_bytes(op, &l, 0);
}

constexpr int64_t kMost = INT32_MAX;

bool whole(PyObject *o, int64_t lo, int64_t hi, int64_t &v)
{
    if (!PyLong_CheckExact(o)) return false;
    int overflow = 0;
    v = PyLong_AsLongLongAndOverflow(o, &overflow);
    return !overflow && v >= lo && v <= hi;
}

// The handle of the stream given, or (None) of the current one.  Asked for last: a call that goes the long way has not touched the GPU.
PyObject *current_stream = nullptr;
bool handle(PyObject *o, void *&stream)
{
    PyObject *h = o == Py_None ? PyObject_CallNoArgs(current_stream) : PyObject_GetAttrString(o, "cuda_stream");
    int64_t v;
    const bool ok = h && whole(h, 0, INT64_MAX, v);
    Py_XDECREF(h);
    if (ok) stream = reinterpret_cast<void *>(v);
    return ok;
}

// The tensor behind an object, if it is an exact one on the GPU with its elements in order (a wrapper of vmap or grad has no storage).
const at::Tensor *tensor(PyObject *o)
{
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor &t = THPVariable_Unpack(o);
    return t.defined() && t.has_storage() && t.layout() == at::kStrided && t.is_cuda() && t.is_contiguous() ? &t : nullptr;
}
const at::Tensor *tensor(PyObject *o, int64_t dims, at::ScalarType type)
{
    const at::Tensor *t = tensor(o);
    return t && t->dim() == dims && t->scalar_type() == type ? t : nullptr;
}
const at::Tensor *matrix(PyObject *o, at::ScalarType type, int64_t rows, int64_t cols)
{
    const at::Tensor *t = tensor(o, 2, type);
    return t && t->size(0) == rows && t->size(1) == cols ? t : nullptr;
}
const at::Tensor *vector(PyObject *o, at::ScalarType type, int64_t n)
{
    const at::Tensor *t = tensor(o, 1, type);
    return t && t->size(0) == n ? t : nullptr;
}
// a matrix of one of the two storage types
const at::Tensor *stored(PyObject *o, int32_t &dtype)
{
    const at::Tensor *t = tensor(o);
    if (!t || t->dim() != 2 || (t->scalar_type() != at::kFloat && t->scalar_type() != at::kBFloat16)) return nullptr;
    dtype = t->scalar_type() == at::kFloat ? DD_F32 : DD_BF16;
    return t;
}

bool sizes(dd_layer &l, int64_t T, int64_t M, int64_t N, int64_t K)
{
    if (M < 1 || N < 1 || K < 1 || M > kMost || N > kMost || K > kMost) return false;
    l.tokens = T, l.in_features = int32_t(M), l.out_features = int32_t(N), l.K = int32_t(K);
    return true;
}

// A block of bytes: the workspace, if it is as large as the call needs and lies on its device (... for the block that binding.py keeps
// for calls without one), or prepared operands.
struct Block {
    void *p = nullptr;
    size_t n = 0;
    PyObject *kept = nullptr;  // a block of binding.py, held for as long as the call is being made
    ~Block() { Py_XDECREF(kept); }
};
PyObject *default_block = nullptr;
bool workspace(PyObject *o, size_t need, PyObject *beside_object, const at::Tensor &beside, PyObject *stream, Block &b)
{
    if (o == Py_Ellipsis) {
        if (need == 0) return true;
        b.kept = PyObject_CallFunction(default_block, "nOO", Py_ssize_t(need), beside_object, stream);
        o = b.kept;
        if (!o) return false;
    }
    const at::Tensor *t = o == Py_None ? nullptr : tensor(o, 1, at::kByte);
    if (o != Py_None && !t) return false;
    if (need == 0) return true;
    if (!t || size_t(t->numel()) < need || t->device() != beside.device()) return false;
    b.p = t->data_ptr(), b.n = size_t(t->numel());
    return true;
}
bool operands(PyObject *o, Block &b)
{
    const at::Tensor *t = tensor(o, 1, at::kByte);
    if (!t) return false;
    b.p = t->data_ptr(), b.n = size_t(t->numel());
    return true;
}

// Python's lock laid down while the allocator or a launch may wait, as torch and ctypes do
struct Unlocked {
    PyThreadState *const state = PyEval_SaveThread();
    ~Unlocked() { PyEval_RestoreThread(state); }
};

// An output: the tensor given for it, if it is one of that type and shape, or (None) a new one.
struct Output {
    PyObject *given = nullptr;
    at::Tensor t;
    bool take(PyObject *o, at::ScalarType type, at::IntArrayRef shape, const at::Tensor &beside)
    {
        if (o == Py_None) {
            const Unlocked free;
            t = at::empty(shape, at::TensorOptions().dtype(type).device(beside.device()));
            return true;
        }
        const at::Tensor *have = tensor(o, int64_t(shape.size()), type);
        if (!have || have->sizes() != shape) return false;
        given = o;
        t = *have;
        return true;
    }
    PyObject *object() const
    {
        if (!given) return THPVariable_Wrap(t);
        Py_INCREF(given);
        return given;
    }
};
PyObject *result(const Output &a) { return a.object(); }
PyObject *result(const Output &a, const Output &b)
{
    PyObject *x = a.object(), *y = b.object(), *both = x && y ? PyTuple_Pack(2, x, y) : nullptr;
    Py_XDECREF(x);
    Py_XDECREF(y);
    return both;
}

template <typename... P, typename... A>
dd_status call(dd_status (*entry)(P...), A... args)
{
    const Unlocked free;
    return entry(args...);
}

// What body returns for a call that it has made: its result, or for another status the exception that binding.py's check raises.
// None where body gives up before (it answers kLongWay); what torch throws on the way binding.py will meet again.
constexpr int kLongWay = -1;
PyObject *check = nullptr;
template <typename F, typename... R>
PyObject *answer(F body, R &...results)
{
    int status = kLongWay;
    try {
        status = body();
    } catch (...) {
    }
    if (status == kLongWay) {
        if (PyErr_Occurred() && !PyErr_ExceptionMatches(PyExc_Exception)) return nullptr;  // an interrupt is not a refusal
        PyErr_Clear();
        Py_RETURN_NONE;
    }
    try {
        return status == DD_OK ? result(results...) : PyObject_CallFunction(check, "i", status);
    } catch (const std::exception &e) {  // a new output that cannot be wrapped
        if (!PyErr_Occurred()) PyErr_SetString(PyExc_RuntimeError, e.what());
        return nullptr;
    }
}

// product(transposed, src, offsets, values, dst, features of dst, algo, workspace, stream)
PyObject *product(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    Output dst;
    return answer(
        [&] {
            int64_t back, wide, algo;
            void *stream;
            dd_layer l;
            Block ws;
            if (n != 9 || !whole(a[0], 0, 1, back) || !whole(a[5], 1, kMost, wide) || !whole(a[6], 0, kMost, algo)) return kLongWay;
            const at::Tensor *src = stored(a[1], l.dtype), *offsets = tensor(a[2], 1, at::kInt);
            if (!src || !offsets) return kLongWay;
            const int64_t T = src->size(0), M = back ? wide : src->size(1), N = back ? src->size(1) : wide, K = offsets->size(0);
            const at::Tensor *values = matrix(a[3], src->scalar_type(), K, std::min(M, N));
            if (!values || !sizes(l, T, M, N, K)) return kLongWay;
            l.algo = int32_t(algo);
            if (!workspace(a[7], scratch(back ? DD_OP_BWD_INPUT : DD_OP_FWD, l), a[1], *src, a[8], ws) || !dst.take(a[4], src->scalar_type(), {T, wide}, *src) ||
                !handle(a[8], stream))
                return kLongWay;
            return int(call(back ? lib.bwd_input : lib.fwd, &l, src->data_ptr(), offsets->data_ptr<int32_t>(), values->data_ptr(),
                            dst.t.data_ptr(), ws.p, ws.n, stream));
        },
        dst);
}

// product_prepared(transposed, src, offsets (read for blocks alone), dst, in_features, out_features, K, algo, operands, stream)
PyObject *product_prepared(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    Output dst;
    return answer(
        [&] {
            int64_t back, M, N, K, algo;
            void *stream;
            dd_layer l;
            Block prepared;
            if (n != 10 || !whole(a[0], 0, 1, back) || !whole(a[4], 1, kMost, M) || !whole(a[5], 1, kMost, N) || !whole(a[6], 1, kMost, K) ||
                !whole(a[7], DD_ALGO_PREPARED, DD_ALGO_BLOCKS, algo) || !operands(a[8], prepared))
                return kLongWay;
            const at::Tensor *src = stored(a[1], l.dtype), *offsets = algo == DD_ALGO_BLOCKS ? vector(a[2], at::kInt, K) : nullptr;
            if (!src || (algo == DD_ALGO_BLOCKS && !offsets) || src->size(1) != (back ? N : M)) return kLongWay;
            if (!sizes(l, src->size(0), M, N, K)) return kLongWay;
            l.algo = int32_t(algo);
            if (!dst.take(a[3], src->scalar_type(), {l.tokens, back ? M : N}, *src) || !handle(a[9], stream)) return kLongWay;
            return int(call(back ? lib.bwd_input : lib.fwd, &l, src->data_ptr(), offsets ? offsets->data_ptr<int32_t>() : nullptr, nullptr,
                            dst.t.data_ptr(), prepared.p, prepared.n, stream));
        },
        dst);
}

// bwd(X, dY, offsets, values or None, operands or None, dX, dValues, algo, workspace, stream)
PyObject *bwd(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    Output dX, dV;
    return answer(
        [&] {
            int64_t algo;
            void *stream;
            dd_layer l;
            Block prepared, ws;
            if (n != 10 || !whole(a[7], 0, kMost, algo) || (a[4] != Py_None && !operands(a[4], prepared))) return kLongWay;
            const at::Tensor *X = stored(a[0], l.dtype), *offsets = tensor(a[2], 1, at::kInt);
            if (!X || !offsets) return kLongWay;
            const auto type = X->scalar_type();
            const at::Tensor *dY = tensor(a[1], 2, type);
            if (!dY || dY->size(0) != X->size(0) || !sizes(l, X->size(0), X->size(1), dY->size(1), offsets->size(0))) return kLongWay;
            const int64_t L = std::min(l.in_features, l.out_features);
            const at::Tensor *values = a[3] == Py_None ? nullptr : matrix(a[3], type, l.K, L);
            if (!values && (a[3] != Py_None || a[4] == Py_None)) return kLongWay;
            l.algo = int32_t(algo);
            if (!workspace(a[8], scratch(DD_OP_BWD, l), a[0], *X, a[9], ws) || !dX.take(a[5], type, {l.tokens, l.in_features}, *X) ||
                !dV.take(a[6], at::kFloat, {l.K, L}, *X) || !handle(a[9], stream))
                return kLongWay;
            return int(call(lib.bwd, &l, X->data_ptr(), dY->data_ptr(), offsets->data_ptr<int32_t>(), values ? values->data_ptr() : nullptr,
                            prepared.p, prepared.n, dX.t.data_ptr(), dV.t.data_ptr<float>(), ws.p, ws.n, stream));
        },
        dX, dV);
}

// bwd_weight(X, dY, offsets, dValues, algo, workspace, stream)
PyObject *bwd_weight(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    Output dV;
    return answer(
        [&] {
            int64_t algo;
            void *stream;
            dd_layer l;
            Block ws;
            if (n != 7 || !whole(a[4], 0, kMost, algo)) return kLongWay;
            const at::Tensor *X = stored(a[0], l.dtype), *offsets = tensor(a[2], 1, at::kInt);
            if (!X || !offsets) return kLongWay;
            const at::Tensor *dY = tensor(a[1], 2, X->scalar_type());
            if (!dY || dY->size(0) != X->size(0) || !sizes(l, X->size(0), X->size(1), dY->size(1), offsets->size(0))) return kLongWay;
            l.algo = int32_t(algo);
            if (!workspace(a[5], scratch(DD_OP_BWD_WEIGHT, l), a[0], *X, a[6], ws) ||
                !dV.take(a[3], at::kFloat, {l.K, std::min(l.in_features, l.out_features)}, *X) || !handle(a[6], stream))
                return kLongWay;
            return int(call(lib.bwd_weight, &l, X->data_ptr(), dY->data_ptr(), offsets->data_ptr<int32_t>(), dV.t.data_ptr<float>(), ws.p, ws.n, stream));
        },
        dV);
}

// select_diagonals(scores, K, offsets_out, stream): the selection takes no scratch
PyObject *select_diagonals(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    Output out;
    return answer(
        [&] {
            int64_t K;
            void *stream;
            if (n != 4 || !whole(a[1], 1, kMost, K)) return kLongWay;
            const at::Tensor *scores = tensor(a[0], 2, at::kFloat);
            if (!scores || scores->size(0) > kMost || scores->size(1) > kMost) return kLongWay;
            if (!out.take(a[2], at::kInt, {scores->size(0), K}, *scores) || !handle(a[3], stream)) return kLongWay;
            return int(call(lib.select_diagonals, int32_t(scores->size(0)), int32_t(scores->size(1)), int32_t(K), scores->data_ptr<float>(),
                            out.t.data_ptr<int32_t>(), nullptr, size_t(0), stream));
        },
        out);
}

// select_prepare(scores, values, in_features, out_features, offsets_out, operands, stream)
PyObject *select_prepare(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    Output out;
    return answer(
        [&] {
            int64_t M, N;
            void *stream;
            dd_layer l;
            Block prepared;
            if (n != 7 || !whole(a[2], 1, kMost, M) || !whole(a[3], 1, kMost, N) || !operands(a[5], prepared)) return kLongWay;
            const at::Tensor *values = stored(a[1], l.dtype), *scores = vector(a[0], at::kFloat, std::max(M, N));
            if (!values || !scores || values->size(1) != std::min(M, N) || !sizes(l, 0, M, N, values->size(0))) return kLongWay;
            l.algo = DD_ALGO_PREPARED;
            if (!out.take(a[4], at::kInt, {l.K}, *values) || !handle(a[6], stream)) return kLongWay;
            return int(call(lib.select_prepare, &l, scores->data_ptr<float>(), values->data_ptr(), out.t.data_ptr<int32_t>(), prepared.p, prepared.n, stream));
        },
        out);
}

// diag_magnitude(values, magnitudes, stream)
PyObject *diag_magnitude(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    Output out;
    return answer(
        [&] {
            void *stream;
            int32_t dtype;
            if (n != 3) return kLongWay;
            const at::Tensor *values = stored(a[0], dtype);
            if (!values || values->size(0) > kMost || values->size(1) > kMost) return kLongWay;
            if (!out.take(a[1], at::kFloat, {values->size(0)}, *values) || !handle(a[2], stream)) return kLongWay;
            return int(call(lib.diag_magnitude, int32_t(values->size(0)), int32_t(values->size(1)), dtype, values->data_ptr(),
                            out.t.data_ptr<float>(), stream));
        },
        out);
}

// diagheur_update(D, n_drop, offsets, magnitudes, random, new_offsets, source, workspace, stream)
PyObject *diagheur_update(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    Output fresh, source;
    return answer(
        [&] {
            int64_t D, drop;
            void *stream;
            dd_layer l;
            Block ws;
            if (n != 9 || !whole(a[0], 1, kMost, D) || !whole(a[1], 0, kMost, drop)) return kLongWay;
            const at::Tensor *offsets = tensor(a[2], 1, at::kInt);
            if (!offsets || !sizes(l, 0, D, D, offsets->size(0))) return kLongWay;
            const at::Tensor *magnitudes = vector(a[3], at::kFloat, l.K), *random = vector(a[4], at::kFloat, D);
            if (!magnitudes || !random) return kLongWay;
            l.dtype = DD_F32, l.algo = DD_ALGO_AUTO;
            if (!workspace(a[7], scratch(DD_OP_DIAGHEUR, l), a[2], *offsets, a[8], ws) || !fresh.take(a[5], at::kInt, {l.K}, *offsets) ||
                !source.take(a[6], at::kInt, {l.K}, *offsets) || !handle(a[8], stream))
                return kLongWay;
            return int(call(lib.diagheur_update, int32_t(D), l.K, int32_t(drop), offsets->data_ptr<int32_t>(), magnitudes->data_ptr<float>(),
                            random->data_ptr<float>(), fresh.t.data_ptr<int32_t>(), source.t.data_ptr<int32_t>(), ws.p, ws.n, stream));
        },
        fresh, source);
}

// bind(function that answers the current stream's handle, function that raises for a status, function that answers the scratch of
// calls without a workspace, addresses of Entries in order)
PyObject *bind(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    constexpr int kEntries = sizeof(Entries) / sizeof(void *);
    if (n != 3 + kEntries) return PyErr_Format(PyExc_TypeError, "bind takes three functions and %d addresses", kEntries);
    void *p[kEntries];
    for (int i = 0; i < kEntries; ++i) {
        p[i] = PyLong_AsVoidPtr(a[3 + i]);
        if (PyErr_Occurred()) return nullptr;
    }
    PyObject **const functions[] = {&current_stream, &check, &default_block};
    for (int i = 0; i < 3; ++i) {
        Py_INCREF(a[i]);
        Py_XSETREF(*functions[i], a[i]);
    }
    memcpy(&lib, p, sizeof lib);
    Py_RETURN_NONE;
}

#define DD_METHOD(name_) {#name_, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(&name_)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {DD_METHOD(bind), DD_METHOD(product), DD_METHOD(product_prepared), DD_METHOD(bwd), DD_METHOD(bwd_weight), DD_METHOD(select_diagonals),
                         DD_METHOD(select_prepare), DD_METHOD(diag_magnitude), DD_METHOD(diagheur_update), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_fastcall", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__fastcall(void) { return PyModule_Create(&module); }
