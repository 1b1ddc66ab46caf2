// The short way from Python to the entry points of include/spin.h: a CPython extension that reads the tensors' pointers, allocates
// the results and calls the library, for well-formed arguments.  A call of the ctypes binding spends 1 to 2.7 us on looking at its
// arguments and up to 2.5 on allocating in Python, as long as its kernels run on the smallest inputs: a 64^3 layer of three parties
// (two sharings, a product, a truncation) took 22 us back to back, of which its kernels are 12.
//
// Every function returns the result, or None for whatever it does not take (other types, shapes that disagree, an `out` that is too short, subclasses, modes that
// look at calls, workspaces beyond what needs no look at the device's memory, no memory left): spin.py then goes the way that
// says what is wrong, or does it.  A status of the library other than SPIN_OK comes back as an int.  Nothing is kept between calls but the
// addresses of the library's functions.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/ATen.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/hip/HIPFunctions.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/csrc/utils/object_ptr.h>

#include <array>
#include <vector>

#include "../../include/spin.h"

namespace {

struct Library {
    decltype(&spin_share) share, bshare;
    decltype(&spin_open) open, bopen;
    decltype(&spin_beaver_mul) beaver_mul, beaver_and;
    decltype(&spin_trunc) trunc;
    decltype(&spin_beaver_matmul) matmul, matmul_nt;
    decltype(&spin_beaver_matmul_preferred_workspace_bytes) matmul_preferred;
    decltype(&spin_beaver_matmul_grouped) grouped;
    decltype(&spin_beaver_matmul_grouped_workspace_bytes) grouped_bytes;
    decltype(&spin_completed_square_trunc) completed_square;
} lib;
constexpr int kEntries = sizeof(Library) / sizeof(void *);
size_t unasked_bytes;                                    // workspaces up to this size are taken without a look at the device's memory

// ---- arguments ------------------------------------------------------------------------------------------------
// A contiguous int64 CUDA tensor with memory of its own; null for anything else.
inline const at::Tensor *ring_tensor(PyObject *o)
{
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor &t = THPVariable_Unpack(o);
    if (!t.defined() || !t.has_storage() || !t.is_cuda() || t.scalar_type() != at::kLong || !t.is_contiguous()) return nullptr;
    return &t;
}
inline uint64_t *words(const at::Tensor &t) { return (uint64_t *)t.mutable_data_ptr(); }

// Plain ints only; 64-bit ones wrap as they do in ctypes.
inline bool word(PyObject *o, uint64_t &v)
{
    if (!PyLong_CheckExact(o)) return false;
    v = PyLong_AsUnsignedLongLongMask(o);
    return true;
}
inline bool integer(PyObject *o, int least, int most, int &v)
{
    if (!PyLong_CheckExact(o)) return false;
    int overflow = 0;
    const long n = PyLong_AsLongAndOverflow(o, &overflow);
    if (overflow || n < least || n > most) return false;
    v = (int)n;
    return true;
}
inline bool parties(int64_t n) { return n >= 1 && n <= SPIN_MAX_PARTIES; }

PyObject *none() { Py_RETURN_NONE; }

// The interpreter's lock is given up for a library call, and taken again however that ends: guarded() answers exceptions with it.
struct Unlocked {
    PyThreadState *state = PyEval_SaveThread();
    ~Unlocked() { PyEval_RestoreThread(state); }
};
// The call on torch's current stream (which is asked for before: that may throw).
template <class F> inline spin_status unlocked(F &&call)
{
    const spin_stream stream = (spin_stream)c10::hip::getCurrentHIPStream(c10::hip::current_device()).stream();
    const Unlocked scope;
    return call(stream);
}
// The result, or the status as an int.
template <class F> inline PyObject *run(const at::Tensor &result, F &&call)
{
    const spin_status st = unlocked(call);
    return st == SPIN_OK ? THPVariable_Wrap(result) : PyLong_FromLong(st);
}

// What a function's body throws (torch's allocator, above all) is left to the long way.
template <class F> inline PyObject *guarded(F &&body)
{
    if (at::impl::torch_function_mode_enabled()) return none();
    try {
        return body();
    } catch (...) {
        PyErr_Clear();
        return none();
    }
}

// ---- calls ----------------------------------------------------------------------------------------------------
// (x, n, seed, stream_id, out)
PyObject *sharing(PyObject *const *a, Py_ssize_t count, decltype(lib.share) fn)
{
    return guarded([&]() -> PyObject * {
        const at::Tensor *x = count == 5 ? ring_tensor(a[0]) : nullptr, *out = nullptr;
        int n;
        uint64_t seed, stream_id;
        if (!x || !integer(a[1], 1, SPIN_MAX_PARTIES, n) || !word(a[2], seed) || !word(a[3], stream_id)) return none();
        if (a[4] != Py_None && (!(out = ring_tensor(a[4])) || out->numel() < n * x->numel())) return none();
        at::Tensor fresh;
        if (!out) {
            c10::SmallVector<int64_t, 8> shape{n};
            shape.append(x->sizes().begin(), x->sizes().end());
            fresh = at::empty(shape, x->options());
            out = &fresh;
        }
        const uint64_t *from = words(*x);
        uint64_t *to = words(*out);
        const size_t each = (size_t)x->numel();
        return run(*out, [&](spin_stream s) { return fn(from, each, n, seed, stream_id, to, s); });
    });
}

// (shares, mask, out)
PyObject *opening(PyObject *const *a, Py_ssize_t count, decltype(lib.open) fn)
{
    return guarded([&]() -> PyObject * {
        const at::Tensor *shares = count == 3 ? ring_tensor(a[0]) : nullptr, *mask = nullptr, *out = nullptr;
        if (!shares || shares->dim() < 1 || !parties(shares->size(0))) return none();
        if (a[1] != Py_None && (!(mask = ring_tensor(a[1])) || mask->sizes() != shares->sizes())) return none();
        // the library reads the number of elements off `out`
        if (a[2] != Py_None && (!(out = ring_tensor(a[2])) || out->numel() != shares->numel() / shares->size(0))) return none();
        at::Tensor fresh;
        if (!out) {
            fresh = at::empty(shares->sizes().slice(1), shares->options());
            out = &fresh;
        }
        const uint64_t *from = words(*shares), *masks = mask ? words(*mask) : nullptr;
        uint64_t *to = words(*out);
        const size_t each = (size_t)out->numel();
        const int n = (int)shares->size(0);
        return run(*out, [&](spin_stream s) { return fn(from, masks, each, n, to, s); });
    });
}

// the first `inputs` of a are tensors of one shape, the next but `extra` is out
template <int INPUTS, class F> inline PyObject *elementwise(PyObject *const *a, PyObject *out_arg, F &&call)
{
    const at::Tensor *t[INPUTS], *out = nullptr;
    for (int i = 0; i < INPUTS; ++i) {
        t[i] = ring_tensor(a[i]);
        if (!t[i] || t[i]->sizes() != t[0]->sizes()) return none();
    }
    if (t[0]->dim() < 1 || !parties(t[0]->size(0))) return none();
    if (out_arg != Py_None && (!(out = ring_tensor(out_arg)) || out->numel() < t[0]->numel())) return none();
    at::Tensor fresh;
    if (!out) {
        fresh = at::empty(t[0]->sizes(), t[0]->options());
        out = &fresh;
    }
    const uint64_t *v[INPUTS];
    for (int i = 0; i < INPUTS; ++i) v[i] = words(*t[i]);
    uint64_t *to = words(*out);
    const int n = (int)t[0]->size(0);
    const size_t each = (size_t)(t[0]->numel() / n);
    return run(*out, [&](spin_stream s) { return call(n, each, v, to, s); });
}

// (x, y, a, b, c, out)
PyObject *multiplying(PyObject *const *a, Py_ssize_t count, decltype(lib.beaver_mul) fn)
{
    return guarded([&]() -> PyObject * {
        if (count != 6) return none();
        return elementwise<5>(a, a[5], [&](int n, size_t each, const uint64_t *const *v, uint64_t *out, spin_stream s) {
            return fn(n, each, v[0], v[1], v[2], v[3], v[4], out, s);
        });
    });
}

// (x, r, r_top, r_msb, f, out)
PyObject *truncating(PyObject *const *a, Py_ssize_t count)
{
    return guarded([&]() -> PyObject * {
        int f;
        if (count != 6 || !integer(a[4], 1, 61, f)) return none();
        return elementwise<4>(a, a[5], [&](int n, size_t each, const uint64_t *const *v, uint64_t *out, spin_stream s) {
            return lib.trunc(n, each, f, v[0], v[1], v[2], v[3], out, s);
        });
    });
}

struct Product {
    const at::Tensor *X, *Y, *A, *B, *C, *out;
    at::Tensor fresh;
    int n, batch, M, N, K;
};
// X, Y, A, B, C (null or of another shape than they should have: false) and out or None; allocates out.
inline bool product(PyObject *const *a, PyObject *out, bool transposed, Product &p)
{
    if (!(p.X = ring_tensor(a[0])) || !(p.Y = ring_tensor(a[1])) || !(p.A = ring_tensor(a[2])) || !(p.B = ring_tensor(a[3])) ||
        !(p.C = ring_tensor(a[4])) || p.X->dim() != 4 || p.Y->dim() != 4)
        return false;
    const int64_t n = p.X->size(0), batch = p.X->size(1), M = p.X->size(2), K = p.X->size(3), N = p.Y->size(transposed ? 2 : 3);
    if (!parties(n) || std::max({batch, M, N, K}) > 0x7fffffff) return false;
    const std::array<int64_t, 4> y{n, batch, transposed ? N : K, transposed ? K : N}, z{n, batch, M, N};
    if (p.Y->sizes() != at::IntArrayRef(y) || p.A->sizes() != p.X->sizes() || p.B->sizes() != p.Y->sizes() || p.C->sizes() != at::IntArrayRef(z))
        return false;
    p.out = nullptr;
    if (out != Py_None && (!(p.out = ring_tensor(out)) || p.out->numel() < p.C->numel())) return false;
    if (!p.out) {
        p.fresh = at::empty(p.C->sizes(), p.C->options());
        p.out = &p.fresh;
    }
    p.n = (int)n, p.batch = (int)batch, p.M = (int)M, p.N = (int)N, p.K = (int)K;
    return true;
}
// workspace: a contiguous CUDA tensor
inline const at::Tensor *workspace_tensor(PyObject *o)
{
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor &t = THPVariable_Unpack(o);
    return t.defined() && t.has_storage() && t.is_cuda() && t.is_contiguous() ? &t : nullptr;
}

// (X, Y, A, B, C, path, out, workspace, y_transposed)
PyObject *matmul(PyObject *const *a, Py_ssize_t count)
{
    return guarded([&]() -> PyObject * {
        int path;
        Product p;
        if (count != 9 || !integer(a[5], 0, 1, path) || !PyBool_Check(a[8])) return none();
        const bool transposed = a[8] == Py_True;
        if (!product(a, a[6], transposed, p)) return none();
        const at::Tensor *ws = nullptr;
        at::Tensor fresh;
        if (a[7] != Py_None) {
            if (!(ws = workspace_tensor(a[7]))) return none();
        } else {
            const size_t size = lib.matmul_preferred(p.n, p.batch, p.M, p.N, p.K, path);
            if (size == 0 || size > unasked_bytes) return none();
            fresh = at::empty({(int64_t)size}, p.X->options().dtype(at::kByte));
            ws = &fresh;
        }
        auto fn = transposed ? lib.matmul_nt : lib.matmul;
        const uint64_t *X = words(*p.X), *Y = words(*p.Y), *A = words(*p.A), *B = words(*p.B), *C = words(*p.C);
        uint64_t *Z = words(*p.out);
        void *space = ws->mutable_data_ptr();
        const size_t bytes = (size_t)ws->numel() * ws->element_size();
        return run(*p.out, [&](spin_stream s) { return fn(p.n, p.batch, p.M, p.N, p.K, X, Y, A, B, C, Z, path, space, bytes, s); });
    });
}

// (groups, path, workspace): a list of dicts
PyObject *grouped(PyObject *const *a, Py_ssize_t count)
{
    return guarded([&]() -> PyObject * {
        int path;
        if (count != 3 || !PyList_CheckExact(a[0]) || !integer(a[1], 0, 1, path)) return none();
        const Py_ssize_t groups = PyList_GET_SIZE(a[0]);
        if (groups < 1 || groups > SPIN_MAX_GROUPS) return none();
        static PyObject *keys[7];
        if (!keys[0]) {
            const char *names[7] = {"X", "Y", "A", "B", "C", "out", "y_transposed"};
            for (int i = 6; i >= 0; --i) keys[i] = PyUnicode_InternFromString(names[i]);
        }
        std::vector<Product> p((size_t)groups);
        std::vector<spin_matmul_group> desc((size_t)groups);
        for (Py_ssize_t i = 0; i < groups; ++i) {
            PyObject *g = PyList_GET_ITEM(a[0], i), *v[7];
            if (!PyDict_CheckExact(g)) return none();
            for (int k = 0; k < 7; ++k) {
                v[k] = PyDict_GetItemWithError(g, keys[k]);
                if (!v[k] && (k < 5 || PyErr_Occurred())) return PyErr_Clear(), none();
            }
            if (v[6] && !PyBool_Check(v[6])) return none();
            const bool transposed = v[6] == Py_True;
            if (!product(v, v[5] ? v[5] : Py_None, transposed, p[i]) || p[i].n != p[0].n) return none();
            desc[i] = spin_matmul_group{p[i].batch, p[i].M, p[i].N, p[i].K, words(*p[i].X), words(*p[i].Y), words(*p[i].A), words(*p[i].B),
                                        words(*p[i].C), words(p[i].fresh.defined() ? p[i].fresh : *p[i].out), transposed ? 1 : 0};
        }
        const size_t need = lib.grouped_bytes(p[0].n, (int)groups, desc.data(), path);
        if (need == 0) return none();
        const at::Tensor *ws = nullptr;
        at::Tensor fresh;
        if (a[2] != Py_None) {
            if (!(ws = workspace_tensor(a[2]))) return none();
        } else {
            fresh = at::empty({(int64_t)need}, p[0].X->options().dtype(at::kByte));
            ws = &fresh;
        }
        void *space = ws->mutable_data_ptr();
        const size_t bytes = (size_t)ws->numel() * ws->element_size();
        THPObjectPtr list(PyList_New(groups));
        if (!list) return PyErr_Clear(), none();
        for (Py_ssize_t i = 0; i < groups; ++i) {
            PyObject *out = PyDict_GetItemWithError(PyList_GET_ITEM(a[0], i), keys[5]);
            PyObject *z = p[i].fresh.defined() ? THPVariable_Wrap(p[i].fresh) : Py_NewRef(out);
            if (!z) return PyErr_Clear(), none();
            PyList_SET_ITEM(list.get(), i, z);
        }
        const spin_status st = unlocked([&](spin_stream s) { return lib.grouped(p[0].n, (int)groups, desc.data(), path, space, bytes, s); });
        return st == SPIN_OK ? list.release() : PyLong_FromLong(st);
    });
}

// (x, t3, t2, lin, t0, triples, tuples, f, out): triples and tuples two sequences of three tensors
PyObject *completed_square(PyObject *const *a, Py_ssize_t count)
{
    return guarded([&]() -> PyObject * {
        uint64_t c[4];
        int f[2];
        if (count != 9 || !PyTuple_CheckExact(a[7]) || PyTuple_GET_SIZE(a[7]) != 2) return none();
        for (int i = 0; i < 4; ++i)
            if (!word(a[1 + i], c[i])) return none();
        for (int i = 0; i < 2; ++i)
            if (!integer(PyTuple_GET_ITEM(a[7], i), 1, 61, f[i])) return none();
        PyObject *t[13] = {a[0]};
        int filled = 1;
        for (int k = 0; k < 2; ++k) {
            PyObject *two = a[5 + k];
            if (!PyList_CheckExact(two) && !PyTuple_CheckExact(two)) return none();
            if (PySequence_Fast_GET_SIZE(two) != 2) return none();
            for (int i = 0; i < 2; ++i) {
                PyObject *three = PySequence_Fast_GET_ITEM(two, i);
                if (!PyTuple_CheckExact(three) || PyTuple_GET_SIZE(three) != 3) return none();
                for (int j = 0; j < 3; ++j) t[filled++] = PyTuple_GET_ITEM(three, j);
            }
        }
        return elementwise<13>(t, a[8], [&](int n, size_t each, const uint64_t *const *v, uint64_t *out, spin_stream s) {
            return lib.completed_square(n, each, v[0], c[0], c[1], c[2], c[3], v + 1, v + 7, f, out, s);
        });
    });
}

// ---- module ---------------------------------------------------------------------------------------------------
// bind(addresses of the library's functions in the order of Library, bytes that need no look at the device's memory)
PyObject *bind(PyObject *, PyObject *const *a, Py_ssize_t count)
{
    if (count != 2 || !PyTuple_CheckExact(a[0]) || PyTuple_GET_SIZE(a[0]) != kEntries) {
        PyErr_SetString(PyExc_TypeError, "bind takes the library's addresses and a size");
        return nullptr;
    }
    void *entries[kEntries];
    for (int i = 0; i < kEntries; ++i) entries[i] = PyLong_AsVoidPtr(PyTuple_GET_ITEM(a[0], i));
    unasked_bytes = PyLong_AsSize_t(a[1]);
    if (PyErr_Occurred()) return nullptr;
    memcpy(&lib, entries, sizeof lib);
    return none();
}

#define FAST(name, call) \
    {name, (PyCFunction)(void *)+[](PyObject *, PyObject *const *a, Py_ssize_t count) -> PyObject * { return call; }, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {{"bind", (PyCFunction)(void *)bind, METH_FASTCALL, nullptr},
                         FAST("share", sharing(a, count, lib.share)),
                         FAST("bshare", sharing(a, count, lib.bshare)),
                         FAST("open", opening(a, count, lib.open)),
                         FAST("bopen", opening(a, count, lib.bopen)),
                         FAST("beaver_mul", multiplying(a, count, lib.beaver_mul)),
                         FAST("beaver_and", multiplying(a, count, lib.beaver_and)),
                         FAST("trunc", truncating(a, count)),
                         FAST("matmul", matmul(a, count)),
                         FAST("grouped", grouped(a, count)),
                         FAST("completed_square", completed_square(a, count)),
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_binding", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__binding() { return PyModule_Create(&module); }
