// The entry points of the Python binding for plain calls, as one native function each: the checks of the arguments, the output
// tensor and the call of the C-ABI.  In Python a call takes the host 5.5 to 12 us, here 4.1 to 5.6, and small kernels take 4 to 10.
//
// A function returns the result, or None when anything about its arguments is not plain (no exact torch.Tensor on the current
// device, not contiguous, another number of dimensions or element type, a chunk size there is no kernel for, an argument of the
// wrong kind) or when the C-ABI refused the call.  No matrix has been formed or written then, and the caller goes through the Python route,
// which raises what there is to raise: this file has no error messages of its own.  (Packed sequences: their offsets may have been
// written already, by a kernel on the call's stream, into a tensor that is then given back to the allocator of that stream.  Whoever gets its
// memory next uses it behind that kernel, in a captured graph too.)  The same goes for C++ exceptions: libtorch throws them for
// tensors that do not have what they are asked for, and none may pass the C boundary to the interpreter.
//
// Device -1 stands for host memory: not for the library, whose kernels cannot read it, but for tests with a stand-in for the C-ABI.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <ATen/core/Tensor.h>
#include <ATen/ops/empty.h>
#include <torch/csrc/Dtype.h>
#include <torch/csrc/autograd/python_variable.h>
#include <stdint.h>
#include <vector>

namespace {

enum : int { F32 = 0, F16 = 1, BF16 = 2, FLAG_OUT_F16 = 0x2, FLAG_OUT_BF16 = 0x4 };

// The C-ABI, by address: the library is the one the ctypes binding has loaded.
struct Abi {
    int (*tri_inv_ex)(const void*, void*, int64_t, int, int, int, int, void*, uint32_t);
    int (*inv_ex)(const void*, const void*, const void*, void*, int, int64_t, int, int, int, int, int, int, int, void*, uint32_t);
    int (*inv_varlen)(const void*, const void*, const void*, void*, const int64_t*, const int64_t*, int, int64_t, int64_t, int, int, int, int,
                      int, int, int, void*, uint32_t);
    int (*solve_multi)(const void*, const void*, const void*, int, const void* const*, const float* const*, void* const*, const int*, int,
                       int64_t, int, int, int, int, int, int, int, void*, uint32_t);
    int (*solve_varlen)(const void*, const void*, const void*, const void*, const void*, void*, const int64_t*, const int64_t*, int, int64_t,
                        int64_t, int, int, int, int, int, int, int, int, void*, uint32_t);
    int (*offsets)(const int64_t*, int, int, int64_t, int64_t*, int64_t*, void*);
    // may be absent
    int (*inv_packed)(const void*, const void*, const void*, void*, const int64_t*, int, int64_t, int, int, int, int, int, int, int, void*, uint32_t);
    int (*solve_packed)(const void*, const void*, const void*, const void*, const void*, void*, const int64_t*, int, int64_t, int, int, int, int, int,
                        int, int, int, void*, uint32_t);
} abi;

int code_of(at::ScalarType t) { return t == at::kFloat ? F32 : t == at::kHalf ? F16 : t == at::kBFloat16 ? BF16 : -1; }

// Reads the arguments of one call in order; ok() is false once one of them was not plain.
class Args {
public:
    Args(PyObject* const* v, Py_ssize_t n, Py_ssize_t expected) : v_(v), ok_(n == expected) {}
    bool ok() const { return ok_; }
    int64_t integer()
    {
        PyObject* const o = next();
        if (!ok_ || !PyLong_Check(o)) return fail();
        const long long x = PyLong_AsLongLong(o);
        if (x == -1 && PyErr_Occurred()) {
            PyErr_Clear();
            return fail();
        }
        return x;
    }
    int small() { return narrow(integer()); }
    // None stands for `otherwise`
    int small_or(int otherwise) { return ok_ && *v_ == Py_None ? (next(), otherwise) : small(); }
    // a contiguous tensor on the device of the call, with `dims` dimensions (any number: -1); none: None may stand for it (undefined tensor)
    at::Tensor tensor(int dims, bool none = false) { return as_tensor(next(), dims, none); }
    at::Tensor as_tensor(PyObject* o, int dims, bool none = false)
    {
        if (!ok_ || (none && o == Py_None)) return {};
        if (!THPVariable_CheckExact(o)) return fail(), at::Tensor();
        at::Tensor t = THPVariable_Unpack(o);
        if ((device_ < 0 ? !t.is_cpu() : !t.is_cuda() || t.get_device() != device_) || t.is_nested() || t.layout() != at::kStrided ||
            !t.is_contiguous() || (dims >= 0 && t.dim() != dims) || code_of(t.scalar_type()) < 0)
            return fail(), at::Tensor();
        return t;
    }
    // an element type of the result: None (fp32) or a torch.dtype
    at::ScalarType dtype(bool& given)
    {
        PyObject* const o = next();
        given = ok_ && o != Py_None;
        if (!given) return at::kFloat;
        if (!THPDtype_Check(o)) return fail(), at::kFloat;
        return reinterpret_cast<THPDtype*>(o)->scalar_type;
    }
    PyObject* next() { return ok_ ? *v_++ : nullptr; }
    int fail() { return ok_ = false, 0; }
    int narrow(int64_t x) { return x < INT32_MIN || x > INT32_MAX ? fail() : (int)x; }
    void device_and_stream()
    {
        device_ = small();
        stream_ = reinterpret_cast<void*>(integer());
    }
    int device() const { return device_; }
    void* stream() const { return stream_; }

private:
    PyObject* const* v_;
    bool ok_;
    int device_ = -1;
    void* stream_ = nullptr;
};

bool chunk_ok(int C) { return C == 16 || C == 32 || C == 64 || C == 128; }

// The result tensor (allocated if none is given) and the bit of its element type in flags.
bool result(at::Tensor& T, at::IntArrayRef shape, at::ScalarType type, bool type_given, const at::Tensor& like, uint32_t& flags)
{
    if (!T.defined())
        T = at::empty(shape, like.options().dtype(type));
    else if (type_given && T.scalar_type() != type)
        return false;
    const int c = code_of(T.scalar_type());
    flags = (flags & ~(uint32_t)(FLAG_OUT_F16 | FLAG_OUT_BF16)) | (c == F16 ? FLAG_OUT_F16 : c == BF16 ? FLAG_OUT_BF16 : 0);
    return c >= 0;
}

const void* ptr(const at::Tensor& t) { return t.defined() && t.numel() ? t.data_ptr() : nullptr; }
void* out(const at::Tensor& t) { return t.numel() ? t.data_ptr() : nullptr; }

// Runs f (allocation and launch) without the interpreter's lock; false, too, for what it throws: out of memory comes again on the Python route.
template <class F> bool unlocked(F f)
{
    bool done = false;
    PyThreadState* const state = PyEval_SaveThread();
    try {
        done = f();
    } catch (...) {
        done = false;
    }
    PyEval_RestoreThread(state);
    return done;
}

PyObject* none() { Py_RETURN_NONE; }

// (device, stream, A, T, method, op_dtype or None for A's own, flags, out_dtype)
PyObject* tri_inv(PyObject*, PyObject* const* v, Py_ssize_t n)
{
    Args a(v, n, 8);
    a.device_and_stream();
    const at::Tensor A = a.tensor(3);
    at::Tensor T = a.tensor(-1, true);
    const int in = A.defined() ? code_of(A.scalar_type()) : -1, method = a.small(), op = a.small_or(in);
    uint32_t flags = (uint32_t)a.small();
    bool given;
    const at::ScalarType type = a.dtype(given);
    if (!a.ok() || !chunk_ok((int)A.size(1)) || A.size(2) != A.size(1)) return none();
    const int64_t n_mat = A.size(0), C = A.size(1);
    if (T.defined() && T.numel() != A.numel()) return none();
    if (!unlocked([&] {
            return result(T, {n_mat, C, C}, type, given, A, flags) &&
                   abi.tri_inv_ex(A.data_ptr(), T.data_ptr(), n_mat, (int)C, in, method, op, a.stream(), flags) == 0;
        }))
        return none();
    return THPVariable_Wrap(T);
}

// (device, stream, K, beta, g, C, T, gate_kind, method, op_dtype, flags, out_dtype)
PyObject* gdn_inv(PyObject*, PyObject* const* v, Py_ssize_t n)
{
    Args a(v, n, 12);
    a.device_and_stream();
    const at::Tensor K = a.tensor(4), beta = a.tensor(-1), g = a.tensor(-1, true);
    const int C = a.small();
    at::Tensor T = a.tensor(-1, true);
    const int gate = a.small(), method = a.small(), op = a.small();
    uint32_t flags = (uint32_t)a.small();
    bool given;
    const at::ScalarType type = a.dtype(given);
    if (!a.ok() || !chunk_ok(C)) return none();
    const int64_t B = K.size(0), len = K.size(1), H = K.size(2), n_mat = B * ((len + C - 1) / C) * H;
    if (a.narrow(B), a.narrow(H), !a.ok()) return none();
    if (!unlocked([&] {
            return result(T, {n_mat, C, C}, type, given, K, flags) &&
                   abi.inv_ex(K.data_ptr(), beta.data_ptr(), g.defined() ? g.data_ptr() : nullptr, T.data_ptr(), (int)B, len, (int)H, (int)K.size(3), C,
                              code_of(K.scalar_type()), gate, method, op, a.stream(), flags) == 0;
        }))
        return none();
    return THPVariable_Wrap(T);
}

// (device, stream, K, beta, g, [X], C, [row_scale] or None, [W] or None, gate_kind, method, flags): a list of results
PyObject* gdn_solve(PyObject*, PyObject* const* v, Py_ssize_t n)
{
    Args a(v, n, 12);
    a.device_and_stream();
    const at::Tensor K = a.tensor(4), beta = a.tensor(-1), g = a.tensor(-1, true);
    PyObject* const xs = a.next();
    const int C = a.small();
    PyObject *const scales = a.next(), *const ws = a.next();
    const int gate = a.small(), method = a.small();
    const uint32_t flags = (uint32_t)a.small();
    const auto list = [](PyObject* o) { return PyList_CheckExact(o) || PyTuple_CheckExact(o); };
    if (!a.ok() || !chunk_ok(C) || !list(xs) || (scales != Py_None && !list(scales)) || (ws != Py_None && !list(ws))) return none();
    const Py_ssize_t k = PySequence_Fast_GET_SIZE(xs);
    if (k < 1 || k > 2 || (scales != Py_None && PySequence_Fast_GET_SIZE(scales) != k) || (ws != Py_None && PySequence_Fast_GET_SIZE(ws) != k)) return none();
    at::Tensor X[2], S[2], W[2];
    const void* xp[2];
    const float* sp[2];
    void* wp[2];
    int dx[2];
    for (Py_ssize_t i = 0; i < k; ++i) {
        X[i] = a.as_tensor(PySequence_Fast_GET_ITEM(xs, i), 4);
        if (scales != Py_None) S[i] = a.as_tensor(PySequence_Fast_GET_ITEM(scales, i), -1, true);
        if (ws != Py_None) W[i] = a.as_tensor(PySequence_Fast_GET_ITEM(ws, i), 4);
        if (!a.ok() || X[i].size(0) != K.size(0) || X[i].size(1) != K.size(1) || X[i].size(2) != K.size(2) ||
            X[i].scalar_type() != X[0].scalar_type() || (W[i].defined() && (W[i].sizes() != X[i].sizes() || W[i].scalar_type() != X[i].scalar_type())))
            return none();
        dx[i] = a.narrow(X[i].size(3));
    }
    if (a.narrow(K.size(0)), a.narrow(K.size(2)), !a.ok()) return none();
    if (!unlocked([&] {
            for (Py_ssize_t i = 0; i < k; ++i) {
                if (!W[i].defined()) W[i] = at::empty(X[i].sizes(), X[i].options());
                xp[i] = ptr(X[i]);
                sp[i] = S[i].defined() ? static_cast<const float*>(S[i].data_ptr()) : nullptr;
                wp[i] = out(W[i]);
            }
            return abi.solve_multi(K.data_ptr(), beta.data_ptr(), g.defined() ? g.data_ptr() : nullptr, (int)k, xp, sp, wp, dx, (int)K.size(0), K.size(1),
                                   (int)K.size(2), (int)K.size(3), C, code_of(K.scalar_type()), gate, method, code_of(X[0].scalar_type()), a.stream(),
                                   flags) == 0;
        }))
        return none();
    if (ws != Py_None) return Py_NewRef(ws);
    PyObject* const r = PyList_New(k);
    for (Py_ssize_t i = 0; r && i < k; ++i) {
        PyObject* const w = THPVariable_Wrap(W[i]);
        if (!w) return Py_DECREF(r), nullptr;
        PyList_SET_ITEM(r, i, w);
    }
    return r;
}

// Lengths of packed sequences from a list or tuple of ints (at most 900, what the offsets kernel takes).
bool lengths(PyObject* o, std::vector<int64_t>& lens)
{
    if (!PyList_CheckExact(o) && !PyTuple_CheckExact(o)) return false;
    const Py_ssize_t n = PySequence_Fast_GET_SIZE(o);
    if (n > 900) return false;
    lens.resize(n);
    for (Py_ssize_t i = 0; i < n; ++i) {
        PyObject* const x = PySequence_Fast_GET_ITEM(o, i);
        if (!PyLong_CheckExact(x)) return false;
        lens[i] = PyLong_AsLongLong(x);
        if (lens[i] == -1 && PyErr_Occurred()) {
            PyErr_Clear();
            return false;
        }
    }
    return true;
}

// Number of chunks of up to 64 sequences, whose lengths may go with the arguments of the kernel that uses them (csrc/chunk_map.hpp): one launch and
// no offsets in memory.  false: more of them, or lengths that do not add up to the tokens there are.
bool with_arguments(const std::vector<int64_t>& lens, int64_t total, int64_t C, int64_t& n_chunk)
{
    if (!abi.inv_packed || lens.empty() || lens.size() > 64) return false;
    int64_t sum = 0;
    n_chunk = 0;
    for (const int64_t n : lens) {
        if (n < 0 || n > total) return false;
        sum += n;
        n_chunk += (n + C - 1) / C;
    }
    return sum == total;
}

// The launches are asynchronous: the offsets live as long as the result.
PyObject* with_offsets(const at::Tensor& result, const at::Tensor& cu)
{
    PyObject* const r = THPVariable_Wrap(result);
    PyObject* const c = r && cu.defined() ? THPVariable_Wrap(cu) : nullptr;
    PyObject* const keep = c ? PyTuple_Pack(1, c) : r && !cu.defined() ? PyTuple_New(0) : nullptr;
    const bool good = keep && PyObject_SetAttrString(r, "_triinv_keepalive", keep) == 0;
    Py_XDECREF(c);
    Py_XDECREF(keep);
    if (good) return r;
    Py_XDECREF(r);
    return nullptr;
}

// (device, stream, K, beta, g, seqlens, C, T, gate_kind, method, op_dtype, flags, out_dtype)
PyObject* gdn_inv_varlen(PyObject*, PyObject* const* v, Py_ssize_t n)
{
    Args a(v, n, 13);
    a.device_and_stream();
    const at::Tensor K = a.tensor(3), beta = a.tensor(-1), g = a.tensor(-1, true);
    PyObject* const seqlens = a.next();
    const int C = a.small();
    at::Tensor T = a.tensor(-1, true), cu;
    const int gate = a.small(), method = a.small(), op = a.small();
    uint32_t flags = (uint32_t)a.small();
    bool given;
    const at::ScalarType type = a.dtype(given);
    std::vector<int64_t> lens;
    if (!a.ok() || !chunk_ok(C) || !lengths(seqlens, lens)) return none();
    const int64_t total = K.size(0), H = K.size(1), ns = (int64_t)lens.size();
    if (a.narrow(H), !a.ok()) return none();
    if (!unlocked([&] {
            int64_t n_chunk = 0;
            if (with_arguments(lens, total, C, n_chunk)) {
                if (!result(T, {n_chunk * H, C, C}, type, given, K, flags)) return false;
                if (abi.inv_packed(K.data_ptr(), beta.data_ptr(), g.defined() ? g.data_ptr() : nullptr, out(T), lens.data(), (int)ns, total, (int)H,
                                   (int)K.size(2), C, code_of(K.scalar_type()), gate, method, op, a.stream(), flags) == 0)
                    return true;
            }
            cu = at::empty({2 * (ns + 1)}, K.options().dtype(at::kLong));
            int64_t* const c = cu.data_ptr<int64_t>();
            if (abi.offsets(lens.data(), (int)ns, C, total, c, &n_chunk, a.stream()) != 0) return false;
            return result(T, {n_chunk * H, C, C}, type, given, K, flags) &&
                   abi.inv_varlen(K.data_ptr(), beta.data_ptr(), g.defined() ? g.data_ptr() : nullptr, out(T), c, c + ns + 1, (int)ns, total, n_chunk, (int)H,
                                  (int)K.size(2), C, code_of(K.scalar_type()), gate, method, op, a.stream(), flags) == 0;
        }))
        return none();
    return with_offsets(T, cu);
}

// (device, stream, K, beta, g, X, seqlens, C, row_scale, W, gate_kind, method, flags)
PyObject* gdn_solve_varlen(PyObject*, PyObject* const* v, Py_ssize_t n)
{
    Args a(v, n, 13);
    a.device_and_stream();
    const at::Tensor K = a.tensor(3), beta = a.tensor(-1), g = a.tensor(-1, true), X = a.tensor(3);
    PyObject* const seqlens = a.next();
    const int C = a.small();
    const at::Tensor scale = a.tensor(-1, true);
    at::Tensor W = a.tensor(3, true), cu;
    const int gate = a.small(), method = a.small();
    const uint32_t flags = (uint32_t)a.small();
    std::vector<int64_t> lens;
    if (!a.ok() || !chunk_ok(C) || X.size(0) != K.size(0) || X.size(1) != K.size(1) ||
        (W.defined() && (W.sizes() != X.sizes() || W.scalar_type() != X.scalar_type())) || !lengths(seqlens, lens))
        return none();
    const int64_t total = K.size(0), H = K.size(1), ns = (int64_t)lens.size();
    if (a.narrow(H), a.narrow(X.size(2)), !a.ok()) return none();
    if (!unlocked([&] {
            int64_t n_chunk = 0;
            if (with_arguments(lens, total, C, n_chunk)) {
                if (!W.defined()) W = at::empty(X.sizes(), X.options());
                if (abi.solve_packed(K.data_ptr(), beta.data_ptr(), g.defined() ? g.data_ptr() : nullptr, ptr(X), scale.defined() ? scale.data_ptr() : nullptr,
                                     out(W), lens.data(), (int)ns, total, (int)H, (int)K.size(2), (int)X.size(2), C, code_of(K.scalar_type()), gate,
                                     method, code_of(X.scalar_type()), a.stream(), flags) == 0)
                    return true;
            }
            cu = at::empty({2 * (ns + 1)}, K.options().dtype(at::kLong));
            int64_t* const c = cu.data_ptr<int64_t>();
            if (abi.offsets(lens.data(), (int)ns, C, total, c, &n_chunk, a.stream()) != 0) return false;
            if (!W.defined()) W = at::empty(X.sizes(), X.options());
            return abi.solve_varlen(K.data_ptr(), beta.data_ptr(), g.defined() ? g.data_ptr() : nullptr, ptr(X), scale.defined() ? scale.data_ptr() : nullptr,
                                    out(W), c, c + ns + 1, (int)ns, total, n_chunk, (int)H, (int)K.size(2), (int)X.size(2), C,
                                    code_of(K.scalar_type()), gate, method, code_of(X.scalar_type()), a.stream(), flags) == 0;
        }))
        return none();
    return with_offsets(W, cu);
}

// connect(addresses): the C-ABI functions in the order of Abi, without or with the last two
PyObject* connect(PyObject*, PyObject* const* v, Py_ssize_t n)
{
    void* p[8] = {};
    if (n != 6 && n != 8) return PyErr_SetString(PyExc_TypeError, "six or eight addresses"), nullptr;
    for (int i = 0; i < n; ++i) {
        p[i] = PyLong_AsVoidPtr(v[i]);
        if (!p[i]) return PyErr_Occurred() ? nullptr : (PyErr_SetString(PyExc_ValueError, "null address"), nullptr);
    }
    abi.tri_inv_ex = reinterpret_cast<decltype(abi.tri_inv_ex)>(p[0]);
    abi.inv_ex = reinterpret_cast<decltype(abi.inv_ex)>(p[1]);
    abi.inv_varlen = reinterpret_cast<decltype(abi.inv_varlen)>(p[2]);
    abi.solve_multi = reinterpret_cast<decltype(abi.solve_multi)>(p[3]);
    abi.solve_varlen = reinterpret_cast<decltype(abi.solve_varlen)>(p[4]);
    abi.offsets = reinterpret_cast<decltype(abi.offsets)>(p[5]);
    abi.inv_packed = reinterpret_cast<decltype(abi.inv_packed)>(p[6]);
    abi.solve_packed = reinterpret_cast<decltype(abi.solve_packed)>(p[7]);
    Py_RETURN_NONE;
}

// f with its exceptions turned into None.
template <PyObject* (*f)(PyObject*, PyObject* const*, Py_ssize_t)> PyObject* guarded(PyObject* self, PyObject* const* v, Py_ssize_t n) noexcept
{
    try {
        return f(self, v, n);
    } catch (...) {
        PyErr_Clear();  // (an exception that came from Python code may have left its error set)
        return none();
    }
}

#define TRIINV_METHOD(f) {#f, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(guarded<f>)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {TRIINV_METHOD(connect), TRIINV_METHOD(tri_inv), TRIINV_METHOD(gdn_inv), TRIINV_METHOD(gdn_solve),
                         TRIINV_METHOD(gdn_inv_varlen), TRIINV_METHOD(gdn_solve_varlen), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_fastcall", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

// BUILT_FOR: the Python and the torch whose headers this was compiled with; the binding compares them with the ones it runs in.
PyMODINIT_FUNC PyInit__fastcall()
{
    PyObject* const m = PyModule_Create(&module);
    if (m && PyModule_AddStringConstant(m, "BUILT_FOR", TRIINV_BUILT_FOR) != 0) return Py_DECREF(m), nullptr;
    return m;
}
