// The binding's ordinary calls in native code: operands are plain contiguous device tensors, outputs and workspace come from
// torch's allocator, the stream is the current one.  What binding.py does for such a call, in the same order, without the
// interpreter: a small call is bound by the host (fp32 256^3 with row sums, two launches and three
// allocations, 15.4 us through the interpreter and 7.7 to 9.2 so, calls of one launch and one allocation 8.5 and 5.1).  Everything else -- a caller's outputs, workspace or stream, operands that are to be refused, subclasses and
// wrapped tensors, numbers that are no plain ints -- is answered with None, and binding.py goes its general way.
//
// Functions return a tensor or a tuple of them, the library's status (an int) where that is not zero, or None.
#include <Python.h>

#include <array>
#include <cstdint>

#include <ATen/ATen.h>
#include <c10/hip/HIPFunctions.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/pgk.h"

namespace {

// the library that binding.py has loaded, by the addresses of its entry points
struct Library {
    decltype(&pgk_gemm_fused) gemm[2];                            // [b_transposed]
    decltype(&pgk_gemm_splitk) gemm_splitk[2];
    decltype(&pgk_gemm_fused_workspace_bytes) gemm_bytes;
    decltype(&pgk_gemm_splitk_workspace_bytes) gemm_splitk_bytes;
    decltype(&pgk_reduce_max) reduce_max;
    decltype(&pgk_reduce_max_workspace_bytes) reduce_max_bytes;
    decltype(&pgk_conv1d) conv1d;
    decltype(&pgk_conv1d_workspace_least_bytes) conv1d_bytes;
    decltype(&pgk_conv1d_out_len) conv1d_out_len;
};
Library lib{};

// Answers of the size queries, pure functions of the sizes: a program calls with the same few again and again.  Bounded, one table per
// thread, forgotten when another library is bound.
struct Answers {
    struct Entry { std::array<int64_t, 10> key; size_t value; };
    std::array<Entry, 256> entries{};
    uint64_t of = 0;
};
uint64_t bound = 0;               // counts the libraries (changed under the interpreter's lock, as all here that is not released)

template <typename F>
size_t answer(const std::array<int64_t, 10>& key, F&& ask)
{
    static thread_local Answers table;
    if (table.of != bound) { table = Answers{}; table.of = bound; }
    uint64_t h = 1469598103934665603ull;
    for (int64_t k : key) h = (h ^ (uint64_t)k) * 1099511628211ull;
    Answers::Entry& e = table.entries[(h >> 32) % table.entries.size()];
    if (e.key != key) e = {key, ask()};                           // (no call has the key of zeros that entries start with)
    return e.value;
}

// a plain device tensor that the kernels can read or write, or nullptr
const at::Tensor* plain(PyObject* o)
{
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor& t = THPVariable_Unpack(o);
    if (!t.defined() || t.layout() != at::kStrided || !t.is_cuda() || !t.unsafeGetTensorImpl()->has_storage() || !t.is_contiguous()) return nullptr;
    return &t;
}

bool plain_int(PyObject* o, int64_t* v)
{
    if (!PyLong_CheckExact(o)) return false;
    int overflow = 0;
    *v = PyLong_AsLongLongAndOverflow(o, &overflow);
    return overflow == 0;
}

// the element type of both, or -1
int type_of(const at::Tensor& a, const at::Tensor& b)
{
    if (a.scalar_type() != b.scalar_type()) return -1;
    return a.scalar_type() == at::kFloat ? PGK_DTYPE_F32 : a.scalar_type() == at::kBFloat16 ? PGK_DTYPE_BF16 : -1;
}

bool bias_of(PyObject* o, int64_t n, const at::Tensor& operand, const float** bias)
{
    *bias = nullptr;
    if (o == Py_None) return true;
    const at::Tensor* t = plain(o);
    if (!t || t->scalar_type() != at::kFloat || t->numel() != n || t->device() != operand.device()) return false;
    *bias = static_cast<const float*>(t->data_ptr());
    return true;
}

at::Tensor empty(at::IntArrayRef sizes, const at::Tensor& like, at::ScalarType type)
{
    return at::empty(sizes, at::TensorOptions().dtype(type).device(like.device()));
}

struct Space { at::Tensor tensor; void* at = nullptr; size_t bytes = 0; };
Space workspace(size_t bytes, const at::Tensor& like)
{
    if (!bytes) return {};
    Space s{empty({(int64_t)bytes}, like, at::kByte), nullptr, bytes};
    s.at = s.tensor.data_ptr();
    return s;
}

void* stream() { return c10::hip::getCurrentHIPStream(c10::hip::current_device()).stream(); }

// the library's calls enqueue and may wait for room in a queue: without the interpreter's lock
template <typename F>
int call(F&& f)
{
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = f();
    Py_END_ALLOW_THREADS
    return rc;
}

PyObject* pair(const at::Tensor& a, const at::Tensor& b)
{
    PyObject* first = THPVariable_Wrap(a);
    PyObject* second = b.defined() ? THPVariable_Wrap(b) : Py_NewRef(Py_None);
    PyObject* out = first && second ? PyTuple_Pack(2, first, second) : nullptr;
    Py_XDECREF(first);
    Py_XDECREF(second);
    return out;
}

// gemm(A, B, bias, act, rowsum, b_transposed, splits): splits None for the fused call
PyObject* gemm(PyObject*, PyObject* const* args, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    int64_t act, splits = 0;
    const at::Tensor *A, *B;
    if (n != 7 || !(A = plain(args[0])) || !(B = plain(args[1])) || !plain_int(args[3], &act) || !PyBool_Check(args[4]) || !PyBool_Check(args[5]))
        Py_RETURN_NONE;
    const bool rowsum = args[4] == Py_True, bt = args[5] == Py_True, split = args[6] != Py_None;
    if (split && !plain_int(args[6], &splits)) Py_RETURN_NONE;
    if (act != (int)act || splits != (int)splits) Py_RETURN_NONE;
    const int64_t da = A->dim(), db = B->dim();
    const int dtype = type_of(*A, *B);
    if ((da != 2 && da != 3) || (db != 2 && db != 3) || dtype < 0 || A->device() != B->device()) Py_RETURN_NONE;
    const int64_t batch = da == 3 ? A->size(0) : 1, M = A->size(da - 2), K = A->size(da - 1);
    const int64_t N = B->size(bt ? db - 2 : db - 1);
    if ((db == 3 ? B->size(0) : 1) != batch || B->size(bt ? db - 1 : db - 2) != K) Py_RETURN_NONE;
    const float* bias;
    if (!bias_of(args[2], N, *A, &bias)) Py_RETURN_NONE;

    const void *a = A->data_ptr(), *b = B->data_ptr();
    const int flags = (rowsum ? PGK_WS_ROWSUM : 0) | (bt ? PGK_WS_B_TRANSPOSED : 0) |
                      (((reinterpret_cast<uintptr_t>(a) | reinterpret_cast<uintptr_t>(b)) & 15u) ? PGK_WS_UNALIGNED : 0);
    size_t need = answer({1 + split, M, N, K, batch, dtype, flags, splits, 0, 0}, [&] {
        return split ? lib.gemm_splitk_bytes(M, N, K, batch, dtype, (int)splits, flags) : lib.gemm_bytes(M, N, K, batch, dtype, flags);
    });
    if (split && need < 16) need = 16;
    const Space ws = workspace(need, *A);
    const at::Tensor C = empty({batch, M, N}, *A, A->scalar_type());
    at::Tensor rs;
    if (rowsum) rs = empty({batch, M}, *A, at::kFloat);
    void* const c = C.data_ptr();
    float* const r = rowsum ? static_cast<float*>(rs.data_ptr()) : nullptr;
    void* const st = stream();
    const auto fused = lib.gemm[bt];
    const auto in_slices = lib.gemm_splitk[bt];
    const int rc = call([&] {
        return split ? in_slices(a, b, bias, c, r, M, N, K, batch, (int)act, dtype, (int)splits, ws.at, ws.bytes, st)
                     : fused(a, b, bias, c, r, M, N, K, batch, (int)act, dtype, ws.at, ws.bytes, st);
    });
    return rc ? PyLong_FromLong(rc) : pair(C, rs);
    END_HANDLE_TH_ERRORS
}

// reduce_max(X, dim, want_idx)
PyObject* reduce_max(PyObject*, PyObject* const* args, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    int64_t dim;
    const at::Tensor* X;
    if (n != 3 || !(X = plain(args[0])) || !plain_int(args[1], &dim) || !PyBool_Check(args[2])) Py_RETURN_NONE;
    const int dtype = type_of(*X, *X);
    const int64_t dims = X->dim();
    if (dtype < 0 || dims == 0) Py_RETURN_NONE;
    dim = (dim % dims + dims) % dims;
    int64_t outer = 1, inner = 1;
    c10::SmallVector<int64_t, 8> shape;
    for (int64_t d = 0; d < dims; ++d) {
        if (d == dim) continue;
        (d < dim ? outer : inner) *= X->size(d);
        shape.push_back(X->size(d));
    }
    const int64_t red = X->size(dim);
    const size_t need = answer({3, outer, red, inner, dtype, 0, 0, 0, 0, 0}, [&] { return lib.reduce_max_bytes(outer, red, inner, dtype); });
    const Space ws = workspace(need, *X);
    const at::Tensor vals = empty(shape, *X, X->scalar_type());
    at::Tensor idx;
    if (args[2] == Py_True) idx = empty(shape, *X, at::kInt);
    const void* const x = X->data_ptr();
    void* const v = vals.data_ptr();
    int32_t* const i = idx.defined() ? static_cast<int32_t*>(idx.data_ptr()) : nullptr;
    void* const st = stream();
    const auto entry = lib.reduce_max;
    const int rc = call([&] { return entry(x, v, i, outer, red, inner, dtype, ws.at, ws.bytes, st); });
    return rc ? PyLong_FromLong(rc) : pair(vals, idx);
    END_HANDLE_TH_ERRORS
}

// conv1d(x, w, bias, act, stride, pad, dilation)
PyObject* conv1d(PyObject*, PyObject* const* args, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    int64_t act, stride, pad, dilation;
    const at::Tensor *x, *w;
    if (n != 7 || !(x = plain(args[0])) || !(w = plain(args[1])) || !plain_int(args[3], &act) || !plain_int(args[4], &stride) ||
        !plain_int(args[5], &pad) || !plain_int(args[6], &dilation) || act != (int)act) Py_RETURN_NONE;
    const int dtype = type_of(*x, *w);
    if (x->dim() != 3 || w->dim() != 3 || x->size(1) != w->size(1) || dtype < 0 || x->device() != w->device()) Py_RETURN_NONE;
    const int64_t B = x->size(0), Cin = x->size(1), L = x->size(2), Cout = w->size(0), Kw = w->size(2);
    const float* bias;
    if (!bias_of(args[2], Cout, *x, &bias)) Py_RETURN_NONE;
    const int64_t Lout = lib.conv1d_out_len(L, Kw, stride, pad, dilation);
    if (Lout <= 0) Py_RETURN_NONE;
    const size_t need = answer({4, B, Cin, L, Cout, Kw, stride, pad, dilation, dtype},
                               [&] { return lib.conv1d_bytes(B, Cin, L, Cout, Kw, stride, pad, dilation, dtype); });
    const Space ws = workspace(need, *x);
    const at::Tensor y = empty({B, Cout, Lout}, *x, x->scalar_type());
    const void *px = x->data_ptr(), *pw = w->data_ptr();
    void* const py = y.data_ptr();
    void* const st = stream();
    const auto entry = lib.conv1d;
    const int rc = call([&] { return entry(px, pw, bias, py, B, Cin, L, Cout, Kw, stride, pad, dilation, (int)act, dtype, ws.at, ws.bytes, st); });
    return rc ? PyLong_FromLong(rc) : THPVariable_Wrap(y);
    END_HANDLE_TH_ERRORS
}

// bind(addresses): of the entry points of Library, in its order
PyObject* bind(PyObject*, PyObject* const* args, Py_ssize_t n)
{
    void* at[11];
    static_assert(sizeof(Library) == sizeof(at), "one address per entry point");
    if (n != 11) return PyErr_Format(PyExc_TypeError, "bind takes 11 addresses, not %zd", n);
    for (int k = 0; k < 11; ++k) {
        at[k] = PyLong_AsVoidPtr(args[k]);
        if (!at[k]) return PyErr_Occurred() ? nullptr : PyErr_Format(PyExc_ValueError, "entry point %d has no address", k);
    }
    __builtin_memcpy(&lib, at, sizeof(at));
    ++bound;
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"bind", reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(bind)), METH_FASTCALL, nullptr},
    {"gemm", reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(gemm)), METH_FASTCALL, nullptr},
    {"reduce_max", reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(reduce_max)), METH_FASTCALL, nullptr},
    {"conv1d", reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(conv1d)), METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_pgk_torch", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__pgk_torch() { return PyModule_Create(&module); }
