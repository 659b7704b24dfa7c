// The host side of one product call of the Python binding: arguments out of their Python objects, the C entry point, views of the
// workspace.  The same steps through ctypes and torch's Python functions took 10.7 us of the 17.3 us in which a 256 x 256 x 256 product
// was enqueued (five views 5.3, the index list 2.3, structures and arguments 3; its two launches are 6), and its kernels take 7 us.
#include <Python.h>

#include <ATen/ops/as_strided.h>
#include <ATen/ops/empty.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <string.h>

#include "../../include/adahop.h"

namespace {

decltype(&adahop_gemm) gemm = nullptr;
decltype(&adahop_gemm_ex) gemm_ex = nullptr;
PyObject *operand_type = nullptr;
PyObject *n_tensor, *n_outer, *n_K, *n_ld, *n_k_contig;

// What is read here is the plain form of a call: int objects, tensors that are exactly torch's, the binding's own operands.  Everything else that
// ctypes takes (an object with __index__, as numpy's integers, a c_int, _as_parameter_, an operand with a c() of its own, other objects with a
// data_ptr()) is left to it, and so is what it refuses: these functions return false without an exception to be kept.

struct object_t { // one reference
    PyObject *p;
    explicit object_t(PyObject *o) : p(o) {}
    ~object_t() { Py_XDECREF(p); }
    object_t(const object_t &) = delete;
    object_t &operator=(const object_t &) = delete;
    explicit operator bool() const { return p != nullptr; }
};

bool integer(PyObject *o, int64_t *out)
{
    if (!o || !PyLong_Check(o)) return false;
    *out = (int64_t)PyLong_AsUnsignedLongLongMask(o); // the low bits of larger ones, as ctypes
    return !PyErr_Occurred();
}

bool attribute(PyObject *o, PyObject *name, int64_t *out)
{
    const object_t r(PyObject_GetAttr(o, name));
    return integer(r.p, out);
}

// None is a null pointer.
bool pointer(PyObject *o, void **out)
{
    *out = nullptr;
    if (!o || (o != Py_None && !THPVariable_CheckExact(o))) return false;
    if (o != Py_None) *out = THPVariable_Unpack(o).data_ptr();
    return true;
}

bool operand(PyObject *o, adahop_operand_t *x)
{
    if (reinterpret_cast<PyObject *>(Py_TYPE(o)) != operand_type) return false;
    const object_t t(PyObject_GetAttr(o, n_tensor));
    void *data;
    int64_t outer, K, ld;
    if (t.p == Py_None || !pointer(t.p, &data) || !attribute(o, n_outer, &outer) || !attribute(o, n_K, &K) || !attribute(o, n_ld, &ld)) return false;
    const object_t kc(PyObject_GetAttr(o, n_k_contig));
    if (!kc || !PyBool_Check(kc.p)) return false;
    *x = {static_cast<uint16_t *>(data), outer, K, ld, kc.p == Py_True};
    return true;
}

template <typename T> bool structure(PyObject *o, T *out)
{
    Py_buffer b;
    if (PyObject_GetBuffer(o, &b, PyBUF_SIMPLE) != 0) return false;
    const bool fits = b.len == (Py_ssize_t)sizeof *out;
    if (fits) memcpy(out, b.buf, sizeof *out);
    PyBuffer_Release(&b);
    return fits;
}

// product(A, B, Cout, strategy, iht_block, k, idx, workspace, stream, opts, layout)
//   idx: the caller's list, or None: a new one of k entries on A's device (none: no memory); opts: adahop_gemm_opts_t or None.
// -> (status, idx, a_codes, a_scales, b_codes, b_scales, mask): the list, and views of the workspace, which are None
// where the call failed; or None, nothing having been done, where the call is not in the plain form above.
PyObject *product(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    if (n != 11) {
        PyErr_SetString(PyExc_TypeError, "product takes 11 arguments");
        return nullptr;
    }
    PyObject *const pa = args[0], *const pb = args[1], *const pc = args[2], *const pidx = args[6], *const pws = args[7];
    const bool given = pidx != Py_None;
    adahop_operand_t A, B;
    adahop_gemm_opts_t opts;
    adahop_ws_layout_t L;
    int64_t strategy, block, k, stream = 0;
    void *C, *ws, *idx;
    if (!operand(pa, &A) || !operand(pb, &B) || pc == Py_None || !pointer(pc, &C) || !integer(args[3], &strategy) || !integer(args[4], &block) ||
        !integer(args[5], &k) || k != (int)k || !pointer(pidx, &idx) || pws == Py_None || !pointer(pws, &ws) || (args[8] != Py_None && !integer(args[8], &stream)) ||
        (args[9] != Py_None && !structure(args[9], &opts)) || !structure(args[10], &L) || THPVariable_Unpack(pc).dim() == 0 ||
        THPVariable_Unpack(pws).dim() != 1 || THPVariable_Unpack(pws).stride(0) != 1) {
        PyErr_Clear();
        Py_RETURN_NONE;
    }
    const int64_t ldc = THPVariable_Unpack(pc).stride(0), ws_bytes = THPVariable_Unpack(pws).numel();
    at::Tensor list;
    if (!given) {
        const object_t t(PyObject_GetAttr(pa, n_tensor));
        if (!t) return nullptr;
        list = at::empty({(int)k > 0 ? (int)k : 0}, at::TensorOptions().dtype(at::kInt).device(THPVariable_Unpack(t.p).device()));
        idx = list.data_ptr();
    }
    int status;
    Py_BEGIN_ALLOW_THREADS;
    const adahop_strategy_t s = static_cast<adahop_strategy_t>((int)strategy);
    status = args[9] == Py_None
                 ? gemm(&A, &B, static_cast<float *>(C), ldc, s, (int)block, (int)k, static_cast<int32_t *>(idx), given, ws,
                        (size_t)ws_bytes, reinterpret_cast<void *>(stream))
                 : gemm_ex(&A, &B, C, ldc, s, (int)block, (int)k, static_cast<int32_t *>(idx), given, &opts, ws, (size_t)ws_bytes,
                           reinterpret_cast<void *>(stream));
    Py_END_ALLOW_THREADS;
    const object_t result(PyTuple_New(7));
    if (!result) return nullptr;
    auto set = [&](int i, PyObject *o) {
        if (o) PyTuple_SET_ITEM(result.p, i, o);
        return o != nullptr;
    };
    Py_XINCREF(given ? pidx : nullptr);
    if (!set(0, PyLong_FromLong(status)) || !set(1, given ? pidx : THPVariable_Wrap(std::move(list)))) return nullptr;
    if (status == ADAHOP_OK) {
        const at::Tensor &w = THPVariable_Unpack(pws);
        const int64_t at0 = w.storage_offset(), M = A.outer, N = B.outer, K = A.K;
        auto matrix = [&](int i, size_t off, int64_t rows, int64_t cols) {
            return set(i, THPVariable_Wrap(at::as_strided(w, {rows, cols}, {cols, 1}, at0 + (int64_t)off)));
        };
        const int which = (int)strategy;
        const int64_t dim = which == ADAHOP_IHT_OE_ROW ? M : which == ADAHOP_IHT_OE_COL ? N : which == ADAHOP_IHT_OE_K ? K : 0;
        if (!matrix(2, L.a_codes, M, K / 2) || !matrix(3, L.a_scales, M, K / 32) || !matrix(4, L.b_codes, N, K / 2) ||
            !matrix(5, L.b_scales, N, K / 32) || !set(6, THPVariable_Wrap(at::as_strided(w, {dim}, {1}, at0 + (int64_t)L.mask))))
            return nullptr;
    } else {
        for (int i = 2; i < 7; ++i) {
            Py_INCREF(Py_None);
            set(i, Py_None);
        }
    }
    Py_INCREF(result.p);
    return result.p;
    END_HANDLE_TH_ERRORS
}

// init(address of adahop_gemm, address of adahop_gemm_ex, the operand's type)
PyObject *init(PyObject *, PyObject *args)
{
    unsigned long long g, ge;
    PyObject *type;
    if (!PyArg_ParseTuple(args, "KKO", &g, &ge, &type)) return nullptr;
    Py_INCREF(type); // (for the life of the process)
    gemm = reinterpret_cast<decltype(gemm)>(g);
    gemm_ex = reinterpret_cast<decltype(gemm_ex)>(ge);
    operand_type = type;
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {{"init", init, METH_VARARGS, nullptr},
                         {"product", reinterpret_cast<PyCFunction>(reinterpret_cast<void *>(product)), METH_FASTCALL, nullptr},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_call", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

} // namespace

PyMODINIT_FUNC PyInit__call(void)
{
    struct {
        PyObject **name;
        const char *text;
    } const names[] = {{&n_tensor, "tensor"}, {&n_outer, "outer"}, {&n_K, "K"}, {&n_ld, "ld"}, {&n_k_contig, "k_contig"}};
    for (const auto &x : names)
        if (!(*x.name = PyUnicode_InternFromString(x.text))) return nullptr;
    return PyModule_Create(&module);
}
