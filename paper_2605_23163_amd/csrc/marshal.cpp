// Arguments of the two calls of a denoise step, and of a fork, from tensors to the C structs of fdd.h.
//
// Host code, a CPython module: `attn` and `unmask` check shapes, types and placement as binding.py does and fill the
// struct at the given address.  They return True, or False (and set no exception) for anything that is not the ordinary
// case - a wrong shape, a tensor subclass, an active torch function mode - and binding.py's own checks then accept it or
// raise their errors.  Nothing is kept between calls.  In Python a tensor property costs about 0.1 us, and a call reads
// 40 to 60 of them: 2.3 us for attention, 4.5 us for unmasking, beside 2.5 us per kernel launch.
#include <Python.h>

#include <ATen/PythonTorchFunctionTLS.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/version.h>

#include <climits>

#include "fdd.h"

namespace {

struct NotOrdinary {};

void need(bool ok)
{
    if (!ok) throw NotOrdinary();
}

const at::Tensor& tensor(PyObject* o)
{
    need(THPVariable_CheckExact(o));
    const at::Tensor& t = THPVariable_Unpack(o);
    need(t.defined() && t.layout() == at::kStrided && t.has_storage() && !t.unsafeGetTensorImpl()->has_symbolic_sizes_strides());
    return t;
}

void* pointer(const at::Tensor& t)
{
    need(t.is_cuda() && t.is_contiguous());
    return t.data_ptr();
}

void* pointer_or_null(PyObject* o) { return o == Py_None ? nullptr : pointer(tensor(o)); }

int32_t int32_of(int64_t x)
{
    need(x >= 0 && x <= INT32_MAX);
    return (int32_t)x;
}

int32_t int32_of(PyObject* o)
{
    need(PyLong_CheckExact(o));
    int over = 0;
    const long x = PyLong_AsLongAndOverflow(o, &over);
    need(!over && x >= INT32_MIN && x <= INT32_MAX);
    return (int32_t)x;
}

float float_of(PyObject* o)
{
    need(PyFloat_CheckExact(o) || PyLong_CheckExact(o));
    const double x = PyFloat_AsDouble(o);
    need(!PyErr_Occurred());
    return (float)x;
}

int dtype_code(const at::Tensor& t)
{
    if (t.scalar_type() == at::kBFloat16) return FDD_BF16;
    need(t.scalar_type() == at::kFloat);
    return FDD_F32;
}

// q, prefix_k, prefix_v, block_k, block_v, scaffold_mask, out, prefix_v_packed, ext_k, ext_v, q_positions, E, causal_block,
// splits, scale
void fill_attn(fdd_attn_params* p, PyObject* const* a)
{
    const at::Tensor &q = tensor(a[0]), &pk = tensor(a[1]), &pv = tensor(a[2]), &bk = tensor(a[3]), &bv = tensor(a[4]);
    need(q.dim() == 4 && pk.dim() == 3 && bk.dim() == 4);
    const int64_t N = q.size(0), B = q.size(1), Hkv = bk.size(2), D = q.size(3);
    need(pk.size(1) == Hkv && pk.size(2) == D && pv.sizes() == pk.sizes());
    need(bk.size(0) == N && bk.size(1) == B && bk.size(3) == D && bv.sizes() == bk.sizes());
    const auto type = q.scalar_type();
    need(pk.scalar_type() == type && pv.scalar_type() == type && bk.scalar_type() == type && bv.scalar_type() == type);
    p->N = int32_of(N); p->B = int32_of(B); p->L = int32_of(pk.size(0));
    p->Hq = int32_of(q.size(2)); p->Hkv = int32_of(Hkv); p->D = int32_of(D);
    p->dtype = (decltype(p->dtype))dtype_code(q);
    p->scale = a[14] == Py_None ? 0.f : float_of(a[14]);
    p->q = pointer(q);
    if (p->L > 0) { p->prefix_k = pointer(pk); p->prefix_v = pointer(pv); }
    p->block_k = pointer(bk); p->block_v = pointer(bv);
    p->scaffold_mask = (decltype(p->scaffold_mask))pointer_or_null(a[5]);
    p->out = pointer_or_null(a[6]);
    p->prefix_v_packed = pointer_or_null(a[7]);
    if (a[8] != Py_None) {
        const at::Tensor &ek = tensor(a[8]), &ev = tensor(a[9]);
        need(ek.dim() == 4 && ek.size(0) == N && ek.size(2) == Hkv && ek.size(3) == D && ev.sizes() == ek.sizes());
        need(ek.scalar_type() == type && ev.scalar_type() == type);
        p->ext_k = pointer(ek); p->ext_v = pointer(ev); p->ext_capacity = int32_of(ek.size(1));
    }
    if (a[10] != Py_None) {
        const at::Tensor& qp = tensor(a[10]);
        need(qp.scalar_type() == at::kInt && qp.dim() == 1);
        p->q_positions = (decltype(p->q_positions))pointer(qp);
        p->n_q_positions = int32_of(qp.numel());
    }
    p->E = int32_of(a[11]);
    const int causal = PyObject_IsTrue(a[12]);
    need(causal >= 0);
    p->flags = causal ? FDD_ATTN_CAUSAL_BLOCK : 0;
    p->splits = int32_of(a[13]);
}

// logits, mask, scaffold_mask, tokens, confidences, n_unmasked, committed, tau, refresh
void fill_unmask(fdd_unmask_params* p, PyObject* const* a)
{
    const at::Tensor &x = tensor(a[0]), &mask = tensor(a[1]), &tok = tensor(a[3]);
    need(x.dim() == 3);
    const int64_t N = x.size(0), B = x.size(1);
    auto per_position = [&](const at::Tensor& t, at::ScalarType type) {
        need(t.scalar_type() == type && t.dim() == 2 && t.size(0) == N && t.size(1) == B);
    };
    per_position(mask, at::kByte);
    per_position(tok, at::kInt);
    if (a[2] != Py_None) per_position(tensor(a[2]), at::kByte);
    p->N = int32_of(N); p->B = int32_of(B); p->V = x.size(2);
    p->dtype = (decltype(p->dtype))dtype_code(x);
    p->tau = float_of(a[7]);
    p->logits = pointer(x);
    p->mask = (decltype(p->mask))pointer(mask);
    p->scaffold_mask = (decltype(p->scaffold_mask))pointer_or_null(a[2]);
    p->tokens = (decltype(p->tokens))pointer(tok);
    p->confidences = (decltype(p->confidences))pointer_or_null(a[4]);
    p->n_unmasked = (decltype(p->n_unmasked))pointer_or_null(a[5]);
    p->committed = (decltype(p->committed))pointer_or_null(a[6]);
    if (a[8] != Py_None) {
        need(PyTuple_CheckExact(a[8]) && PyTuple_GET_SIZE(a[8]) == 4);
        auto item = [&](int i) -> const at::Tensor& { return tensor(PyTuple_GET_ITEM(a[8], i)); };
        const at::Tensor &tk = item(0), &tv = item(1), &bk = item(2), &bv = item(3);
        need(tk.dim() == 3 && bk.dim() == 4 && bk.size(0) == N && bk.size(1) == B);
        need(tk.size(1) == bk.size(2) && tk.size(2) == bk.size(3) && tv.sizes() == tk.sizes() && bv.sizes() == bk.sizes());
        p->refresh_table_k = pointer(tk); p->refresh_table_v = pointer(tv);
        p->refresh_block_k = pointer(bk); p->refresh_block_v = pointer(bv);
        p->refresh_T = int32_of(tk.size(0)); p->refresh_Hkv = int32_of(tk.size(1)); p->refresh_D = int32_of(tk.size(2));
        p->refresh_dtype = (decltype(p->refresh_dtype))dtype_code(tk);
    }
}

// address of a zeroed struct, then the arguments
template <typename P, int ARGS, void (*FILL)(P*, PyObject* const*)>
PyObject* call(PyObject*, PyObject* const* args, Py_ssize_t n)
{
    if (n != ARGS + 1) {
        PyErr_SetString(PyExc_TypeError, "wrong number of arguments");
        return nullptr;
    }
    void* p = PyLong_AsVoidPtr(args[0]);
    if (!p) {
        if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "no address");
        return nullptr;
    }
    bool ok = !at::impl::torch_function_mode_enabled();
    if (ok) {
        try {
            FILL(static_cast<P*>(p), args + 1);
        } catch (...) {       // (NotOrdinary, or an exception of torch's own)
            ok = false;
            PyErr_Clear();
        }
    }
    return PyBool_FromLong(ok);
}

// src, N, dst of a fork into a tensor of the caller's: (bytes, address of src, address of dst), or None
PyObject* fork(PyObject*, PyObject* const* args, Py_ssize_t n)
{
    if (n != 3) {
        PyErr_SetString(PyExc_TypeError, "wrong number of arguments");
        return nullptr;
    }
    if (!at::impl::torch_function_mode_enabled()) {
        try {
            const at::Tensor &src = tensor(args[0]), &dst = tensor(args[2]);
            const int64_t N = int32_of(args[1]);
            need(N > 0 && dst.numel() % N == 0 && dst.numel() / N * (int64_t)dst.element_size() == src.numel() * (int64_t)src.element_size());
            void *const from = pointer(src), *const to = pointer(dst);
            return Py_BuildValue("(nKK)", (Py_ssize_t)(src.numel() * src.element_size()), (unsigned long long)reinterpret_cast<uintptr_t>(from),
                                 (unsigned long long)reinterpret_cast<uintptr_t>(to));
        } catch (...) {       // (NotOrdinary, or an exception of torch's own)
            PyErr_Clear();
        }
    }
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"fork", reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(&fork)), METH_FASTCALL, "arguments of fdd_fork_block"},
    {"attn", reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(&call<fdd_attn_params, 15, fill_attn>)), METH_FASTCALL, "fill an fdd_attn_params"},
    {"unmask", reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(&call<fdd_unmask_params, 9, fill_unmask>)), METH_FASTCALL, "fill an fdd_unmask_params"},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal()
{
    PyObject* m = PyModule_Create(&module);
    if (m && (PyModule_AddStringConstant(m, "torch_version", TORCH_VERSION) < 0 ||
              PyModule_AddIntConstant(m, "attn_bytes", sizeof(fdd_attn_params)) < 0 ||
              PyModule_AddIntConstant(m, "unmask_bytes", sizeof(fdd_unmask_params)) < 0)) {
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
