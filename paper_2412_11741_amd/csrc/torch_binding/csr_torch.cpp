// Native half of the Python binding: reads PyTorch tensors and calls the C ABI of include/csr.h.
//
// The calls of this path take 10 to 30 us on the GPU in their small shapes; marshalled in Python (tensor attributes,
// ctypes structures and arguments, two torch.empty) they took about 25 us of host time each, so a decoding step was
// bound by the interpreter.  Here the same marshalling is 1 to 2 us plus the launches.
//
// Three functions: encode, decode, reconstruct.  Each takes the arguments of the Python function of the same name by
// position and returns its result - or None for anything out of the ordinary (an argument that is not a GPU tensor, a
// shape or type that does not fit, a status other than CSR_OK): the Python function then goes through its own checks,
// which name the mistake.  Nothing has been launched in that case, except where the runtime itself reports an error.
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <ATen/ops/empty.h>
#include <c10/hip/HIPCachingAllocator.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Dtype.h>
#include <torch/csrc/autograd/python_variable.h>

#include "csr.h"

namespace {

using at::ScalarType;
using at::Tensor;

// entry points of libcsr_hip.so, handed over by address when the Python side has loaded it
struct Api {
    size_t (*encode_workspace)(const csr_encode_desc *);
    decltype(&csr_encode) encode;
    size_t (*decode_workspace)(const csr_decode_desc *);
    decltype(&csr_decode_attn) decode;
    decltype(&csr_reconstruct) reconstruct;
} api;

constexpr size_t kInvalid = (size_t)-1;

// A GPU tensor, or nullptr
const Tensor *gpu_tensor(PyObject *o)
{
    if (!THPVariable_Check(o)) return nullptr;
    const Tensor &t = THPVariable_Unpack(o);
    return t.is_cuda() && t.layout() == at::kStrided ? &t : nullptr;
}

int dtype_code(ScalarType t) { return t == ScalarType::Half ? CSR_F16 : t == ScalarType::Float ? CSR_F32 : -1; }
int itype_code(ScalarType t) { return t == ScalarType::Short ? CSR_I16 : t == ScalarType::Int ? CSR_I32 : -1; }

bool dtype_arg(PyObject *o, ScalarType otherwise, ScalarType *t)
{
    if (o == Py_None) { *t = otherwise; return true; }
    if (!THPDtype_Check(o)) return false;
    *t = reinterpret_cast<THPDtype *>(o)->scalar_type;
    return true;
}

bool int_arg(PyObject *o, int64_t *v)
{
    if (!PyLong_CheckExact(o)) return false;
    *v = PyLong_AsLongLong(o);
    if (*v == -1 && PyErr_Occurred()) { PyErr_Clear(); return false; }
    return true;
}

bool float_arg(PyObject *o, float *v)
{
    if (PyFloat_CheckExact(o)) { *v = (float)PyFloat_AS_DOUBLE(o); return true; }
    int64_t i;
    if (!int_arg(o, &i)) return false;
    *v = (float)i;
    return true;
}

// What Tensor::contiguous(idx) of one block means here: the dimensions after the first are dense
bool blocks_dense(const Tensor &t)
{
    int64_t want = 1;
    for (int64_t k = t.dim() - 1; k >= 1; --k) {
        if (t.size(k) != 1 && t.stride(k) != want) return false;
        want *= t.size(k);
    }
    return true;
}

// Device scratch for one call: the caller's tensor, or a block of PyTorch's allocator that returns to its pool when
// the call is enqueued (later users of the pool on this stream come behind it).
struct Workspace {
    c10::DataPtr own;
    void *ptr = nullptr;
    size_t bytes = 0;
    Workspace(const Tensor *given, size_t need)
    {
        if (given) {
            ptr = given->data_ptr();
            bytes = (size_t)given->numel() * given->element_size();
        } else if (need) {
            own = c10::hip::HIPCachingAllocator::get()->allocate(need);
            ptr = own.get();
            bytes = need;
        }
    }
};

void *stream() { return c10::hip::getCurrentHIPStream().stream(); }

Tensor fresh(at::IntArrayRef shape, ScalarType t, const Tensor &like)
{
    return at::empty(shape, at::TensorOptions().dtype(t).device(like.device()));
}

// The interpreter's lock given up while memory is taken and kernels are launched: other threads' Python runs meanwhile.
struct Unlocked {
    PyThreadState *state = PyEval_SaveThread();
    ~Unlocked() { PyEval_RestoreThread(state); }
};

// The caller's output, or the one that was made for the call; nullptr (with Python's error set) if it cannot be wrapped
PyObject *output(PyObject *given, Tensor &made)
{
    if (given == Py_None) return THPVariable_Wrap(std::move(made));
    Py_INCREF(given);
    return given;
}

#define CSR_PUNT() Py_RETURN_NONE

// (X, D, s, coef_dtype, idx_dtype, algo, idx, coef, workspace, res_norm2, gram, closed_loop) -> (idx, coef)
PyObject *encode(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    if (n != 12) CSR_PUNT();
    const Tensor *X = gpu_tensor(a[0]), *D = gpu_tensor(a[1]);
    int64_t s, algo;
    if (!X || !D || !int_arg(a[2], &s) || !int_arg(a[5], &algo)) CSR_PUNT();
    const bool chunked = D->dim() == 4;
    if (X->dim() != 3 || (D->dim() != 3 && !chunked) || !D->is_contiguous() || dtype_code(X->scalar_type()) < 0 ||
        dtype_code(D->scalar_type()) < 0)
        CSR_PUNT();
    const int64_t H = X->size(0), T = X->size(1), d = X->size(2), HD = D->size(0), sn = chunked ? D->size(1) : 1;
    if (HD < 1 || H % HD != 0 || D->size(-1) * sn != d || X->stride(2) != 1 || H > INT32_MAX || s < 1 || s > 32) CSR_PUNT();
    ScalarType ct, it;
    if (!dtype_arg(a[3], X->scalar_type(), &ct) ||
        !dtype_arg(a[4], X->scalar_type() == ScalarType::Half ? ScalarType::Short : ScalarType::Int, &it) ||
        dtype_code(ct) < 0 || itype_code(it) < 0)
        CSR_PUNT();
    const int64_t shape4[4] = {H, T, chunked ? sn : s, s};
    const at::IntArrayRef shape(shape4, chunked ? 4 : 3);
    const Tensor *given[2] = {nullptr, nullptr};
    for (int k = 0; k < 2; ++k) {
        if (a[6 + k] == Py_None) continue;
        given[k] = gpu_tensor(a[6 + k]);
        if (!given[k] || given[k]->sizes() != shape || given[k]->scalar_type() != (k == 0 ? it : ct) || !blocks_dense(*given[k])) CSR_PUNT();
    }
    csr_encode_desc e{};
    e.H = (int32_t)H; e.T = T; e.d = (int32_t)d; e.N = (int32_t)D->size(-2); e.s = (int32_t)s; e.s_n = (int32_t)sn;
    e.x_dtype = dtype_code(X->scalar_type()); e.dict_dtype = dtype_code(D->scalar_type());
    e.coef_dtype = dtype_code(ct); e.idx_dtype = itype_code(it);
    e.x_stride_h = H > 1 && T > 0 ? X->stride(0) : 0;
    e.x_stride_t = T > 1 ? X->stride(1) : 0;
    e.dict_count = HD != H ? (int32_t)HD : 0;
    e.algo = (int32_t)algo;
    const int closed = PyObject_IsTrue(a[11]);
    if (closed < 0) { PyErr_Clear(); CSR_PUNT(); }
    e.flags = closed ? CSR_FLAG_CLOSED_LOOP : 0u;
    if (a[9] != Py_None) {
        const Tensor *r = gpu_tensor(a[9]);
        const int64_t want[3] = {H, T, sn};
        if (!r || r->sizes() != at::IntArrayRef(want, chunked ? 3 : 2) || r->scalar_type() != ScalarType::Float || !r->is_contiguous()) CSR_PUNT();
        e.res_norm2 = static_cast<float *>(r->data_ptr());
    }
    if (a[10] != Py_None) {
        const Tensor *g = gpu_tensor(a[10]);
        if (!g || g->dim() != D->dim() || g->scalar_type() != ScalarType::Half || !g->is_contiguous() || g->size(-1) != D->size(-2)) CSR_PUNT();
        for (int64_t k = 0; k + 1 < D->dim(); ++k)
            if (g->size(k) != D->size(k)) CSR_PUNT();
        e.gram = g->data_ptr();
    }
    if (H > 1 && T > 0) {
        const int64_t block = T * sn * s;
        const int64_t si = given[0] ? given[0]->stride(0) : block, sc = given[1] ? given[1]->stride(0) : block;
        if (si != sc) CSR_PUNT();
        e.code_stride_h = si;
    }
    const Tensor *workspace = nullptr;
    if (a[8] != Py_None && !(workspace = gpu_tensor(a[8]))) CSR_PUNT();
    Tensor made[2];   // owned here until the call has been made: an allocation that throws takes the other one along
    csr_status st;
    {
        Unlocked unlocked;
        const size_t need = api.encode_workspace(&e);
        void *out[2];
        st = need == kInvalid ? CSR_ERR_WORKSPACE : CSR_OK;
        const Workspace ws(workspace, st == CSR_OK ? need : 0);
        for (int k = 0; k < 2 && st == CSR_OK; ++k) {
            if (!given[k]) made[k] = fresh(shape, k == 0 ? it : ct, *X);
            out[k] = given[k] ? given[k]->data_ptr() : made[k].data_ptr();
        }
        if (st == CSR_OK) st = api.encode(&e, X->data_ptr(), D->data_ptr(), out[0], out[1], ws.ptr, ws.bytes, stream());
    }
    if (st != CSR_OK) CSR_PUNT();
    PyObject *pair = PyTuple_New(2);
    for (int k = 0; k < 2 && pair; ++k) {
        PyObject *o = output(a[6 + k], made[k]);
        if (o) PyTuple_SET_ITEM(pair, k, o);
        else Py_CLEAR(pair);
    }
    return pair;
}

// (q, DK, idxK, coefK, DV, idxV, coefV, scale, seq_lens, out, out_dtype, workspace, rope_base, rope_layout, rope_pos0) -> out
PyObject *decode(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    if (n != 15) CSR_PUNT();
    const Tensor *t[7];
    for (int k = 0; k < 7; ++k) {
        t[k] = gpu_tensor(a[k]);
        if (!t[k] || !t[k]->is_contiguous()) CSR_PUNT();
    }
    const Tensor &q = *t[0], &DK = *t[1], &iK = *t[2], &cK = *t[3], &DV = *t[4], &iV = *t[5], &cV = *t[6];
    if (q.dim() != 3 || (iK.dim() != 4 && iK.dim() != 5) || (iV.dim() != 4 && iV.dim() != 5)) CSR_PUNT();
    if (DK.scalar_type() != DV.scalar_type() || cK.scalar_type() != cV.scalar_type() || iK.scalar_type() != iV.scalar_type() ||
        dtype_code(q.scalar_type()) < 0 || dtype_code(DK.scalar_type()) < 0 || dtype_code(cK.scalar_type()) < 0 ||
        itype_code(iK.scalar_type()) < 0 || cK.sizes() != iK.sizes() || cV.sizes() != iV.sizes())
        CSR_PUNT();
    const int64_t B = q.size(0), Hq = q.size(1), d = q.size(2), Hkv = DK.size(0);
    if (DK.dim() < 3 || DV.dim() < 3 || B > INT32_MAX || Hq > INT32_MAX) CSR_PUNT();
    const int64_t N = DK.size(-2), T = iK.size(2);
    for (int side = 0; side < 2; ++side) {   // dictionaries [Hkv, N, d] or [Hkv, sn, N, d / sn] as their codes say
        const Tensor &Dict = side ? DV : DK, &idx = side ? iV : iK;
        const bool ch = idx.dim() == 5;
        const int64_t sn = ch ? idx.size(3) : 1;
        if (sn < 1 || Dict.dim() != (ch ? 4 : 3) || Dict.size(0) != Hkv || (ch && Dict.size(1) != sn) || Dict.size(-2) != N ||
            Dict.size(-1) != d / sn)
            CSR_PUNT();
        for (int k = 0; k < 3; ++k)
            if (idx.size(k) != iK.size(k)) CSR_PUNT();
    }
    if (iK.size(0) != B || iK.size(1) != Hkv) CSR_PUNT();
    ScalarType ot;
    int64_t layout, pos0;
    csr_decode_desc e{};
    if (!float_arg(a[7], &e.scale) || !dtype_arg(a[10], q.scalar_type(), &ot) || dtype_code(ot) < 0 || !float_arg(a[12], &e.rope_base) ||
        !int_arg(a[13], &layout) || !int_arg(a[14], &pos0))
        CSR_PUNT();
    e.B = (int32_t)B; e.Hq = (int32_t)Hq; e.Hkv = (int32_t)Hkv; e.T = T; e.d = (int32_t)d; e.N = (int32_t)N;
    e.sK = (int32_t)iK.size(-1); e.sV = (int32_t)iV.size(-1);
    e.snK = iK.dim() == 5 ? (int32_t)iK.size(3) : 1; e.snV = iV.dim() == 5 ? (int32_t)iV.size(3) : 1;
    e.q_dtype = dtype_code(q.scalar_type()); e.dict_dtype = dtype_code(DK.scalar_type());
    e.coef_dtype = dtype_code(cK.scalar_type()); e.idx_dtype = itype_code(iK.scalar_type()); e.out_dtype = dtype_code(ot);
    e.rope_layout = (int32_t)layout; e.rope_pos0 = pos0;
    const int32_t *lens = nullptr;
    if (a[8] != Py_None) {
        const Tensor *l = gpu_tensor(a[8]);
        if (!l || l->scalar_type() != ScalarType::Int || l->numel() != B) CSR_PUNT();
        lens = static_cast<const int32_t *>(l->data_ptr());
    }
    const Tensor *given = nullptr;
    if (a[9] != Py_None && !(given = gpu_tensor(a[9]))) CSR_PUNT();
    const Tensor *workspace = nullptr;
    if (a[11] != Py_None && !(workspace = gpu_tensor(a[11]))) CSR_PUNT();
    Tensor made;
    csr_status st = CSR_ERR_WORKSPACE;
    {
        Unlocked unlocked;
        const size_t need = api.decode_workspace(&e);
        if (need != kInvalid) {
            const Workspace ws(workspace, need);
            if (!given) made = fresh(q.sizes(), ot, q);
            st = api.decode(&e, q.data_ptr(), DK.data_ptr(), iK.data_ptr(), cK.data_ptr(), DV.data_ptr(), iV.data_ptr(), cV.data_ptr(),
                            lens, given ? given->data_ptr() : made.data_ptr(), ws.ptr, ws.bytes, stream());
        }
    }
    if (st != CSR_OK) CSR_PUNT();
    return output(a[9], made);
}

// (D, idx, coef, out, out_dtype) -> out
PyObject *reconstruct(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    if (n != 5) CSR_PUNT();
    const Tensor *D = gpu_tensor(a[0]), *idx = gpu_tensor(a[1]), *coef = gpu_tensor(a[2]);
    if (!D || !idx || !coef) CSR_PUNT();
    const bool chunked = D->dim() == 4;
    if ((D->dim() != 3 && !chunked) || idx->dim() != D->dim() || coef->sizes() != idx->sizes() || D->size(0) < 1 ||
        idx->size(0) % D->size(0) != 0 || (chunked && idx->size(2) != D->size(1)) || !D->is_contiguous() ||
        dtype_code(D->scalar_type()) < 0 || dtype_code(coef->scalar_type()) < 0 || itype_code(idx->scalar_type()) < 0)
        CSR_PUNT();
    const int64_t H = idx->size(0), T = idx->size(1), sn = chunked ? D->size(1) : 1, d = D->size(-1) * sn;
    ScalarType ot;
    if (!dtype_arg(a[4], D->scalar_type(), &ot) || dtype_code(ot) < 0 || H > INT32_MAX || d > INT32_MAX) CSR_PUNT();
    if (H > 0 && T > 0 && (!blocks_dense(*idx) || !blocks_dense(*coef) || (H > 1 && idx->stride(0) != coef->stride(0)))) CSR_PUNT();
    const int64_t shape3[3] = {H, T, d};
    const at::IntArrayRef shape(shape3, 3);
    const Tensor *given = nullptr;
    if (a[3] != Py_None) {
        given = gpu_tensor(a[3]);
        if (!given || given->sizes() != shape || given->scalar_type() != ot || given->stride(2) != 1) CSR_PUNT();
    }
    Tensor made;
    if (!given) {
        Unlocked unlocked;
        made = fresh(shape, ot, *D);
    }
    const Tensor &o = given ? *given : made;
    csr_reconstruct_desc e{};
    e.H = (int32_t)H; e.T = T; e.d = (int32_t)d; e.N = (int32_t)D->size(-2); e.s = (int32_t)idx->size(-1); e.s_n = (int32_t)sn;
    e.dict_dtype = dtype_code(D->scalar_type()); e.coef_dtype = dtype_code(coef->scalar_type());
    e.idx_dtype = itype_code(idx->scalar_type()); e.out_dtype = dtype_code(ot);
    e.dict_count = D->size(0) != H ? (int32_t)D->size(0) : 0;
    e.code_stride_h = H > 1 && T > 0 ? idx->stride(0) : 0;
    e.out_stride_h = H > 1 && T > 0 ? o.stride(0) : 0;
    e.out_stride_t = T > 1 ? o.stride(1) : 0;
    csr_status st;
    {
        Unlocked unlocked;
        st = api.reconstruct(&e, D->data_ptr(), idx->data_ptr(), coef->data_ptr(), o.data_ptr(), stream());
    }
    if (st != CSR_OK) CSR_PUNT();
    return output(a[3], made);
}

// C++ exceptions of PyTorch (an allocation that fails) must not cross into the interpreter: the Python path meets the
// same condition and reports it in PyTorch's own way.
template <PyObject *(*F)(PyObject *, PyObject *const *, Py_ssize_t)>
PyObject *guarded(PyObject *self, PyObject *const *a, Py_ssize_t n)
{
    try {
        return F(self, a, n);
    } catch (...) {
        CSR_PUNT();
    }
}

// bind(encode_workspace_bytes, encode, decode_workspace_bytes, decode_attn, reconstruct): addresses of the entry points
PyObject *bind(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    void *p[5];
    if (n != 5) {
        PyErr_SetString(PyExc_TypeError, "bind takes five addresses");
        return nullptr;
    }
    for (int k = 0; k < 5; ++k) {
        p[k] = PyLong_AsVoidPtr(a[k]);
        if (!p[k]) {
            if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "bind: null address");
            return nullptr;
        }
    }
    api.encode_workspace = reinterpret_cast<decltype(api.encode_workspace)>(p[0]);
    api.encode = reinterpret_cast<decltype(api.encode)>(p[1]);
    api.decode_workspace = reinterpret_cast<decltype(api.decode_workspace)>(p[2]);
    api.decode = reinterpret_cast<decltype(api.decode)>(p[3]);
    api.reconstruct = reinterpret_cast<decltype(api.reconstruct)>(p[4]);
    Py_RETURN_NONE;
}

#define CSR_FN(f) reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(f))
PyMethodDef methods[] = {{"bind", CSR_FN(bind), METH_FASTCALL, nullptr},
                         {"encode", CSR_FN(guarded<encode>), METH_FASTCALL, nullptr},
                         {"decode", CSR_FN(guarded<decode>), METH_FASTCALL, nullptr},
                         {"reconstruct", CSR_FN(guarded<reconstruct>), METH_FASTCALL, nullptr},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_csr_torch", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__csr_torch(void) { return PyModule_Create(&module); }
