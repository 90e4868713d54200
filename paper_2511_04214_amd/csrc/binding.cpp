// The calls that a layer and an analysis make, without the interpreter's share of them: arguments are read from the tensors here, checked
// as __init__.py checks them, and handed to the C ABI.  With Python and ctypes in between a call cost the host 6 to 9 us, of
// which the launch is 3: a small layer (16 x 256 x 256, two calls and a result tensor) took 15.0 us, the GPU 6.7.
//
// Only what is plainly right is done here: tensors of torch's own type on the GPU with no other dispatch key than that,
// plain integers, the current stream.  Anything else (a subclass, a traced or batched tensor, an argument that does not
// fit, buffers that are to be made) returns None, and the caller goes its way through Python, which accepts or refuses it
// as it always did.  Otherwise a call returns the library's status, 0 or not, or the result tensor.
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <ATen/ops/_foreach_zero.h>
#include <ATen/ops/empty.h>
#include <ATen/ops/zeros.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Dtype.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/brq.h"

namespace {

// The interpreter's lock is not held while one of these lives (an exception gives it back too).
struct Unlocked {
    PyThreadState* const state = PyEval_SaveThread();
    Unlocked() = default;
    Unlocked(const Unlocked&) = delete;
    ~Unlocked() { PyEval_RestoreThread(state); }
};

// The library's entry points, set by bind() when it is loaded.
decltype(&brq_rotate_quantize_fused) f_rotate_quantize;
decltype(&brq_swiglu_rotate_quantize_fused) f_swiglu;
decltype(&brq_matrix_rotate_quantize_fused) f_matrix;
decltype(&brq_mxfp4_gemm) f_gemm;
decltype(&brq_rotate_quantize_gemm_fused) f_decode;
decltype(&brq_block_stats) f_stats;
decltype(&brq_block_stats_summary) f_summary;

// A tensor of torch's own type, on the GPU, that nothing watches or stands in for: beside the dispatch keys that every such
// tensor has (autograd's, autocast's) it has the device's alone.
bool on_gpu(const at::Tensor& t) {
    return t.defined() && t.key_set() - c10::autograd_dispatch_keyset_with_ADInplaceOrView - c10::autocast_dispatch_keyset ==
                              c10::DispatchKeySet(c10::DispatchKey::CUDA);
}
const at::Tensor* plain(PyObject* o) {
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor& t = THPVariable_Unpack(o);
    return on_gpu(t) ? &t : nullptr;
}

const at::Tensor* bytes(PyObject* o) {
    const at::Tensor* t = plain(o);
    return t && t->scalar_type() == at::kByte && t->is_contiguous() ? t : nullptr;
}

bool dtype_of(at::ScalarType s, brq_dtype* d) {
    *d = s == at::kFloat ? BRQ_F32 : BRQ_BF16;
    return s == at::kFloat || s == at::kBFloat16;
}

bool dtype_arg(PyObject* o, at::ScalarType* s, brq_dtype* d) {
    if (!THPDtype_Check(o)) return false;
    *s = reinterpret_cast<THPDtype*>(o)->scalar_type;
    return dtype_of(*s, d);
}

// A matrix with contiguous rows.
struct Rows {
    const at::Tensor* t;
    int64_t M, K, ld;
    brq_dtype dt;
};
bool rows(PyObject* o, Rows* r) {
    r->t = plain(o);
    if (!r->t || r->t->dim() != 2 || !dtype_of(r->t->scalar_type(), &r->dt)) return false;
    r->M = r->t->size(0);
    r->K = r->t->size(1);
    if (r->K > 1 && r->t->stride(1) != 1) return false;
    r->ld = r->M > 1 ? r->t->stride(0) : r->K;
    return true;
}

bool integer(PyObject* o, int64_t* v) {
    if (!PyLong_CheckExact(o)) return false;
    int overflow = 0;
    *v = PyLong_AsLongLongAndOverflow(o, &overflow);
    return overflow == 0;
}

PyObject *s_rowmajor, *s_tiled;
bool layout(PyObject* o, brq_layout* l) {
    if (!PyUnicode_CheckExact(o)) return false;
    const bool rm = o == s_rowmajor || PyUnicode_Compare(o, s_rowmajor) == 0;
    *l = rm ? BRQ_LAYOUT_ROWMAJOR : BRQ_LAYOUT_TILED;
    return rm || o == s_tiled || PyUnicode_Compare(o, s_tiled) == 0;
}

// Bytes of a quantized [rows][K] operand; sizes that are no operand's are left to Python.
bool operand_size(int64_t n, int64_t K, brq_layout l, int64_t* codes, int64_t* scales) {
    if (n < 0 || K <= 0 || K % 32 != 0 || n >= int64_t(1) << 31 || K >= int64_t(1) << 31) return false;
    if (l == BRQ_LAYOUT_TILED) {
        n = (n + 63) / 64 * 64;
        K = (K + 511) / 512 * 512;
    }
    *codes = n * (K / 2);
    *scales = n * (K / 32);
    return true;
}

bool signs_arg(PyObject* o, int64_t K, const int8_t** p) {
    *p = nullptr;
    if (o == Py_None) return true;
    const at::Tensor* t = plain(o);
    if (!t || !t->is_contiguous() || t->scalar_type() != at::kChar || t->numel() != K) return false;
    *p = static_cast<const int8_t*>(t->const_data_ptr());
    return true;
}

// Buffers that a quantizing call fills.
bool buffers(PyObject* c, PyObject* s, int64_t M, int64_t K, brq_layout l, uint8_t** codes, uint8_t** scales) {
    int64_t nc, ns;
    const at::Tensor *tc = bytes(c), *ts = bytes(s);
    if (!tc || !ts || !operand_size(M, K, l, &nc, &ns) || tc->numel() < nc || ts->numel() < ns) return false;
    *codes = static_cast<uint8_t*>(tc->data_ptr());
    *scales = static_cast<uint8_t*>(ts->data_ptr());
    return true;
}

// An operand of a product: codes and scales, `n` rows of K (either may be -1: not given; a row-major operand says).
bool operand(PyObject* c, PyObject* s, brq_layout l, int64_t* n, int64_t* K) {
    const at::Tensor *tc = bytes(c), *ts = bytes(s);
    if (!tc || !ts) return false;
    if (l == BRQ_LAYOUT_ROWMAJOR) {
        if (tc->dim() != 2 || (*n >= 0 && *n != tc->size(0)) || (*K >= 0 && *K != tc->size(1) * 2)) return false;
        *n = tc->size(0);
        *K = tc->size(1) * 2;
        if (ts->dim() != 2 || ts->size(0) != *n || ts->size(1) != *K / 32) return false;
    }
    return true;
}
const uint8_t* data(PyObject* o) { return static_cast<const uint8_t*>(THPVariable_Unpack(o).const_data_ptr()); }
bool operand_fits(PyObject* c, PyObject* s, brq_layout l, int64_t n, int64_t K) {
    int64_t nc, ns;
    return operand_size(n, K, l, &nc, &ns) && THPVariable_Unpack(c).numel() >= nc && THPVariable_Unpack(s).numel() >= ns;
}

// None or a size
bool size_arg(PyObject* o, int64_t* v) {
    *v = -1;
    return o == Py_None || (integer(o, v) && *v >= 0);
}

// The product's result: `out`, or a new tensor on the device of `like`.  The allocator may have to wait for the GPU, and the GPU
// for work that another thread has yet to launch: the lock is not held meanwhile, and addresses are read after it.
bool result(PyObject* out, PyObject* dtype, const at::Tensor& like, int64_t M, int64_t N, at::Tensor* y, brq_dtype* dt, int64_t* ldy) {
    if (out != Py_None) {
        Rows r;
        if (!rows(out, &r) || r.M != M || r.K != N) return false;
        *y = *r.t;
        *dt = r.dt;
        *ldy = r.ld;
        return true;
    }
    at::ScalarType s;
    if (!dtype_arg(dtype, &s, dt)) return false;
    const at::TensorOptions options = at::TensorOptions().dtype(s).device(like.device());
    {
        const Unlocked u;
        *y = at::empty({M, N}, options);
    }
    *ldy = N;
    return on_gpu(*y);
}

void* current_stream() { return c10::hip::getCurrentHIPStream().stream(); }

// Nobody looks at what is done with tensors from outside (a function mode sees every look at a shape).
bool quiet() { return !at::impl::torch_function_mode_enabled(); }

template <class F>
brq_status released(F call) {
    const Unlocked u;
    return call();
}

PyObject* status(brq_status st) { return PyLong_FromLong((long)st); }
PyObject* result_or(brq_status st, PyObject* out, at::Tensor& y) {
    if (st != BRQ_OK) return status(st);
    if (out == Py_None) return THPVariable_Wrap(std::move(y));
    Py_INCREF(out);
    return out;
}

// rotate_quantize(x, B, codes, scales, layout, signs)
PyObject* rotate_quantize(PyObject*, PyObject* const* a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    Rows x;
    int64_t B;
    brq_layout l;
    const int8_t* signs;
    uint8_t *codes, *scales;
    if (n != 6 || !f_rotate_quantize || !quiet() || !rows(a[0], &x) || !integer(a[1], &B) || !layout(a[4], &l) || !buffers(a[2], a[3], x.M, x.K, l, &codes, &scales) ||
        !signs_arg(a[5], x.K, &signs)) Py_RETURN_NONE;
    const void* p = x.t->const_data_ptr();
    void* s = current_stream();
    return status(released([&] { return f_rotate_quantize(p, x.dt, x.M, x.K, x.ld, B, signs, codes, scales, l, s); }));
    END_HANDLE_TH_ERRORS
}

// swiglu_rotate_quantize(gate, up, B, h_dtype, codes, scales, layout, signs)
PyObject* swiglu_rotate_quantize(PyObject*, PyObject* const* a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    Rows g, u;
    int64_t B;
    brq_layout l;
    brq_dtype hd;
    at::ScalarType hs;
    const int8_t* signs;
    uint8_t *codes, *scales;
    if (n != 8 || !f_swiglu || !quiet() || !rows(a[0], &g) || !rows(a[1], &u) || g.M != u.M || g.K != u.K || g.dt != u.dt || !integer(a[2], &B) ||
        !dtype_arg(a[3], &hs, &hd) || !layout(a[6], &l) || !buffers(a[4], a[5], g.M, g.K, l, &codes, &scales) ||
        !signs_arg(a[7], g.K, &signs)) Py_RETURN_NONE;
    const void *pg = g.t->const_data_ptr(), *pu = u.t->const_data_ptr();
    void* s = current_stream();
    return status(released([&] { return f_swiglu(pg, pu, g.dt, g.M, g.K, g.ld, u.ld, hd, B, signs, codes, scales, l, s); }));
    END_HANDLE_TH_ERRORS
}

// matrix_rotate_quantize(x, R, codes, scales, layout)
PyObject* matrix_rotate_quantize(PyObject*, PyObject* const* a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    Rows x;
    brq_layout l;
    uint8_t *codes, *scales;
    const at::Tensor* R = n == 5 && f_matrix && quiet() ? plain(a[1]) : nullptr;
    if (!R || !R->is_contiguous() || R->scalar_type() != at::kFloat || R->dim() < 2 || R->dim() > 3 || R->size(-1) != 32 || R->size(-2) != 32 ||
        !rows(a[0], &x) || !layout(a[4], &l) || !buffers(a[2], a[3], x.M, x.K, l, &codes, &scales)) Py_RETURN_NONE;
    const int64_t nR = R->dim() == 3 ? R->size(0) : 1;
    const void* p = x.t->const_data_ptr();
    const float* r = static_cast<const float*>(R->const_data_ptr());
    void* s = current_stream();
    return status(released([&] { return f_matrix(p, x.dt, x.M, x.K, x.ld, r, nR, codes, scales, l, s); }));
    END_HANDLE_TH_ERRORS
}

// gemm(aq, as, wq, ws, out_dtype, out, a_layout, w_layout, M, N, K)
PyObject* gemm(PyObject*, PyObject* const* a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    brq_layout la, lw;
    int64_t M, N, K, ldy;
    at::Tensor y;
    brq_dtype dt;
    if (n != 11 || !f_gemm || !quiet() || !layout(a[6], &la) || !layout(a[7], &lw) || !size_arg(a[8], &M) || !size_arg(a[9], &N) || !size_arg(a[10], &K) ||
        !operand(a[0], a[1], la, &M, &K) || !operand(a[2], a[3], lw, &N, &K) || M < 0 || N < 0 || K < 0 ||
        !operand_fits(a[0], a[1], la, M, K) || !operand_fits(a[2], a[3], lw, N, K) ||
        !result(a[5], a[4], THPVariable_Unpack(a[0]), M, N, &y, &dt, &ldy)) Py_RETURN_NONE;
    const uint8_t *ac = data(a[0]), *as = data(a[1]), *wc = data(a[2]), *ws = data(a[3]);
    void *p = y.data_ptr(), *s = current_stream();
    return result_or(released([&] { return f_gemm(ac, as, la, wc, ws, lw, M, N, K, p, dt, ldy, s); }), a[5], y);
    END_HANDLE_TH_ERRORS
}

// rotate_quantize_gemm(x, B, wq, ws, N, out_dtype, out, w_layout, signs)
PyObject* rotate_quantize_gemm(PyObject*, PyObject* const* a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    Rows x;
    brq_layout l;
    int64_t B, N, ldy;
    const int8_t* signs;
    at::Tensor y;
    brq_dtype dt;
    if (n != 9 || !f_decode || !quiet() || !rows(a[0], &x) || !integer(a[1], &B) || !bytes(a[2]) || !bytes(a[3]) || !integer(a[4], &N) || !layout(a[7], &l) ||
        !signs_arg(a[8], x.K, &signs) || !operand_fits(a[2], a[3], l, N, x.K) || !result(a[6], a[5], *x.t, x.M, N, &y, &dt, &ldy)) Py_RETURN_NONE;
    const void* p = x.t->const_data_ptr();
    if (signs) signs = reinterpret_cast<const int8_t*>(data(a[8]));
    const uint8_t *wc = data(a[2]), *ws = data(a[3]);
    void *q = y.data_ptr(), *s = current_stream();
    return result_or(released([&] { return f_decode(p, x.dt, x.M, x.K, x.ld, B, signs, wc, ws, l, N, q, dt, ldy, s); }), a[6], y);
    END_HANDLE_TH_ERRORS
}

// ---- the analysis: the two statistics calls and the summary of a comparison of up to 8 M values took 45 us, all of it the
// host; 33 now (six launches, seven new tensors).

// Numbers as float32, as ctypes makes them of float(t): up to `most`.
bool number(PyObject* o, double* v) {
    if (PyFloat_CheckExact(o)) *v = PyFloat_AS_DOUBLE(o);
    else if (PyLong_CheckExact(o)) *v = PyLong_AsDouble(o);
    else return false;
    if (!PyErr_Occurred()) return true;
    PyErr_Clear();
    return false;
}
bool numbers(PyObject* o, float* v, int most, int* n) {
    if (!PyTuple_CheckExact(o) && !PyList_CheckExact(o)) return false;
    const Py_ssize_t len = PySequence_Fast_GET_SIZE(o);
    if (len > most) return false;
    *n = (int)len;
    for (int i = 0; i < *n; ++i) {
        double d;
        if (!number(PySequence_Fast_GET_ITEM(o, i), &d)) return false;
        v[i] = (float)d;
    }
    return true;
}

// An output or input of one type: None (`*t` stays undefined), or contiguous with its sizes.
bool array(PyObject* o, at::ScalarType s, at::IntArrayRef sizes, at::Tensor* t) {
    if (o == Py_None) return true;
    const at::Tensor* p = plain(o);
    if (!p || p->scalar_type() != s || !p->is_contiguous() || p->sizes() != sizes) return false;
    *t = *p;
    return true;
}
bool flat_array(PyObject* o, at::ScalarType s, int64_t n, at::Tensor* t) {
    if (o == Py_None) return true;
    const at::Tensor* p = plain(o);
    if (!p || p->scalar_type() != s || !p->is_contiguous() || p->numel() != n) return false;
    *t = *p;
    return true;
}
template <class T>
T* address(const at::Tensor& t) { return t.defined() ? static_cast<T*>(t.data_ptr()) : nullptr; }
// the caller's own object, or the new tensor, or None
PyObject* handed(PyObject* given, at::Tensor& t) {
    if (given == Py_None && t.defined()) return THPVariable_Wrap(std::move(t));
    Py_INCREF(given);
    return given;
}
PyObject* three(PyObject* a, PyObject* b, PyObject* c) {
    PyObject* r = a && b && c ? PyTuple_Pack(3, a, b, c) : nullptr;
    Py_XDECREF(a);
    Py_XDECREF(b);
    Py_XDECREF(c);
    return r;
}

// block_stats(x, B, thresholds, signs, counts, want_amax, want_sqerr, amax, sqerr)
PyObject* block_stats(PyObject*, PyObject* const* a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    Rows x;
    int64_t B;
    float th[8];
    int nt;
    const int8_t* signs;
    at::Tensor counts, amax, sqerr;
    if (n != 9 || !f_stats || !quiet() || !rows(a[0], &x) || x.M <= 0 || x.K <= 0 || x.K % 32 != 0 || !integer(a[1], &B) || !numbers(a[2], th, 8, &nt) ||
        !signs_arg(a[3], x.K, &signs) || !flat_array(a[4], at::kLong, nt, &counts) || !PyBool_Check(a[5]) || !PyBool_Check(a[6])) Py_RETURN_NONE;
    const int64_t shape[2] = {x.M, x.K / 32};
    if (!array(a[7], at::kFloat, shape, &amax) || !array(a[8], at::kFloat, shape, &sqerr)) Py_RETURN_NONE;
    const at::TensorOptions f32 = at::TensorOptions().dtype(at::kFloat).device(x.t->device());
    {
        const Unlocked u;
        if (!amax.defined() && a[5] == Py_True) amax = at::empty(shape, f32);
        if (!sqerr.defined() && a[6] == Py_True) sqerr = at::empty(shape, f32);
        if (!counts.defined() && nt) counts = at::zeros({nt}, f32.dtype(at::kLong));
    }
    for (const at::Tensor* t : {&amax, &sqerr, &counts})
        if (t->defined() && !on_gpu(*t)) Py_RETURN_NONE;
    const void* p = x.t->const_data_ptr();
    if (signs) signs = reinterpret_cast<const int8_t*>(data(a[3]));
    float *pa = address<float>(amax), *ps = address<float>(sqerr);
    uint64_t* pc = address<uint64_t>(counts);
    void* s = current_stream();
    const brq_status st = released([&] { return f_stats(p, x.dt, x.M, x.K, x.ld, B, signs, th, nt, pa, pc, ps, nullptr, s); });
    return st != BRQ_OK ? status(st) : three(handed(a[7], amax), handed(a[4], counts), handed(a[8], sqerr));
    END_HANDLE_TH_ERRORS
}

// block_stats_summary(amax, sqerr, amax_ref, outlier_threshold, edges, hist, counts, sums)
PyObject* block_stats_summary(PyObject*, PyObject* const* a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    const at::Tensor* amax = n == 8 && f_summary && quiet() ? plain(a[0]) : nullptr;
    if (!amax || amax->scalar_type() != at::kFloat || !amax->is_contiguous() || amax->numel() == 0) Py_RETURN_NONE;
    const int64_t blocks = amax->numel();
    at::Tensor sqerr, ref, hist, counts, sums;
    double outlier;
    float edges[32];
    int ne;
    if (!flat_array(a[1], at::kFloat, blocks, &sqerr) || !flat_array(a[2], at::kFloat, blocks, &ref) || !number(a[3], &outlier) || !numbers(a[4], edges, 32, &ne) ||
        !flat_array(a[5], at::kLong, ne + 1, &hist) || !flat_array(a[6], at::kLong, 4, &counts) || !flat_array(a[7], at::kDouble, 4, &sums)) Py_RETURN_NONE;
    const at::TensorOptions i64 = at::TensorOptions().dtype(at::kLong).device(amax->device());
    {
        const Unlocked u;
        std::vector<at::Tensor> made;                          // each a tensor of its own, cleared by one launch
        if (!hist.defined()) made.push_back(hist = at::empty({ne + 1}, i64));
        if (!counts.defined()) made.push_back(counts = at::empty({4}, i64));
        if (!sums.defined()) made.push_back((sums = at::empty({4}, i64.dtype(at::kDouble))).view(at::kLong));
        if (!made.empty()) at::_foreach_zero_(made);
    }
    for (const at::Tensor* t : {&hist, &counts, &sums})
        if (!on_gpu(*t)) Py_RETURN_NONE;
    const float *pa = static_cast<const float*>(THPVariable_Unpack(a[0]).const_data_ptr()), *pq = address<float>(sqerr), *pr = address<float>(ref);
    uint64_t *ph = address<uint64_t>(hist), *pc = address<uint64_t>(counts);
    double* pd = address<double>(sums);
    void* s = current_stream();
    const brq_status st = released([&] { return f_summary(pa, pq, pr, blocks, (float)outlier, edges, ne, ph, pc, pd, s); });
    return st != BRQ_OK ? status(st) : three(handed(a[5], hist), handed(a[6], counts), handed(a[7], sums));
    END_HANDLE_TH_ERRORS
}

// bind_stats(addresses of brq_block_stats and brq_block_stats_summary)
PyObject* bind_stats(PyObject*, PyObject* const* a, Py_ssize_t n) {
    void* p[2];
    if (n != 2) {
        PyErr_SetString(PyExc_TypeError, "bind_stats takes the addresses of two entry points");
        return nullptr;
    }
    for (int i = 0; i < 2; ++i) {
        p[i] = PyLong_AsVoidPtr(a[i]);
        if (!p[i]) {
            if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "an entry point's address is NULL");
            return nullptr;
        }
    }
    f_stats = reinterpret_cast<decltype(f_stats)>(p[0]);
    f_summary = reinterpret_cast<decltype(f_summary)>(p[1]);
    Py_RETURN_NONE;
}

// bind(addresses of the entry points of a layer, in the order above)
PyObject* bind(PyObject*, PyObject* const* a, Py_ssize_t n) {
    void* p[5];
    if (n != 5) {
        PyErr_SetString(PyExc_TypeError, "bind takes the addresses of five entry points");
        return nullptr;
    }
    for (int i = 0; i < 5; ++i) {
        p[i] = PyLong_AsVoidPtr(a[i]);
        if (!p[i]) {
            if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "an entry point's address is NULL");
            return nullptr;
        }
    }
    f_rotate_quantize = reinterpret_cast<decltype(f_rotate_quantize)>(p[0]);
    f_swiglu = reinterpret_cast<decltype(f_swiglu)>(p[1]);
    f_matrix = reinterpret_cast<decltype(f_matrix)>(p[2]);
    f_gemm = reinterpret_cast<decltype(f_gemm)>(p[3]);
    f_decode = reinterpret_cast<decltype(f_decode)>(p[4]);
    Py_RETURN_NONE;
}

#define BRQ_METHOD(f) {#f, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(f)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {BRQ_METHOD(bind), BRQ_METHOD(rotate_quantize), BRQ_METHOD(swiglu_rotate_quantize), BRQ_METHOD(matrix_rotate_quantize),
                         BRQ_METHOD(gemm), BRQ_METHOD(rotate_quantize_gemm), BRQ_METHOD(bind_stats), BRQ_METHOD(block_stats), BRQ_METHOD(block_stats_summary), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_binding", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__binding() {
    s_rowmajor = PyUnicode_InternFromString("rowmajor");
    s_tiled = PyUnicode_InternFromString("tiled");
    if (!s_rowmajor || !s_tiled) return nullptr;
    PyObject* m = PyModule_Create(&module);
    // The torch whose headers this was built with: tensors are read through them, so no other will do.
    if (m && PyModule_AddStringConstant(m, "TORCH", BRQ_TORCH) != 0) Py_CLEAR(m);
    return m;
}
