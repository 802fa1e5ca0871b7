// The calls of a decode step, marshalled natively.  A step of a small batch is some ten microseconds of GPU work a call, and
// through ctypes a call was five microseconds of Python before its launch: the struct of the cache built field by field, an
// address and a check per tensor, twelve arguments converted.  Arguments are the binding's own objects; what is passed on
// is what ctypes passed on (see binding.py), and the return value is the library's.  The library is not linked: its entry points are
// handed over by address (bind), since the binding may load another build of it.
#include <torch/csrc/autograd/python_variable.h>

#include <exception>

#include "../../include/lserve.h"

namespace {

decltype(&lserve_append_kv) append_kv;
decltype(&lserve_select_pages) select_pages;
decltype(&lserve_sparse_decode) sparse_decode;

struct PythonError {};  // the interpreter's error is set

const at::Tensor* tensor_or_null(PyObject* o) {
    if (o == Py_None) return nullptr;
    if (!THPVariable_Check(o)) {
        PyErr_Format(PyExc_TypeError, "lserve binding takes tensors, not %.100s", Py_TYPE(o)->tp_name);
        throw PythonError();
    }
    return &THPVariable_Unpack(o);
}

template <class P = void> P* address(const at::Tensor* t) {
    if (!t) return nullptr;
    if (!t->is_contiguous()) {
        PyErr_SetString(PyExc_ValueError, "lserve binding takes contiguous tensors");
        throw PythonError();
    }
    return static_cast<P*>(t->data_ptr());
}
template <class P = void> P* address(PyObject* o) { return address<P>(tensor_or_null(o)); }

// (the low bits, as ctypes takes them)
unsigned long long number(PyObject* o) {
    const unsigned long long x = PyLong_AsUnsignedLongLongMask(o);
    if (x == (unsigned long long)-1 && PyErr_Occurred()) throw PythonError();
    return x;
}
int32_t number32(PyObject* o) { return (int32_t)number(o); }

// A Python object's attribute, held while in use.
struct Attribute {
    PyObject* o;
    Attribute(PyObject* of, PyObject* name) : o(PyObject_GetAttr(of, name)) {
        if (!o) throw PythonError();
    }
    ~Attribute() { Py_DECREF(o); }
    Attribute(const Attribute&) = delete;
};

enum { kKPool, kVPool, kStats, kPageTable, kSeqLens, kPoolHeads, kKStream, kVStream, kRingTable, kBits, kNames };
PyObject* names[kNames];

// binding.PagedKV as lserve_paged_kv.  (The tensors stay alive: the caller holds the object.)
lserve_paged_kv paged(PyObject* kv) {
    const Attribute k(kv, names[kKPool]), v(kv, names[kVPool]), st(kv, names[kStats]), table(kv, names[kPageTable]), lens(kv, names[kSeqLens]),
        heads(kv, names[kPoolHeads]), ks(kv, names[kKStream]), vs(kv, names[kVStream]), ring(kv, names[kRingTable]), bits(kv, names[kBits]);
    const at::Tensor *kt = tensor_or_null(k.o), *vt = tensor_or_null(v.o), *stt = tensor_or_null(st.o), *tt = tensor_or_null(table.o),
                     *kst = tensor_or_null(ks.o);
    const at::Tensor* sized = stt ? stt : vt ? vt : kt;
    if (!tt) {
        PyErr_SetString(PyExc_TypeError, "PagedKV.page_table is None");
        throw PythonError();
    }
    lserve_paged_kv p = {};
    p.k_pool = address(kt);
    p.v_pool = address(vt);
    p.stats = address(stt);
    p.page_table = address<int32_t>(tt);
    p.seq_lens = address<int32_t>(lens.o);
    p.batch = (int32_t)tt->size(0);
    p.max_pages_per_seq = (int32_t)tt->size(1);
    p.num_pages = sized ? (int32_t)sized->size(0) : 0;
    p.pool_heads = number32(heads.o);
    p.k_pool_stream = address(kst);
    p.v_pool_stream = address(vs.o);
    p.ring_table = address<int32_t>(ring.o);
    p.num_pages_stream = kst ? (int32_t)kst->size(0) : 0;
    p.kv_bits = number32(bits.o);
    return p;
}

const lserve_attn_desc* description(PyObject* o) { return reinterpret_cast<const lserve_attn_desc*>((uintptr_t)number(o)); }
void* stream_handle(PyObject* o) { return reinterpret_cast<void*>((uintptr_t)number(o)); }

// Other threads may run while the library is at work (a launch waits where the queue is full).
struct WithoutLock {
    PyThreadState* state = PyEval_SaveThread();
    ~WithoutLock() { PyEval_RestoreThread(state); }
};

template <class F> PyObject* call(Py_ssize_t given, Py_ssize_t wanted, F f) {
    if (given != wanted) return PyErr_Format(PyExc_TypeError, "%zd arguments instead of %zd", given, wanted);
    try {
        const int rc = f();
        return PyLong_FromLong(rc);
    } catch (const PythonError&) {
        return nullptr;
    } catch (const std::exception& e) {
        return PyErr_Format(PyExc_RuntimeError, "%s", e.what());
    }
}

PyObject* py_append(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return call(n, 8, [&] {
        const lserve_attn_desc* desc = description(a[0]);
        const lserve_paged_kv kv = paged(a[1]);
        const void *k = address(a[2]), *v = address(a[3]);
        const int32_t *cu = address<int32_t>(a[4]), *start = address<int32_t>(a[5]), longest = number32(a[6]);
        void* stream = stream_handle(a[7]);
        const WithoutLock w;
        return append_kv(desc, &kv, k, v, cu, start, longest, stream);
    });
}

PyObject* py_select(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return call(n, 11, [&] {
        const lserve_attn_desc* desc = description(a[0]);
        const lserve_paged_kv kv = paged(a[1]);
        const at::Tensor* ws = tensor_or_null(a[9]);
        const void* q = address(a[2]);
        const int32_t budget = number32(a[3]), *valid = address<int32_t>(a[4]);
        int32_t *pages = address<int32_t>(a[5]), *count = address<int32_t>(a[6]), *len = address<int32_t>(a[7]);
        float* scores = address<float>(a[8]);
        void *workspace = address(ws), *stream = stream_handle(a[10]);
        const size_t bytes = ws ? ws->nbytes() : 0;
        const WithoutLock w;
        return select_pages(desc, &kv, q, budget, valid, pages, count, len, scores, workspace, bytes, stream);
    });
}

PyObject* py_decode(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return call(n, 10, [&] {
        const lserve_attn_desc* desc = description(a[0]);
        const lserve_paged_kv kv = paged(a[1]);
        const at::Tensor *sel = tensor_or_null(a[3]), *ws = tensor_or_null(a[8]);
        const void* q = address(a[2]);
        const int32_t *pages = address<int32_t>(sel), *count = address<int32_t>(a[4]), *len = address<int32_t>(a[5]);
        const int32_t stride = sel ? (int32_t)sel->size(-1) : 0;
        void *out = address(a[6]), *workspace = address(ws), *stream = stream_handle(a[9]);
        float* lse = address<float>(a[7]);
        const size_t bytes = ws ? ws->nbytes() : 0;
        const WithoutLock w;
        return sparse_decode(desc, &kv, q, pages, count, len, stride, out, lse, workspace, bytes, stream);
    });
}

PyObject* py_bind(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return call(n, 3, [&] {
        append_kv = reinterpret_cast<decltype(append_kv)>((uintptr_t)number(a[0]));
        select_pages = reinterpret_cast<decltype(select_pages)>((uintptr_t)number(a[1]));
        sparse_decode = reinterpret_cast<decltype(sparse_decode)>((uintptr_t)number(a[2]));
        return 0;
    });
}

#define LSERVE_FASTCALL(f) reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(f)), METH_FASTCALL
PyMethodDef methods[] = {
    {"bind", LSERVE_FASTCALL(py_bind), "addresses of lserve_append_kv, lserve_select_pages, lserve_sparse_decode"},
    {"append", LSERVE_FASTCALL(py_append), "desc address, kv, k_new, v_new, cu_new, start_pos, max_new_per_seq, stream"},
    {"select", LSERVE_FASTCALL(py_select),
     "desc address, kv, q, budget_tokens, stats_valid_len, sel_pages, sel_count, sel_seq_len, scores_out, workspace, stream"},
    {"decode", LSERVE_FASTCALL(py_decode), "desc address, kv, q, sel_pages, sel_count, sel_seq_len, out, lse_out, workspace, stream"},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_calls", "native marshalling of the decode step's calls", -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__calls() {
    constexpr const char* spelled[kNames] = {"k_pool", "v_pool", "stats", "page_table", "seq_lens",
                                             "pool_heads", "k_pool_stream", "v_pool_stream", "ring_table", "kv_bits"};
    for (int i = 0; i < kNames; ++i)
        if (!(names[i] = PyUnicode_InternFromString(spelled[i]))) return nullptr;
    PyObject* m = PyModule_Create(&module);
    if (m && PyModule_AddStringConstant(m, "torch_version", LSERVE_TORCH) < 0) {
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
