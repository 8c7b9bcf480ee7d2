// CPython binding of the op calls of libpk.so (include/pk.h), with the conversions of pk.py for arguments of the plain kinds: ints,
// torch.Tensor, the names of the enumerations, None.  Given anything else a function returns None before it has done anything,
// and pk.py converts the arguments itself.
//
// The module is not linked against libpk.so: pk.py hands it the addresses of the entry points of the library that it has loaded (bind),
// so that all calls of a process go to one library, wherever a search path or another copy of the package would lead.  `built_for` names
// what it was compiled against (interface, torch, interpreter), and pk.py takes it only where all of that is what it runs with.
//
// What bounds a small call is the host: a reduce-scatter of 256 x 256 x 512 (two launches, 6.14 us on the device) takes 13.0 us of host
// time on an idle device and 12.0 us a call back to back through ctypes, 10.1 and 9.4 through this (medians of three processes).  What
// is left are 0.7 us here and in pk.py and about 4 us a launch (the runtime writes a launch's arguments to device memory and reads them back).
#include <Python.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/pk.h"

#ifndef PK_BUILT_FOR
#define PK_BUILT_FOR ""
#endif

namespace {

// in the order that bind takes
struct {
    decltype(&pk_gemm_rs) gemm_rs;
    decltype(&pk_gemm_rs_cols) gemm_rs_cols;
    decltype(&pk_gemm_ar) gemm_ar;
    decltype(&pk_ag_gemm) ag_gemm;
    decltype(&pk_ag_gemm_static) ag_gemm_static;
    decltype(&pk_ag_gemm_k) ag_gemm_k;
} lib;

bool as_i64(PyObject* o, int64_t* v) {
    if (!PyLong_CheckExact(o)) return false;
    int overflow = 0;
    *v = PyLong_AsLongLongAndOverflow(o, &overflow);
    return overflow == 0;
}
bool as_int(PyObject* o, int* v) {
    int64_t x;
    if (!as_i64(o, &x) || x != (int)x) return false;
    *v = (int)x;
    return true;
}
bool as_u32(PyObject* o, uint32_t* v) {            // as ctypes does: modulo 2^32
    int64_t x;
    if (!as_i64(o, &x)) return false;
    *v = (uint32_t)x;
    return true;
}
bool as_u64(PyObject* o, uint64_t* v) {
    int64_t x;
    if (!as_i64(o, &x) || x < 0) return false;
    *v = (uint64_t)x;
    return true;
}

// an exact torch.Tensor or Parameter (a subclass may have its own idea of data_ptr) that is a contiguous device tensor with storage
bool as_tensor(PyObject* o, void** p, size_t* bytes = nullptr) {
    if (!THPVariable_CheckExact(o)) return false;
    try {
        const at::Tensor& t = THPVariable_Unpack(o);
        if (!t.is_cuda() || !t.is_contiguous() || !t.has_storage()) return false;
        *p = t.data_ptr();
        if (bytes) *bytes = (size_t)t.numel() * t.element_size();
        return true;
    } catch (...) {
        return false;
    }
}
bool as_ptr(PyObject* o, void** p) {
    *p = nullptr;
    if (o == Py_None) return true;
    uint64_t x;
    if (as_u64(o, &x)) {
        *p = (void*)x;
        return true;
    }
    return as_tensor(o, p);
}

struct Name {
    const char* text;
    int value;
};
constexpr Name kTypes[] = {{"bf16", PK_BF16}, {"fp8", PK_FP8_E4M3}};
constexpr Name kPartials[] = {{"f32", PK_PARTIAL_F32}, {"bf16", PK_PARTIAL_BF16}};
constexpr Name kActivations[] = {{"none", PK_ACT_NONE}, {"relu", PK_ACT_RELU}, {"gelu_tanh", PK_ACT_GELU_TANH}, {"silu", PK_ACT_SILU}};
constexpr Name kLayouts[] = {{"kn", PK_B_ROW_MAJOR}, {"nk", PK_B_K_CONTIGUOUS}};
template <size_t N>
bool as_enum(PyObject* o, const Name (&names)[N], int* v) {
    if (!PyUnicode_CheckExact(o)) return as_int(o, v);
    for (const Name& n : names)
        if (PyUnicode_CompareWithASCIIString(o, n.text) == 0) {
            *v = n.value;
            return true;
        }
    return false;
}

bool as_stream(PyObject* o, void** s) {
    uint64_t x;
    if (o == Py_None) {
        try {
            *s = (void*)c10::hip::getCurrentHIPStream().stream();
            return true;
        } catch (...) {
            return false;
        }
    }
    if (as_u64(o, &x)) {
        *s = (void*)x;
        return true;
    }
    PyObject* h = PyObject_GetAttrString(o, "cuda_stream");
    if (!h) {
        PyErr_Clear();
        return false;
    }
    const bool ok = as_u64(h, &x);
    Py_DECREF(h);
    if (ok) *s = (void*)x;
    return ok;
}

// what all calls begin with: P, rank, M, N, K, dtype, A, B, scale_a, scale_b
struct Problem {
    int P, rank, dt;
    int64_t M, N, K;
    void *A, *B, *sa, *sb;
    bool read(PyObject* const* a) {
        return as_int(a[0], &P) && as_int(a[1], &rank) && as_i64(a[2], &M) && as_i64(a[3], &N) && as_i64(a[4], &K) &&
               as_enum(a[5], kTypes, &dt) && as_ptr(a[6], &A) && as_ptr(a[7], &B) && as_ptr(a[8], &sa) && as_ptr(a[9], &sb);
    }
};

// `call` runs without the interpreter's lock, as under ctypes
template <typename F>
PyObject* run(F call) {
    pk_status st;
    Py_BEGIN_ALLOW_THREADS
    st = call();
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(st);
}

// arguments as those of the functions of the same names in pk.py
PyObject* gemm_rs_of(PyObject* const* a, Py_ssize_t n, bool cols) {
    Problem p;
    void *part, *outg, *fin, *fout, *out, *status, *stream, *ws = nullptr;
    uint32_t epoch, phases;
    int comm_cus, pdt, layout = 0;
    uint64_t timeout;
    size_t ws_bytes = 0;
    if (!lib.gemm_rs || n != (cols ? 22 : 24) || !p.read(a) || !as_ptr(a[10], &part) || !as_ptr(a[11], &outg) || !as_ptr(a[12], &fin) ||
        !as_ptr(a[13], &fout) || !as_u32(a[14], &epoch) || !as_ptr(a[15], &out) || !as_u32(a[16], &phases) || !as_ptr(a[17], &status) ||
        !as_u64(a[18], &timeout) || !as_int(a[20], &comm_cus) || !as_enum(a[21], kPartials, &pdt))
        Py_RETURN_NONE;
    if (!cols && ((a[22] != Py_None && !as_tensor(a[22], &ws, &ws_bytes)) || !as_enum(a[23], kLayouts, &layout) || (layout & ~1)))
        Py_RETURN_NONE;
    if (!as_stream(a[19], &stream)) Py_RETURN_NONE;
    if (cols)
        return run([&] {
            return lib.gemm_rs_cols(p.P, p.rank, p.M, p.N, p.K, (pk_dtype)p.dt, p.A, p.B, (float*)p.sa, (float*)p.sb, part, outg, (uint32_t*)fin,
                                   (uint32_t*)fout, epoch, out, phases, comm_cus, pdt, (uint32_t*)status, timeout, stream);
        });
    return run([&] {
        return lib.gemm_rs(p.P, p.rank, p.M, p.N, p.K, (pk_dtype)p.dt, p.A, p.B, (float*)p.sa, (float*)p.sb, part, outg, (uint32_t*)fin,
                          (uint32_t*)fout, epoch, out, phases, comm_cus, pdt, layout, ws, ws_bytes, (uint32_t*)status, timeout, stream);
    });
}
PyObject* gemm_rs(PyObject*, PyObject* const* a, Py_ssize_t n) { return gemm_rs_of(a, n, false); }
PyObject* gemm_rs_cols(PyObject*, PyObject* const* a, Py_ssize_t n) { return gemm_rs_of(a, n, true); }

PyObject* gemm_ar(PyObject*, PyObject* const* a, Py_ssize_t n) {
    Problem p;
    void *part, *outg, *fin, *fout, *full, *bcast, *arin, *arout, *status, *stream;
    uint32_t epoch, phases;
    int comm_cus, pdt;
    uint64_t timeout;
    if (!lib.gemm_ar || n != 25 || !p.read(a) || !as_ptr(a[10], &part) || !as_ptr(a[11], &outg) || !as_ptr(a[12], &fin) || !as_ptr(a[13], &fout) ||
        !as_ptr(a[14], &full) || !as_ptr(a[15], &bcast) || !as_ptr(a[16], &arin) || !as_ptr(a[17], &arout) || !as_u32(a[18], &epoch) ||
        !as_u32(a[19], &phases) || !as_ptr(a[20], &status) || !as_u64(a[21], &timeout) || !as_int(a[23], &comm_cus) ||
        !as_enum(a[24], kPartials, &pdt) || !as_stream(a[22], &stream))
        Py_RETURN_NONE;
    return run([&] {
        return lib.gemm_ar(p.P, p.rank, p.M, p.N, p.K, (pk_dtype)p.dt, p.A, p.B, (float*)p.sa, (float*)p.sb, part, outg, (uint32_t*)fin,
                          (uint32_t*)fout, full, bcast, (uint32_t*)arin, (uint32_t*)arout, epoch, phases, comm_cus, pdt, (uint32_t*)status,
                          timeout, stream);
    });
}

enum Gather { ROWS, ROWS_STATIC, K_CHUNKS };
PyObject* ag_gemm_of(PyObject* const* a, Py_ssize_t n, Gather kind) {
    Problem p;
    void *flags, *C, *status, *stream, *ws = nullptr;
    uint32_t epoch;
    int comm_cus, act, layout = 0;
    uint64_t timeout;
    size_t ws_bytes = 0;
    if (!lib.ag_gemm || n != (kind == ROWS ? 20 : 18) || !p.read(a) || !as_ptr(a[10], &flags) || !as_u32(a[11], &epoch) || !as_ptr(a[12], &C) ||
        !as_ptr(a[13], &status) || !as_u64(a[14], &timeout) || !as_int(a[16], &comm_cus) || !as_enum(a[17], kActivations, &act))
        Py_RETURN_NONE;
    if (kind == ROWS && ((a[18] != Py_None && !as_tensor(a[18], &ws, &ws_bytes)) || !as_enum(a[19], kLayouts, &layout) || (layout & ~1)))
        Py_RETURN_NONE;
    if (!as_stream(a[15], &stream)) Py_RETURN_NONE;
    if (kind == ROWS)
        return run([&] {
            return lib.ag_gemm(p.P, p.rank, p.M, p.N, p.K, (pk_dtype)p.dt, p.A, p.B, (float*)p.sa, (float*)p.sb, (uint32_t*)flags, epoch, C,
                              comm_cus, act, layout, ws, ws_bytes, (uint32_t*)status, timeout, stream);
        });
    return run([&] {
        return (kind == K_CHUNKS ? lib.ag_gemm_k : lib.ag_gemm_static)(p.P, p.rank, p.M, p.N, p.K, (pk_dtype)p.dt, p.A, p.B, (float*)p.sa,
                                                                     (float*)p.sb, (uint32_t*)flags, epoch, C, comm_cus, act,
                                                                     (uint32_t*)status, timeout, stream);
    });
}
PyObject* ag_gemm(PyObject*, PyObject* const* a, Py_ssize_t n) { return ag_gemm_of(a, n, ROWS); }
PyObject* ag_gemm_static(PyObject*, PyObject* const* a, Py_ssize_t n) { return ag_gemm_of(a, n, ROWS_STATIC); }
PyObject* ag_gemm_k(PyObject*, PyObject* const* a, Py_ssize_t n) { return ag_gemm_of(a, n, K_CHUNKS); }

PyObject* bind(PyObject*, PyObject* const* a, Py_ssize_t n) {
    void* f[6];
    bool ok = n == 6;
    for (int i = 0; ok && i < 6; ++i) ok = as_ptr(a[i], &f[i]) && f[i];
    if (!ok) {
        PyErr_SetString(PyExc_TypeError, "bind takes the addresses of the six entry points");
        return nullptr;
    }
    lib = {(decltype(lib.gemm_rs))f[0], (decltype(lib.gemm_rs_cols))f[1], (decltype(lib.gemm_ar))f[2], (decltype(lib.ag_gemm))f[3],
           (decltype(lib.ag_gemm_static))f[4], (decltype(lib.ag_gemm_k))f[5]};
    Py_RETURN_NONE;
}

#define PK_METHOD(f) {"pk_" #f, (PyCFunction)(void (*)(void))f, METH_FASTCALL, nullptr}
PyMethodDef kMethods[] = {PK_METHOD(gemm_rs), PK_METHOD(gemm_rs_cols), PK_METHOD(gemm_ar), PK_METHOD(ag_gemm),
                          PK_METHOD(ag_gemm_static), PK_METHOD(ag_gemm_k),
                          {"bind", (PyCFunction)(void (*)(void))bind, METH_FASTCALL, nullptr}, {nullptr, nullptr, 0, nullptr}};
PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_pk_call", nullptr, -1, kMethods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__pk_call(void) {
    PyObject* m = PyModule_Create(&kModule);
    if (m && PyModule_AddStringConstant(m, "built_for", PK_BUILT_FOR) < 0) {
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
