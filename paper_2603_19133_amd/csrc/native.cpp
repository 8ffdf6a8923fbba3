// The part of the Python binding that runs on every call, in native code: a call's tensors become device pointers, its
// outputs and scratch are allocated, and the C ABI (include/picospec.h) is entered, without the interpreter in between.
// A round trip through ctypes and torch's Python allocation costs two to three microseconds per tensor allocated and up to
// six per call, more than the kernels of a small call take.  Plain CPython functions; tensors are torch's own.
#include <Python.h>

#include <ATen/ATen.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/csrc/utils/object_ptr.h>

#include <stdexcept>

#include "../../include/picospec.h"

namespace {

struct BadArgument : std::runtime_error { using std::runtime_error::runtime_error; };

// The arguments of one call, converted one by one; an argument of the wrong kind ends the call with a TypeError.
struct Args {
    PyObject* const* a;
    Py_ssize_t n, at = 0;
    PyObject* next() {
        if (at >= n) throw BadArgument("too few arguments");
        return a[at++];
    }
    void* ptr() {                              // tensor or None
        PyObject* o = next();
        if (o == Py_None) return nullptr;
        if (!THPVariable_Check(o)) throw BadArgument("a tensor or None is expected");
        return THPVariable_Unpack(o).data_ptr();
    }
    template <class T> T* ptr() { return static_cast<T*>(ptr()); }
    int64_t i64() {
        const long long v = PyLong_AsLongLong(next());
        if (v == -1 && PyErr_Occurred()) throw BadArgument("");
        return v;
    }
    int i32() { return (int)i64(); }
    float f32() {
        const double v = PyFloat_AsDouble(next());
        if (v == -1.0 && PyErr_Occurred()) throw BadArgument("");
        return (float)v;
    }
    void* stream() { return (void*)(intptr_t)i64(); }
    struct Buffer { void* p; size_t bytes; };
    Buffer buffer() {                          // workspace: tensor or None
        PyObject* o = next();
        if (o == Py_None) return {nullptr, 0};
        if (!THPVariable_Check(o)) throw BadArgument("a tensor or None is expected");
        const at::Tensor& t = THPVariable_Unpack(o);
        return {t.data_ptr(), (size_t)t.nbytes()};
    }
    void done() const { if (at != n) throw BadArgument("too many arguments"); }
};

// Runs `call(args)` - which converts its arguments and returns the C function with them bound - and returns its code.
template <class F>
PyObject* enter(PyObject* const* argv, Py_ssize_t n, F call) {
    HANDLE_TH_ERRORS
    try {
        Args a{argv, n};
        auto bound = call(a);
        a.done();
        int rc;
        Py_BEGIN_ALLOW_THREADS
        rc = bound();
        Py_END_ALLOW_THREADS
        return PyLong_FromLong(rc);
    } catch (const BadArgument& e) {
        if (!PyErr_Occurred()) PyErr_SetString(PyExc_TypeError, e.what());
        return nullptr;
    }
    END_HANDLE_TH_ERRORS
}

PyObject* n_compress(PyObject*, PyObject* const* v, Py_ssize_t n) {
    return enter(v, n, [](Args& a) {
        auto z = a.ptr(); auto dt = a.i32(); auto ld = a.i64(); auto rows = a.i32(), V = a.i32(); auto T = a.f32(); auto k = a.i32(); auto top_p = a.f32();
        auto idx = a.ptr<int32_t>(); auto prob = a.ptr<float>(); auto count = a.ptr<int32_t>(); auto mass = a.ptr<float>(); auto lse = a.ptr<float>();
        auto ws = a.buffer(); auto s = a.stream();
        return [=] { return picospec_compress(z, dt, ld, rows, V, T, k, top_p, idx, prob, count, mass, lse, ws.p, ws.bytes, s); };
    });
}

PyObject* n_sample_draft(PyObject*, PyObject* const* v, Py_ssize_t n) {
    return enter(v, n, [](Args& a) {
        auto idx = a.ptr<int32_t>(); auto prob = a.ptr<float>(); auto count = a.ptr<int32_t>(); auto mass = a.ptr<float>();
        auto k = a.i32(), rows = a.i32(); auto uni = a.ptr<float>(); auto tok = a.ptr<int32_t>(); auto q = a.ptr<float>(); auto s = a.stream();
        return [=] { return picospec_sample_draft(idx, prob, count, mass, k, rows, uni, tok, q, s); };
    });
}

struct Records { const int32_t* idx; const float* prob; const int32_t* count; const float* mass; int k; };
Records records(Args& a) { auto i = a.ptr<int32_t>(); auto p = a.ptr<float>(); auto c = a.ptr<int32_t>(); auto m = a.ptr<float>(); return {i, p, c, m, a.i32()}; }
struct Verdict { int32_t* n; float *p, *q, *mx, *sm, *lse; uint32_t* fl; };
Verdict verdict(Args& a) {
    auto n = a.ptr<int32_t>(); auto p = a.ptr<float>(); auto q = a.ptr<float>(); auto mx = a.ptr<float>(); auto sm = a.ptr<float>(); auto lse = a.ptr<float>();
    return {n, p, q, mx, sm, lse, a.ptr<uint32_t>()};
}
struct Target { const void* z; int dt; int64_t ld; int V; float T; int B, N; const int32_t* off; };
Target target(Args& a) {
    auto z = a.ptr(); auto dt = a.i32(); auto ld = a.i64(); auto V = a.i32(); auto T = a.f32(); auto B = a.i32(), N = a.i32();
    return {z, dt, ld, V, T, B, N, a.ptr<int32_t>()};
}
struct Draw { int32_t* tok; float* mass; uint32_t* fl; };
Draw draw(Args& a) { auto t = a.ptr<int32_t>(); auto m = a.ptr<float>(); return {t, m, a.ptr<uint32_t>()}; }

PyObject* n_verify(PyObject*, PyObject* const* v, Py_ssize_t n) {
    return enter(v, n, [](Args& a) {
        auto t = target(a); auto tok = a.ptr<int32_t>(); auto q = records(a); auto renorm = a.i32(); auto qs = a.ptr<float>(); auto uni = a.ptr<float>();
        auto o = verdict(a); auto ws = a.buffer(); auto s = a.stream();
        return [=] { return picospec_verify(t.z, t.dt, t.ld, t.V, t.T, t.B, t.N, t.off, tok, q.idx, q.prob, q.count, q.mass, q.k, renorm, qs, uni,
                                            o.n, o.p, o.q, o.mx, o.sm, o.lse, o.fl, ws.p, ws.bytes, s); };
    });
}

PyObject* n_verify_range(PyObject*, PyObject* const* v, Py_ssize_t n) {
    return enter(v, n, [](Args& a) {
        auto t = target(a); auto tok = a.ptr<int32_t>(); auto q = records(a); auto renorm = a.i32(); auto qs = a.ptr<float>(); auto uni = a.ptr<float>();
        auto pb = a.ptr<int32_t>(); auto pe = a.ptr<int32_t>(); auto g = a.i32();
        auto o = verdict(a); auto ws = a.buffer(); auto s = a.stream();
        return [=] { return picospec_verify_range(t.z, t.dt, t.ld, t.V, t.T, t.B, t.N, t.off, tok, q.idx, q.prob, q.count, q.mass, q.k, renorm, qs, uni,
                                                  pb, pe, g, o.n, o.p, o.q, o.mx, o.sm, o.lse, o.fl, ws.p, ws.bytes, s); };
    });
}

PyObject* n_round(PyObject*, PyObject* const* v, Py_ssize_t n) {
    return enter(v, n, [](Args& a) {
        auto zd = a.ptr(), zt = a.ptr(); auto dt = a.i32(); auto ldd = a.i64(), ldt = a.i64(); auto V = a.i32(); auto T = a.f32(); auto B = a.i32(), N = a.i32();
        auto off = a.ptr<int32_t>(); auto tok = a.ptr<int32_t>(); auto k = a.i32(); auto top_p = a.f32(); auto renorm = a.i32(); auto uni = a.ptr<float>();
        auto idx = a.ptr<int32_t>(); auto prob = a.ptr<float>(); auto count = a.ptr<int32_t>(); auto mass = a.ptr<float>(); auto lse = a.ptr<float>();
        auto o = verdict(a); auto d = draw(a); auto ws = a.buffer(), own = a.buffer(); auto s = a.stream();
        if (own.p) ws = own;                     // (scratch(..) brings one only where the caller's does not serve)
        return [=] { return picospec_round(zd, zt, dt, ldd, ldt, V, T, B, N, off, tok, k, top_p, renorm, uni, idx, prob, count, mass, lse,
                                           o.n, o.p, o.q, o.mx, o.sm, o.lse, o.fl, d.tok, d.mass, d.fl, ws.p, ws.bytes, s); };
    });
}

PyObject* n_verify_sample(PyObject*, PyObject* const* v, Py_ssize_t n) {
    return enter(v, n, [](Args& a) {
        auto t = target(a); auto tok = a.ptr<int32_t>(); auto q = records(a); auto renorm = a.i32(); auto uni = a.ptr<float>();
        auto o = verdict(a); auto d = draw(a); auto ws = a.buffer(); auto s = a.stream();
        return [=] { return picospec_verify_sample(t.z, t.dt, t.ld, t.V, t.T, t.B, t.N, t.off, tok, q.idx, q.prob, q.count, q.mass, q.k, renorm, uni,
                                                   o.n, o.p, o.q, o.mx, o.sm, o.lse, o.fl, d.tok, d.mass, d.fl, ws.p, ws.bytes, s); };
    });
}

PyObject* n_verify_sample_static(PyObject*, PyObject* const* v, Py_ssize_t n) {
    return enter(v, n, [](Args& a) {
        auto t = target(a); auto tok = a.ptr<int32_t>(); auto q = records(a); auto renorm = a.i32(); auto uni = a.ptr<float>();
        auto o = verdict(a); auto d = draw(a); auto s = a.stream();
        return [=] { return picospec_verify_sample_static(t.z, t.dt, t.ld, t.V, t.T, t.B, t.N, t.off, tok, q.idx, q.prob, q.count, q.mass, q.k, renorm, uni,
                                                          o.n, o.p, o.q, o.mx, o.sm, o.lse, o.fl, d.tok, d.mass, d.fl, s); };
    });
}

template <auto CALL>
PyObject* n_sample_residual(PyObject*, PyObject* const* v, Py_ssize_t n) {
    return enter(v, n, [](Args& a) {
        auto t = target(a); auto na = a.ptr<int32_t>(); auto mx = a.ptr<float>(); auto sm = a.ptr<float>(); auto q = records(a); auto renorm = a.i32();
        auto uni = a.ptr<float>(); auto d = draw(a); auto ws = a.buffer(); auto s = a.stream();
        return [=] { return CALL(t.z, t.dt, t.ld, t.V, t.T, t.B, t.N, t.off, na, mx, sm, q.idx, q.prob, q.count, q.mass, q.k, renorm, uni,
                                 d.tok, d.mass, d.fl, ws.p, ws.bytes, s); };
    });
}

PyObject* n_row_stats(PyObject*, PyObject* const* v, Py_ssize_t n) {
    return enter(v, n, [](Args& a) {
        auto z = a.ptr(); auto dt = a.i32(); auto ld = a.i64(); auto rows = a.i32(), V = a.i32(); auto T = a.f32();
        auto mx = a.ptr<float>(); auto sm = a.ptr<float>(); auto lse = a.ptr<float>(); auto ws = a.buffer(); auto s = a.stream();
        return [=] { return picospec_row_stats_ws(z, dt, ld, rows, V, T, mx, sm, lse, ws.p, ws.bytes, s); };
    });
}

PyObject* n_compress_rejected(PyObject*, PyObject* const* v, Py_ssize_t n) {
    return enter(v, n, [](Args& a) {
        auto t = target(a); auto na = a.ptr<int32_t>(); auto k = a.i32(); auto top_p = a.f32();
        auto idx = a.ptr<int32_t>(); auto prob = a.ptr<float>(); auto count = a.ptr<int32_t>(); auto mass = a.ptr<float>(); auto lse = a.ptr<float>();
        auto ws = a.buffer(); auto s = a.stream();
        return [=] { return picospec_compress_rejected(t.z, t.dt, t.ld, t.V, t.T, t.B, t.N, t.off, na, k, top_p, idx, prob, count, mass, lse, ws.p, ws.bytes, s); };
    });
}

PyObject* n_resample_sparse(PyObject*, PyObject* const* v, Py_ssize_t n) {
    return enter(v, n, [](Args& a) {
        auto t = target(a); auto na = a.ptr<int32_t>(); auto mx = a.ptr<float>(); auto sm = a.ptr<float>(); auto q = records(a); auto renorm = a.i32();
        auto uni = a.ptr<float>(); auto d = draw(a); auto s = a.stream();
        return [=] { return picospec_resample_sparse(t.z, t.dt, t.ld, t.V, t.T, t.B, t.N, t.off, na, mx, sm, q.idx, q.prob, q.count, q.mass, q.k, renorm, uni,
                                                     d.tok, d.mass, d.fl, nullptr, 0, s); };
    });
}

PyObject* n_pack_downlink(PyObject*, PyObject* const* v, Py_ssize_t n) {
    return enter(v, n, [](Args& a) {
        auto B = a.i32(); auto off = a.ptr<int32_t>(); auto na = a.ptr<int32_t>(); auto tok = a.ptr<int32_t>(); auto idx = a.ptr<int32_t>(); auto prob = a.ptr<float>();
        auto count = a.ptr<int32_t>(); auto k = a.i32(), fmt = a.i32(); auto wire = a.ptr(); auto cap = a.i64(); auto nb = a.ptr<int64_t>(); auto st = a.ptr<uint32_t>(); auto s = a.stream();
        return [=] { return picospec_pack_downlink(B, off, na, tok, idx, prob, count, k, fmt, wire, cap, nb, st, s); };
    });
}

PyObject* n_unpack_downlink(PyObject*, PyObject* const* v, Py_ssize_t n) {
    return enter(v, n, [](Args& a) {
        auto wire = a.ptr(); auto bytes = a.i64(); auto B = a.i32(), k = a.i32(); auto na = a.ptr<int32_t>(); auto tok = a.ptr<int32_t>();
        auto idx = a.ptr<int32_t>(); auto prob = a.ptr<float>(); auto count = a.ptr<int32_t>(); auto mass = a.ptr<float>(); auto st = a.ptr<uint32_t>(); auto s = a.stream();
        return [=] { return picospec_unpack_downlink(wire, bytes, B, k, na, tok, idx, prob, count, mass, st, s); };
    });
}

PyObject* n_pack_uplink(PyObject*, PyObject* const* v, Py_ssize_t n) {
    return enter(v, n, [](Args& a) {
        auto B = a.i32(), N = a.i32(); auto off = a.ptr<int32_t>(); auto tok = a.ptr<int32_t>(); auto q = a.ptr<float>(); auto fmt = a.i32();
        auto wire = a.ptr(); auto cap = a.i64(); auto nb = a.ptr<int64_t>(); auto s = a.stream();
        return [=] { return picospec_pack_uplink(B, N, off, tok, q, fmt, wire, cap, nb, s); };
    });
}

PyObject* n_unpack_uplink(PyObject*, PyObject* const* v, Py_ssize_t n) {
    return enter(v, n, [](Args& a) {
        auto wire = a.ptr(); auto bytes = a.i64(); auto B = a.i32(), nm = a.i32(); auto off = a.ptr<int32_t>(); auto tok = a.ptr<int32_t>(); auto q = a.ptr<float>();
        auto st = a.ptr<uint32_t>(); auto s = a.stream();
        return [=] { return picospec_unpack_uplink(wire, bytes, B, nm, off, tok, q, st, s); };
    });
}

// rows2d(tensor) -> (dtype code, stride of a row, rows), or an error code of the library: a 2-d device tensor whose rows are
// contiguous (the strides of a tensor without rows mean nothing)
PyObject* n_rows2d(PyObject*, PyObject* o) {
    HANDLE_TH_ERRORS
    if (!THPVariable_Check(o)) { PyErr_SetString(PyExc_TypeError, "a tensor is expected"); return nullptr; }
    const at::Tensor& t = THPVariable_Unpack(o);
    if (t.dim() != 2 || !t.is_cuda()) return PyLong_FromLong(PICOSPEC_EINVAL);
    int dt;
    if (t.scalar_type() == at::kFloat) dt = PICOSPEC_F32;
    else if (t.scalar_type() == at::kBFloat16) dt = PICOSPEC_BF16;
    else return PyLong_FromLong(t.size(0) != 0 && t.stride(1) != 1 ? PICOSPEC_EINVAL : PICOSPEC_EDTYPE);
    const int64_t rows = t.size(0);
    if (rows != 0 && t.stride(1) != 1) return PyLong_FromLong(PICOSPEC_EINVAL);
    return Py_BuildValue("(iLL)", dt, (long long)(rows ? t.stride(0) : t.size(1)), (long long)rows);
    END_HANDLE_TH_ERRORS
}

at::TensorOptions like(PyObject* o, at::ScalarType type) { return at::TensorOptions().dtype(type).device(THPVariable_Unpack(o).device()); }

// scratch_bytes(which, dtype, n_draft, B, V, k) -> picospec_scratch_bytes(...)
PyObject* n_scratch_bytes(PyObject*, PyObject* const* v, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    try {
        Args a{v, n};
        const int which = a.i32(), dt = a.i32(), N = a.i32(), B = a.i32(), V = a.i32(), k = a.i32();
        a.done();
        return PyLong_FromSize_t(picospec_scratch_bytes(which, dt, N, B, V, k));
    } catch (const BadArgument& e) {
        if (!PyErr_Occurred()) PyErr_SetString(PyExc_TypeError, e.what());
        return nullptr;
    }
    END_HANDLE_TH_ERRORS
}

// scratch(like, which, dtype, n_draft, B, V, k[, given]) -> uint8 tensor of picospec_one_launch_bytes(...) bytes.  None where that is
// 0, where the caller's workspace `given` holds as many, and where the library refuses that one (it still does).
PyObject* n_scratch(PyObject*, PyObject* const* v, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    try {
        if ((n != 7 && n != 8) || !THPVariable_Check(v[0])) throw BadArgument("scratch(tensor, which, dtype, n_draft, B, V, k[, given])");
        Args a{v, n, 1};
        const int which = a.i32(), dt = a.i32(), N = a.i32(), B = a.i32(), V = a.i32(), k = a.i32();
        const size_t bytes = picospec_scratch_bytes(which, dt, N, B, V, k);
        if (!bytes) Py_RETURN_NONE;
        if (n == 8) {
            const Args::Buffer given = a.buffer();
            if (given.p && (given.bytes >= bytes || ((uintptr_t)given.p & 15u) || given.bytes < picospec_workspace_bytes(which, dt, N + B, V, 0))) Py_RETURN_NONE;
        }
        return THPVariable_Wrap(at::empty({(int64_t)picospec_one_launch_bytes(which, dt, N, B, V, k)}, like(v[0], at::kByte)));
    } catch (const BadArgument& e) {
        if (!PyErr_Occurred()) PyErr_SetString(PyExc_TypeError, e.what());
        return nullptr;
    }
    END_HANDLE_TH_ERRORS
}

// empty(like, codes, size, ...) -> one tensor per letter of `codes` (i int32, l int64, f float32, b uint8) on the device of
// `like`; a size is an int (1-d) or a tuple of two.  Outputs of up to kShared bytes share one allocation, each from a 512-byte boundary of it
// on, as slices of a tensor do: an allocation costs 0.45 to 0.85 us, a slice 0.15 (the eight outputs of an unpacked downlink message of 32
// records of 256: 2.1 us, each from torch.empty 6.8).  All of it lives as long as any of them, so larger ones, next to which an allocation is cheap to make and
// dear to keep, have their own.
PyObject* n_empty(PyObject*, PyObject* const* v, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    constexpr Py_ssize_t kMost = 16;
    constexpr int64_t kShared = 64 * 1024;
    Py_ssize_t len = 0;
    const char* codes = n >= 2 && THPVariable_Check(v[0]) ? PyUnicode_AsUTF8AndSize(v[1], &len) : nullptr;
    if (!codes || n != len + 2 || len > kMost) { if (!PyErr_Occurred()) PyErr_SetString(PyExc_TypeError, "empty(tensor, codes, size, ...)"); return nullptr; }
    int64_t dims[kMost][2], bytes[kMost], shared = 0;
    int nd[kMost];
    for (Py_ssize_t i = 0; i < len; ++i) {
        PyObject* s = v[2 + i];
        nd[i] = PyTuple_Check(s) && PyTuple_GET_SIZE(s) == 2 ? 2 : 1;
        dims[i][0] = PyLong_AsLongLong(nd[i] == 2 ? PyTuple_GET_ITEM(s, 0) : s);
        dims[i][1] = nd[i] == 2 ? PyLong_AsLongLong(PyTuple_GET_ITEM(s, 1)) : 1;
        if (PyErr_Occurred()) return nullptr;
        if (dims[i][0] < 0 || dims[i][1] < 0 || __builtin_mul_overflow(dims[i][0], dims[i][1], &bytes[i]) || bytes[i] > (int64_t(1) << 56)) { PyErr_SetString(PyExc_RuntimeError, "empty: a size is out of range"); return nullptr; }
        bytes[i] *= codes[i] == 'l' ? 8 : codes[i] == 'b' ? 1 : 4;
        if (bytes[i] <= kShared) shared += (bytes[i] + 511) / 512 * 512;
    }
    THPObjectPtr out(PyTuple_New(len));
    if (!out) return nullptr;
    at::Tensor block;
    int64_t at_byte = 0;
    for (Py_ssize_t i = 0; i < len; ++i) {
        const at::ScalarType type = codes[i] == 'i' ? at::kInt : codes[i] == 'l' ? at::kLong : codes[i] == 'b' ? at::kByte : at::kFloat;
        at::Tensor piece;
        if (bytes[i] > kShared) {
            piece = at::empty(at::IntArrayRef(dims[i], nd[i]), like(v[0], type));
        } else {
            if (!block.defined()) block = at::empty({shared}, like(v[0], at::kByte));
            piece = at::detail::make_tensor<c10::TensorImpl>(c10::Storage(block.storage()), block.key_set(), c10::scalarTypeToTypeMeta(type));
            piece.unsafeGetTensorImpl()->set_storage_offset(at_byte / (int64_t)c10::elementSize(type));
            piece.unsafeGetTensorImpl()->set_sizes_contiguous(at::IntArrayRef(dims[i], nd[i]));
            at_byte += (bytes[i] + 511) / 512 * 512;
        }
        PyObject* t = THPVariable_Wrap(piece);
        if (!t) return nullptr;
        PyTuple_SET_ITEM(out.get(), i, t);
    }
    return out.release();
    END_HANDLE_TH_ERRORS
}

#define FAST(name, f) {name, (PyCFunction)(void (*)(void))f, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    FAST("compress", n_compress), FAST("sample_draft", n_sample_draft), FAST("verify", n_verify), FAST("verify_range", n_verify_range),
    FAST("round", n_round), FAST("verify_sample", n_verify_sample), FAST("verify_sample_static", n_verify_sample_static),
    FAST("sample_residual", n_sample_residual<picospec_sample_residual>), FAST("sample_residual_ws", n_sample_residual<picospec_sample_residual_ws>), FAST("row_stats", n_row_stats), FAST("compress_rejected", n_compress_rejected),
    FAST("resample_sparse", n_resample_sparse), FAST("pack_downlink", n_pack_downlink), FAST("unpack_downlink", n_unpack_downlink),
    FAST("pack_uplink", n_pack_uplink), FAST("unpack_uplink", n_unpack_uplink), FAST("scratch_bytes", n_scratch_bytes), FAST("scratch", n_scratch), FAST("empty", n_empty),
    {"rows2d", (PyCFunction)n_rows2d, METH_O, nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native(void) { return PyModule_Create(&module); }
