// Argument marshalling between torch tensors and the C ABI of include/signsgd.h, as a CPython module.
//
// A step hands over up to 3 M + 3 tensors; checked and unpacked one attribute at a time in Python that
// took 12 us for M = 7, more than twice what the kernel of a small step takes.  Here every tensor is
// checked (device memory, dtype, contiguous, long enough) and unpacked in a few nanoseconds, the
// library is called without the interpreter lock, and its status goes back as an int.  Nothing
// is computed, kept or synchronised here.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/ATen.h>
#include <c10/hip/HIPCachingAllocator.h>
#include <c10/hip/HIPStream.h>
#include <hip/hip_runtime_api.h>
#include <torch/csrc/autograd/python_variable.h>

#include <algorithm>
#include <cstring>
#include <exception>
#include <stdexcept>

#include "../../include/signsgd.h"

namespace {

// a Python exception is set: unwind to the entry point
struct PyRaised {};

[[noreturn]] void raise_type(const char *name, int index, const char *fmt, ...) {
    char who[64], what[160];
    if (index >= 0) snprintf(who, sizeof who, "%s[%d]", name, index);
    else snprintf(who, sizeof who, "%s", name);
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(what, sizeof what, fmt, ap);
    va_end(ap);
    PyErr_Format(PyExc_TypeError, "%s %s", who, what);
    throw PyRaised();
}

const at::Tensor &tensor(PyObject *o, const char *name, int index = -1) {
    if (!THPVariable_Check(o)) raise_type(name, index, "must be a tensor, got %s", Py_TYPE(o)->tp_name);
    return THPVariable_Unpack(o);
}

enum Kind { kGrad, kF32, kF64, kI64, kI8, kBits };

bool is_kind(at::ScalarType t, Kind kind) {
    switch (kind) {
        case kGrad: return t == at::kFloat || t == at::kBFloat16;
        case kF32: return t == at::kFloat;
        case kF64: return t == at::kDouble;
        case kI64: return t == at::kLong;
        case kI8: return t == at::kChar;
        default: return t == at::kInt || t == at::kUInt32;
    }
}

// device address of a tensor that has `n` elements of the kind, contiguous, in device memory
void *dev(PyObject *o, Kind kind, size_t n, const char *name, int index = -1) {
    const at::Tensor &t = tensor(o, name, index);
    if (!t.is_cuda()) raise_type(name, index, "must live in device memory");
    if (!is_kind(t.scalar_type(), kind)) raise_type(name, index, "has dtype %s", at::toString(t.scalar_type()));
    if (!t.is_contiguous() || (size_t)t.numel() < n) raise_type(name, index, "must be contiguous with at least %zu elements", n);
    return t.data_ptr();
}

void *dev_or_null(PyObject *o, Kind kind, size_t n, const char *name) {
    return o == Py_None ? nullptr : dev(o, kind, n, name);
}

ss_dtype grad_dtype(at::ScalarType t) {
    if (t == at::kFloat) return SS_F32;
    if (t == at::kBFloat16) return SS_BF16;
    PyErr_Format(PyExc_TypeError, "gradient dtype must be float32 or bfloat16, got %s", at::toString(t));
    throw PyRaised();
}

// a number may also come as the ctypes object that a ctypes call would take: what it holds, a new
// reference; anything else unchanged
PyObject *plain(PyObject *o, const char *ctype) {
    if (!strcmp(Py_TYPE(o)->tp_name, ctype)) {
        PyObject *v = PyObject_GetAttrString(o, "value");
        if (!v) throw PyRaised();
        return v;
    }
    Py_INCREF(o);
    return o;
}

// integers wrap to the C type's width, as a ctypes call converts them
uint64_t wrapped(PyObject *o, const char *ctype = "c_ulong") {
    PyObject *number = plain(o, ctype);
    PyObject *i = PyNumber_Index(number);
    Py_DECREF(number);
    if (!i) throw PyRaised();
    const uint64_t v = PyLong_AsUnsignedLongLongMask(i);
    Py_DECREF(i);
    if (v == (uint64_t)-1 && PyErr_Occurred()) throw PyRaised();
    return v;
}

// a number of coordinates does not wrap: it is compared with the tensors' lengths
size_t size_arg(PyObject *o) {
    PyObject *i = PyNumber_Index(o);
    if (!i) throw PyRaised();
    const size_t v = PyLong_AsSize_t(i);
    Py_DECREF(i);
    if (v == (size_t)-1 && PyErr_Occurred()) {
        PyErr_Clear();
        PyErr_Format(PyExc_TypeError, "%R is no number of coordinates", o);
        throw PyRaised();
    }
    return v;
}

int int_arg(PyObject *o) { return (int)(uint32_t)wrapped(o, "c_int"); }

// number of coordinates: as given, or the tensor's own
size_t coords(PyObject *d, PyObject *t, const char *name) {
    return d == Py_None ? (size_t)tensor(t, name).numel() : size_arg(d);
}

float float_arg(PyObject *o) {
    PyObject *number = plain(o, "c_float");
    const double v = PyFloat_AsDouble(number);
    Py_DECREF(number);
    if (v == -1.0 && PyErr_Occurred()) throw PyRaised();
    return (float)v;
}

void *handle_arg(PyObject *o, const char *attribute) {
    PyObject *h = PyObject_GetAttrString(o, attribute);
    if (!h) throw PyRaised();
    void *p = PyLong_AsVoidPtr(h);
    Py_DECREF(h);
    if (!p && PyErr_Occurred()) throw PyRaised();
    return p;
}

hipStream_t stream_arg(PyObject *o) {
    if (o == Py_None) return c10::hip::getCurrentHIPStream().stream();
    return static_cast<hipStream_t>(handle_arg(o, "cuda_stream"));
}

// whether the stream of a call is one of torch's own: the default stream or one of its pools.  A stream that
// torch was handed (ExternalStream) has its handle for an id.
bool own_stream(PyObject *o, hipStream_t handle) {
    if (!handle) return true;
    if (o == Py_None) return reinterpret_cast<void *>(c10::hip::getCurrentHIPStream().id()) != handle;
    if (!PyObject_HasAttrString(o, "stream_id")) return false;
    return handle_arg(o, "stream_id") != handle;
}

// the device addresses of a sequence of tensors, one per worker; of more than SS_MAX_WORKERS all are
// checked and the library refuses their number
struct Workers {
    int n = 0;
    void *p[SS_MAX_WORKERS];

    Workers() = default;
    Workers(PyObject *seq, Kind kind, size_t elems, const char *name, const at::ScalarType *like = nullptr) {
        PyObject *fast = PySequence_Fast(seq, "one tensor per worker is wanted");
        if (!fast) throw PyRaised();
        const Py_ssize_t len = PySequence_Fast_GET_SIZE(fast);
        PyObject **items = PySequence_Fast_ITEMS(fast);
        try {
            for (Py_ssize_t i = 0; i < len; ++i) {
                void *q = dev(items[i], kind, elems, name, (int)i);
                const at::ScalarType t = THPVariable_Unpack(items[i]).scalar_type();
                if (like && t != *like) raise_type(name, (int)i, "has dtype %s", at::toString(t));
                if (i < SS_MAX_WORKERS) p[i] = q;
            }
        } catch (...) {
            Py_DECREF(fast);
            throw;
        }
        Py_DECREF(fast);
        n = (int)len;
    }
    template <typename T>
    T *const *as() const { return reinterpret_cast<T *const *>(p); }
};

// dtype of the first of a sequence of gradients (they all have to have it); the sequence has a length and
// is indexed as Python does it, so that a stacked tensor counts as one
at::ScalarType first_dtype(PyObject *seq) {
    if (PyObject_Size(seq) < 0) throw PyRaised();
    PyObject *zero = PyLong_FromLong(0);
    PyObject *o = zero ? PyObject_GetItem(seq, zero) : nullptr;
    Py_XDECREF(zero);
    if (!o) throw PyRaised();
    const bool is_tensor = THPVariable_Check(o);
    const at::ScalarType t = is_tensor ? THPVariable_Unpack(o).scalar_type() : at::kFloat;
    Py_DECREF(o);
    return t;     // Workers says what is wrong with anything else
}

// What has to be free beyond the memory that a step borrows: the allocator rounds a request up (to 2 or 20 MiB
// blocks, or as it is configured to), and what the program allocates next should not be what does not fit.
constexpr size_t kLeaveFree = (size_t)1 << 30;

// Whether torch's allocator can serve `wanted` bytes without more than a plain allocation.  One that it
// cannot serve makes it wait for the device, give back everything it caches and try again, which a
// step that is as well off with one pass must not cause.  Asked of the device at every call, because
// other processes and other libraries take memory too: 5 us of host time behind queued work, 9 in front of an
// idle device (d = 6.5 M, M = 8 bf16: 15 us a call, 17 before these calls were native).  Anything but
// torch's own caching allocator may synchronise on each allocation.
bool room_for(size_t wanted, int device) {
    namespace allocator = c10::hip::HIPCachingAllocator;
    if (allocator::name() != "native" || !allocator::isEnabled()) return false;
    size_t free = 0, total = 0;
    if (hipMemGetInfo(&free, &total) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    const double fraction = allocator::getMemoryFraction((c10::DeviceIndex)device);
    if (fraction < 1.0) {       // the program bounds what it takes of the device
        const size_t bound = (size_t)(fraction * (double)total);
        const size_t held = (size_t)allocator::getDeviceStats((c10::DeviceIndex)device).reserved_bytes[0].current;
        free = std::min(free, bound > held ? bound - held : 0);
    }
    return free >= wanted + kLeaveFree;
}

// Temporary device memory for one step, from torch's caching allocator and tied to the step's own
// stream (so that its reuse is ordered behind the step); given back when the step is enqueued.  The
// allocator keeps a block for each stream that takes such steps, until it needs the memory or is told to
// empty its cache.
// None where nothing is wanted, there is no room, the tensors are not on the current device,
// the stream is under capture (a replay may not touch memory that has been given back), or
// it is not torch's own: the allocator knows a stream by its handle, and what is queued behind a handle
// from elsewhere need not be one queue - hipStreamPerThread is another stream in every thread, and a
// destroyed stream's handle may come back as a new one - so the next step under it could be lent
// the block of one that still runs.
struct Lent {
    void *p = nullptr;
    size_t bytes = 0;

    Lent(size_t wanted, int device, hipStream_t stream, bool own) {
        int current = -1;
        if (wanted == 0 || !own || hipGetDevice(&current) != hipSuccess || current != device) return;
        hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
        if (hipStreamIsCapturing(stream, &status) != hipSuccess) {
            (void)hipGetLastError();    // the default stream while another one captures
            return;
        }
        if (status != hipStreamCaptureStatusNone) return;
        // nothing here is captured, so a capture that another thread has open must not forbid (nor be
        // broken by) the allocation
        hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
        const bool relaxed = hipThreadExchangeStreamCaptureMode(&mode) == hipSuccess;
        try {
            if (room_for(wanted, device)) p = c10::hip::HIPCachingAllocator::raw_alloc_with_stream(wanted, stream);
            bytes = p ? wanted : 0;
        } catch (const std::exception &) {
            p = nullptr;                // out of memory after all: one pass needs none
        }
        if (relaxed) (void)hipThreadExchangeStreamCaptureMode(&mode);
    }
    ~Lent() {
        if (!p) return;
        try {
            c10::hip::HIPCachingAllocator::raw_delete(p);
        } catch (const std::exception &) {
        }
    }
    Lent(const Lent &) = delete;
    Lent &operator=(const Lent &) = delete;
};

template <typename F>
int unlocked(F call) {
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = call();
    Py_END_ALLOW_THREADS
    return rc;
}

// entry point: argument count, C++ exceptions to Python ones, status as an int
template <int N, typename F>
PyObject *entry(Py_ssize_t nargs, F body) {
    if (nargs != N) {
        PyErr_Format(PyExc_TypeError, "expected %d arguments, got %zd", N, nargs);
        return nullptr;
    }
    try {
        return PyLong_FromLong(body());
    } catch (const PyRaised &) {
    } catch (const std::exception &e) {
        PyErr_SetString(PyExc_RuntimeError, e.what());
    }
    return nullptr;
}

// (g, m, beta, packed, d, stream, warmup)
PyObject *signum_pack(PyObject *, PyObject *const *a, Py_ssize_t n) {
    return entry<7>(n, [&] {
        const size_t d = coords(a[4], a[0], "g");
        void *g = dev(a[0], kGrad, d, "g");
        float *m = (float *)dev_or_null(a[1], kF32, d, "m");
        uint32_t *packed = (uint32_t *)dev(a[3], kBits, ss_packed_bytes(d) / 4, "packed");
        const ss_dtype gdt = grad_dtype(tensor(a[0], "g").scalar_type());
        const float beta = float_arg(a[2]);
        const hipStream_t s = stream_arg(a[5]);
        const bool warmup = PyObject_IsTrue(a[6]) == 1;
        return unlocked([&] { return (warmup ? ss_signum_pack_warmup : ss_signum_pack)(g, gdt, m, beta, packed, d, s); });
    });
}

// (packed, voted, d, stream)
PyObject *majority_vote(PyObject *, PyObject *const *a, Py_ssize_t n) {
    return entry<4>(n, [&] {
        const size_t d = size_arg(a[2]), words = ss_packed_bytes(d) / 4;
        const Workers packed(a[0], kBits, words, "packed");
        uint32_t *voted = (uint32_t *)dev(a[1], kBits, words, "voted");
        const hipStream_t s = stream_arg(a[3]);
        return unlocked([&] { return ss_majority_vote(packed.as<const uint32_t>(), packed.n, voted, d, s); });
    });
}

// (packed, sums, d, stream)
PyObject *vote_sum(PyObject *, PyObject *const *a, Py_ssize_t n) {
    return entry<4>(n, [&] {
        const size_t d = size_arg(a[2]);
        const Workers packed(a[0], kBits, ss_packed_bytes(d) / 4, "packed");
        int8_t *sums = (int8_t *)dev(a[1], kI8, d, "sums");
        const hipStream_t s = stream_arg(a[3]);
        return unlocked([&] { return ss_vote_sum(packed.as<const uint32_t>(), packed.n, sums, d, s); });
    });
}

// (x, bits, delta, d, stream)
PyObject *sign_apply(PyObject *, PyObject *const *a, Py_ssize_t n) {
    return entry<5>(n, [&] {
        const size_t d = coords(a[3], a[0], "x");
        float *x = (float *)dev(a[0], kF32, d, "x");
        uint32_t *bits = (uint32_t *)dev(a[1], kBits, ss_packed_words(d), "bits");
        const float delta = float_arg(a[2]);
        const hipStream_t s = stream_arg(a[4]);
        return unlocked([&] { return ss_sign_apply(x, bits, delta, d, s); });
    });
}

// (x, sums, delta, d, stream)
PyObject *sum_apply(PyObject *, PyObject *const *a, Py_ssize_t n) {
    return entry<5>(n, [&] {
        const size_t d = coords(a[3], a[0], "x");
        float *x = (float *)dev(a[0], kF32, d, "x");
        int8_t *sums = (int8_t *)dev(a[1], kI8, d, "sums");
        const float delta = float_arg(a[2]);
        const hipStream_t s = stream_arg(a[4]);
        return unlocked([&] { return ss_sum_apply(x, sums, delta, d, s); });
    });
}

// (g, m, beta, delta, x, voted, packed_out, sums_out, flags, d, stream)
PyObject *signum_vote_step(PyObject *, PyObject *const *a, Py_ssize_t n) {
    return entry<11>(n, [&] {
        const at::Tensor &x = tensor(a[4], "x");
        const size_t d = coords(a[9], a[4], "x"), words = ss_packed_bytes(d) / 4;
        const at::ScalarType g0 = first_dtype(a[0]);
        const ss_dtype gdt = grad_dtype(g0);
        const Workers g(a[0], kGrad, d, "g", &g0);
        const bool has_m = a[1] != Py_None, has_packed = a[6] != Py_None;
        const Workers m = has_m ? Workers(a[1], kF32, d, "m") : Workers();
        const Workers packed = has_packed ? Workers(a[6], kBits, words, "packed_out") : Workers();
        if ((has_m && m.n != g.n) || (has_packed && packed.n != g.n)) {
            PyErr_SetString(PyExc_ValueError, "g, m and packed_out must have one entry per worker");
            throw PyRaised();
        }
        float *xp = (float *)dev(a[4], kF32, d, "x");
        uint32_t *voted = (uint32_t *)dev(a[5], kBits, words, "voted");
        int8_t *sums = (int8_t *)dev_or_null(a[7], kI8, d, "sums_out");
        const unsigned flags = (unsigned)int_arg(a[8]);
        const float beta = float_arg(a[2]), delta = float_arg(a[3]);
        const hipStream_t s = stream_arg(a[10]);
        float *const *mp = has_m ? m.as<float>() : nullptr;
        if (has_packed)
            return unlocked([&] {
                return ss_signum_vote_step_ex(g.as<const void>(), gdt, mp, g.n, beta, delta, xp, voted, packed.as<uint32_t>(),
                                              sums, d, flags, s);
            });
        const int device = x.device().index();
        const bool own = own_stream(a[10], s);
        return unlocked([&] {
            const Lent scratch(ss_step_scratch_bytes(gdt, has_m, g.n, d), device, s, own);
            return ss_signum_vote_step_scratch(g.as<const void>(), gdt, mp, g.n, beta, delta, xp, voted, sums, scratch.p,
                                               scratch.bytes, d, flags, s);
        });
    });
}

// a copy asks for no more than an address: of a tensor, or of whatever answers data_ptr() (a storage)
void *address(PyObject *o) {
    if (THPVariable_Check(o)) return THPVariable_Unpack(o).data_ptr();
    PyObject *h = PyObject_CallMethod(o, "data_ptr", nullptr);
    if (!h) throw PyRaised();
    void *p = PyLong_AsVoidPtr(h);
    Py_DECREF(h);
    if (!p && PyErr_Occurred()) throw PyRaised();
    return p;
}

// (dst, src, nbytes, stream)
PyObject *stream_copy(PyObject *, PyObject *const *a, Py_ssize_t n) {
    return entry<4>(n, [&] {
        void *dst = address(a[0]);
        const void *src = address(a[1]);
        const size_t nbytes = wrapped(a[2]);
        const hipStream_t s = stream_arg(a[3]);
        return unlocked([&] { return ss_stream_copy(dst, src, nbytes, s); });
    });
}

// (g, mean, m2, n, d, stream)
PyObject *welford_update(PyObject *, PyObject *const *a, Py_ssize_t n) {
    return entry<6>(n, [&] {
        const size_t d = coords(a[4], a[1], "mean");
        void *g = dev(a[0], kGrad, d, "g");
        const ss_dtype gdt = grad_dtype(tensor(a[0], "g").scalar_type());
        float *mean = (float *)dev(a[1], kF32, d, "mean");
        float *m2 = (float *)dev(a[2], kF32, d, "m2");
        const uint64_t k = wrapped(a[3]);
        const hipStream_t s = stream_arg(a[5]);
        return unlocked([&] { return ss_welford_update(g, gdt, mean, m2, k, d, s); });
    });
}

// (m2, n, sigma, d, stream)
PyObject *welford_sigma(PyObject *, PyObject *const *a, Py_ssize_t n) {
    return entry<5>(n, [&] {
        const size_t d = coords(a[3], a[0], "m2");
        float *m2 = (float *)dev(a[0], kF32, d, "m2");
        const uint64_t k = wrapped(a[1]);
        float *sigma = (float *)dev(a[2], kF32, d, "sigma");
        const hipStream_t s = stream_arg(a[4]);
        return unlocked([&] { return ss_welford_sigma(m2, k, sigma, d, s); });
    });
}

// (v, out, workspace, d, stream); workspace None: the library's own fixed array
PyObject *density(PyObject *, PyObject *const *a, Py_ssize_t n) {
    return entry<5>(n, [&] {
        const size_t d = coords(a[3], a[0], "v");
        float *v = d ? (float *)dev(a[0], kF32, d, "v") : nullptr;
        void *ws = dev_or_null(a[2], kI64, ss_density_workspace_bytes() / 8, "workspace");
        double *out = (double *)dev(a[1], kF64, 3, "out");
        const hipStream_t s = stream_arg(a[4]);
        return unlocked([&] { return ws ? ss_density(v, d, out, ws, s) : ss_density_static(v, d, out, s); });
    });
}

// (g, m, beta, tau, neg, zero, d, stream)
PyObject *signum_pack_ternary(PyObject *, PyObject *const *a, Py_ssize_t n) {
    return entry<8>(n, [&] {
        const size_t d = coords(a[6], a[0], "g"), words = ss_packed_bytes(d) / 4;
        void *g = dev(a[0], kGrad, d, "g");
        const ss_dtype gdt = grad_dtype(tensor(a[0], "g").scalar_type());
        float *m = (float *)dev_or_null(a[1], kF32, d, "m");
        const float beta = float_arg(a[2]), tau = float_arg(a[3]);
        uint32_t *neg = (uint32_t *)dev(a[4], kBits, words, "neg");
        uint32_t *zero = (uint32_t *)dev(a[5], kBits, words, "zero");
        const hipStream_t s = stream_arg(a[7]);
        return unlocked([&] { return ss_signum_pack_ternary(g, gdt, m, beta, tau, neg, zero, d, s); });
    });
}

// (neg, zero, quorum, voted_neg, voted_zero, d, stream)
PyObject *quorum_vote(PyObject *, PyObject *const *a, Py_ssize_t n) {
    return entry<7>(n, [&] {
        const size_t d = size_arg(a[5]), words = ss_packed_bytes(d) / 4;
        const Workers neg(a[0], kBits, words, "neg");
        const Workers zero(a[1], kBits, words, "zero");
        if (neg.n != zero.n) {
            PyErr_SetString(PyExc_ValueError, "one neg and one zero plane per worker");
            throw PyRaised();
        }
        const int quorum = int_arg(a[2]);
        uint32_t *vneg = (uint32_t *)dev(a[3], kBits, words, "voted_neg");
        uint32_t *vzero = (uint32_t *)dev(a[4], kBits, words, "voted_zero");
        const hipStream_t s = stream_arg(a[6]);
        return unlocked([&] {
            return ss_quorum_vote(neg.as<const uint32_t>(), zero.as<const uint32_t>(), neg.n, quorum, vneg, vzero, d, s);
        });
    });
}

// (x, neg, zero, delta, d, stream)
PyObject *ternary_apply(PyObject *, PyObject *const *a, Py_ssize_t n) {
    return entry<6>(n, [&] {
        const size_t d = coords(a[4], a[0], "x"), words = ss_packed_words(d);
        float *x = (float *)dev(a[0], kF32, d, "x");
        uint32_t *neg = (uint32_t *)dev(a[1], kBits, words, "neg");
        uint32_t *zero = (uint32_t *)dev(a[2], kBits, words, "zero");
        const float delta = float_arg(a[3]);
        const hipStream_t s = stream_arg(a[5]);
        return unlocked([&] { return ss_ternary_apply(x, neg, zero, delta, d, s); });
    });
}

// (g, m, beta, tau, quorum, delta, x, voted_neg, voted_zero, d, stream)
PyObject *signum_vote_step_ternary(PyObject *, PyObject *const *a, Py_ssize_t n) {
    return entry<11>(n, [&] {
        const size_t d = coords(a[9], a[6], "x"), words = ss_packed_bytes(d) / 4;
        const at::ScalarType g0 = first_dtype(a[0]);
        const Workers g(a[0], kGrad, d, "g", &g0);
        const bool has_m = a[1] != Py_None;
        const Workers m = has_m ? Workers(a[1], kF32, d, "m") : Workers();
        if (has_m && m.n != g.n) {
            PyErr_SetString(PyExc_ValueError, "one momentum buffer per worker");
            throw PyRaised();
        }
        const ss_dtype gdt = grad_dtype(g0);
        const float beta = float_arg(a[2]), tau = float_arg(a[3]), delta = float_arg(a[5]);
        const int quorum = int_arg(a[4]);
        float *x = (float *)dev(a[6], kF32, d, "x");
        uint32_t *vneg = (uint32_t *)dev(a[7], kBits, words, "voted_neg");
        uint32_t *vzero = (uint32_t *)dev(a[8], kBits, words, "voted_zero");
        const hipStream_t s = stream_arg(a[10]);
        const int device = tensor(a[6], "x").device().index();
        const bool own = own_stream(a[10], s);
        return unlocked([&] {
            const Lent scratch(ss_ternary_scratch_bytes(gdt, has_m, g.n, d), device, s, own);
            return ss_signum_vote_step_ternary_scratch(g.as<const void>(), gdt, has_m ? m.as<float>() : nullptr, g.n, beta, tau,
                                                       quorum, delta, x, vneg, vzero, scratch.p, scratch.bytes, d, s);
        });
    });
}

#define SS_METHOD(name) {#name, (PyCFunction)(void (*)(void))name, METH_FASTCALL, nullptr}
PyMethodDef kMethods[] = {
    SS_METHOD(signum_pack), SS_METHOD(majority_vote), SS_METHOD(vote_sum), SS_METHOD(sign_apply), SS_METHOD(sum_apply),
    SS_METHOD(signum_vote_step), SS_METHOD(stream_copy), SS_METHOD(welford_update), SS_METHOD(welford_sigma),
    SS_METHOD(density), SS_METHOD(signum_pack_ternary), SS_METHOD(quorum_vote), SS_METHOD(ternary_apply),
    SS_METHOD(signum_vote_step_ternary), {nullptr, nullptr, 0, nullptr}};
#undef SS_METHOD

PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_marshal", "torch tensors to the C ABI of libsignsgd.so", -1, kMethods,
                       nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal(void) { return PyModule_Create(&kModule); }
