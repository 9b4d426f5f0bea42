// Argument marshalling of the Python calls that a program makes over and over, in native code.
//
// A call on few rows is shorter on the device (4 to 6 us) than its way through the Python binding was (3.6 us of checks and
// ctypes, 1.5 for the result, 2.5 for the launch), so that the host bound it: 1000 rows of 320 floats, C = 16, M = 128 took 8.0 us a
// call whatever the kernel did.  These functions take the tensors apart through torch's C++ interface and call the same entry
// points of libmaddness.  They look at the usual arguments only - plain tensors on the device, of the type and shape the
// call wants - and return NotImplemented for anything else, after which the Python code does the call, or raises.
// A status other than MADDNESS_OK comes back as a number.
#include <Python.h>

#include <ATen/ops/empty.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstdio>
#include <cstring>

#include "maddness.h"

namespace {

struct NotUsual {};

PyObject *s_split_dims, *s_thresholds, *s_prototypes, *s_C, *s_D, *s_cuda_stream;
PyObject *get_stream, *get_device;     // torch._C._cuda_getCurrentRawStream, _cuda_getDevice
PyObject *int_status(int rc) { return PyLong_FromLong(rc); }

// A new reference that ends with the scope.
struct Ref {
    PyObject *p;
    explicit Ref(PyObject *o) : p(o)
    {
        if (!p) {
            PyErr_Clear();
            throw NotUsual();
        }
    }
    ~Ref() { Py_DECREF(p); }
    Ref(const Ref &) = delete;
};

const at::Tensor &tensor(PyObject *o)
{
    if (!THPVariable_CheckExact(o)) throw NotUsual();
    const at::Tensor &t = THPVariable_Unpack(o);
    if (!t.is_cuda() || t.layout() != at::kStrided) throw NotUsual();
    return t;
}

template <typename T>
T *pointer(PyObject *o, at::ScalarType type)
{
    if (o == Py_None) return nullptr;
    const at::Tensor &t = tensor(o);
    if (t.scalar_type() != type) throw NotUsual();
    return static_cast<T *>(t.data_ptr());
}

uint16_t *sums(PyObject *o)
{
    if (o == Py_None) return nullptr;
    const at::Tensor &t = tensor(o);
    if (t.scalar_type() != at::kShort && t.scalar_type() != at::kUInt16) throw NotUsual();
    return static_cast<uint16_t *>(t.data_ptr());
}

struct Rows {
    int64_t rows, cols, ld;
};

// rows, columns and row stride of a matrix whose rows are contiguous
Rows rows_of(const at::Tensor &t)
{
    if (t.dim() != 2) throw NotUsual();
    const int64_t r = t.size(0), c = t.size(1), s = t.stride(0);
    if (c > 1 && t.stride(1) != 1) throw NotUsual();
    return {r, c, r > 1 ? s : std::max(c, s)};
}

int64_t whole(PyObject *o)
{
    if (!PyLong_CheckExact(o)) throw NotUsual();
    const int64_t v = PyLong_AsLongLong(o);
    if (v == -1 && PyErr_Occurred()) {
        PyErr_Clear();
        throw NotUsual();
    }
    return v;
}

void *stream_of(PyObject *stream)
{
    if (stream != Py_None) {
        Ref raw(PyObject_GetAttr(stream, s_cuda_stream));
        return reinterpret_cast<void *>(whole(raw.p));
    }
    Ref device(PyObject_CallNoArgs(get_device));
    Ref raw(PyObject_CallOneArg(get_stream, device.p));
    return reinterpret_cast<void *>(whole(raw.p));
}

// The trees (and D where the parameters know it) of a Params object.
maddness_params params_of(PyObject *o, int64_t D)
{
    maddness_params p{};
    Ref C(PyObject_GetAttr(o, s_C)), split(PyObject_GetAttr(o, s_split_dims)), th(PyObject_GetAttr(o, s_thresholds)),
        proto(PyObject_GetAttr(o, s_prototypes));
    const int64_t c = whole(C.p);
    if (D > INT32_MAX || c > INT32_MAX || c < INT32_MIN) throw NotUsual();
    p.D = (int32_t)D;
    p.C = (int32_t)c;
    p.split_dims = pointer<int32_t>(split.p, at::kInt);
    p.thresholds = pointer<float>(th.p, at::kFloat);
    p.prototypes = pointer<float>(proto.p, at::kFloat);
    return p;
}

int64_t own_D(PyObject *o)
{
    Ref d(PyObject_GetAttr(o, s_D));
    return d.p == Py_None ? -1 : whole(d.p);
}

int32_t narrow(int64_t v)
{
    if (v > INT32_MAX || v < INT32_MIN) throw NotUsual();
    return (int32_t)v;
}

bool truth(PyObject *o)
{
    if (o != Py_True && o != Py_False) throw NotUsual();
    return o == Py_True;
}

int type_of(const at::Tensor &t)
{
    switch (t.scalar_type()) {
    case at::kFloat: return MADDNESS_F32;
    case at::kHalf: return MADDNESS_F16;
    case at::kBFloat16: return MADDNESS_BF16;
    case at::kByte: return MADDNESS_U8;
    default: throw NotUsual();
    }
}

int64_t columns_of_tables(PyObject *luts)
{
    const at::Tensor &t = tensor(luts);
    if (t.dim() != 3) throw NotUsual();
    return t.size(2);
}

// Runs f; whatever is not usual, or goes wrong before the library is called, is left to the Python code.
template <typename F>
PyObject *usual(F f)
{
    try {
        return f();
    } catch (...) {
        PyErr_Clear();
        Py_RETURN_NOTIMPLEMENTED;
    }
}

// (kind, col_major, params, A, luts, scale, offset, out, acc, codes, want_out, stream); kind 0: fp32 rows, 1: fp32 rows and
// averages, 2: typed
PyObject *encode_scan(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return usual([&]() -> PyObject * {
        if (n != 12) throw NotUsual();
        const int64_t kind = whole(a[0]);
        const bool col_major = truth(a[1]);
        const at::Tensor &A = tensor(a[3]);
        const int dtype = type_of(A);
        if (kind != 2 && dtype != MADDNESS_F32) throw NotUsual();
        const Rows ra = rows_of(A);
        const int64_t N = col_major ? ra.cols : ra.rows, D = col_major ? ra.rows : ra.cols;
        const int32_t M = narrow(columns_of_tables(a[4]));
        const maddness_params p = params_of(a[2], D);
        const void *A_p = A.data_ptr();
        const uint8_t *luts = pointer<uint8_t>(a[4], at::kByte);
        const float *scale = pointer<float>(a[5], at::kFloat), *offset = pointer<float>(a[6], at::kFloat);
        uint16_t *acc = sums(a[8]);
        uint8_t *codes = pointer<uint8_t>(a[9], at::kByte);
        void *stream = stream_of(a[11]);
        at::Tensor made;
        float *out = nullptr;
        int64_t ldo = 0;
        if (a[7] != Py_None) {
            out = pointer<float>(a[7], at::kFloat);
            ldo = rows_of(tensor(a[7])).ld;
        } else if (truth(a[10])) {
            made = at::empty({N, M}, at::TensorOptions().dtype(at::kFloat).device(A.device()));
            out = static_cast<float *>(made.data_ptr());
            ldo = rows_of(made).ld;
        }
        int rc;
        Py_BEGIN_ALLOW_THREADS
        if (kind == 2)
            rc = maddness_encode_scan_typed(&p, A_p, dtype, col_major ? MADDNESS_COL_MAJOR : MADDNESS_ROW_MAJOR, N, ra.ld, M, luts, scale,
                                            offset, out, ldo, acc, codes, stream);
        else if (kind == 1)
            rc = maddness_encode_scan_averaged(&p, static_cast<const float *>(A_p), N, ra.ld, M, luts, scale, offset, out, ldo, acc, codes,
                                               stream);
        else
            rc = maddness_encode_scan(&p, static_cast<const float *>(A_p), N, ra.ld, M, luts, scale, offset, out, ldo, acc, codes, stream);
        Py_END_ALLOW_THREADS
        if (rc != MADDNESS_OK) return int_status(rc);
        if (made.defined()) return THPVariable_Wrap(std::move(made));
        Py_INCREF(a[7]);
        return a[7];
    });
}

// (kind, col_major, params, A, codes, stream); kind 0: fp32 rows, 2: typed
PyObject *encode(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return usual([&]() -> PyObject * {
        if (n != 6) throw NotUsual();
        const int64_t kind = whole(a[0]);
        const bool col_major = truth(a[1]);
        const at::Tensor &A = tensor(a[3]);
        const int dtype = type_of(A);
        if (kind != 2 && dtype != MADDNESS_F32) throw NotUsual();
        const Rows ra = rows_of(A);
        const int64_t N = col_major ? ra.cols : ra.rows, D = col_major ? ra.rows : ra.cols, known = own_D(a[2]);
        if (known != -1 && known != D) throw NotUsual();
        const maddness_params p = params_of(a[2], D);
        const void *A_p = A.data_ptr();
        void *stream = stream_of(a[5]);
        at::Tensor made;
        uint8_t *codes;
        if (a[4] != Py_None) {
            codes = pointer<uint8_t>(a[4], at::kByte);
        } else {
            made = at::empty({N, ((int64_t)p.C + 1) / 2}, at::TensorOptions().dtype(at::kByte).device(A.device()));
            codes = static_cast<uint8_t *>(made.data_ptr());
        }
        int rc;
        Py_BEGIN_ALLOW_THREADS
        rc = kind == 2 ? maddness_encode_typed(&p, A_p, dtype, col_major ? MADDNESS_COL_MAJOR : MADDNESS_ROW_MAJOR, N, ra.ld, codes, stream)
                       : maddness_encode(&p, static_cast<const float *>(A_p), N, ra.ld, codes, stream);
        Py_END_ALLOW_THREADS
        if (rc != MADDNESS_OK) return int_status(rc);
        if (made.defined()) return THPVariable_Wrap(std::move(made));
        Py_INCREF(a[4]);
        return a[4];
    });
}

// (averaged, n_codebooks, codes, luts, scale, offset, out, acc, want_out, stream) -> out
PyObject *scan(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return usual([&]() -> PyObject * {
        if (n != 10) throw NotUsual();
        const bool averaged = truth(a[0]);
        const int32_t C = narrow(whole(a[1]));
        const at::Tensor &codes = tensor(a[2]);
        if (codes.dim() < 1) throw NotUsual();
        const int64_t N = codes.size(0);
        const int32_t M = narrow(columns_of_tables(a[3]));
        const uint8_t *codes_p = pointer<uint8_t>(a[2], at::kByte), *luts = pointer<uint8_t>(a[3], at::kByte);
        const float *scale = pointer<float>(a[4], at::kFloat), *offset = pointer<float>(a[5], at::kFloat);
        uint16_t *acc = sums(a[7]);
        void *stream = stream_of(a[9]);
        at::Tensor made;
        float *out = nullptr;
        int64_t ldo = 0;
        if (a[6] != Py_None) {
            out = pointer<float>(a[6], at::kFloat);
            ldo = rows_of(tensor(a[6])).ld;
        } else if (truth(a[8])) {
            made = at::empty({N, M}, at::TensorOptions().dtype(at::kFloat).device(codes.device()));
            out = static_cast<float *>(made.data_ptr());
            ldo = rows_of(made).ld;
        }
        int rc;
        Py_BEGIN_ALLOW_THREADS
        rc = averaged ? maddness_scan_averaged(C, M, codes_p, N, luts, scale, offset, out, ldo, acc, stream)
                      : maddness_scan(C, M, codes_p, N, luts, scale, offset, out, ldo, acc, stream);
        Py_END_ALLOW_THREADS
        if (rc != MADDNESS_OK) return int_status(rc);
        if (made.defined()) return THPVariable_Wrap(std::move(made));
        Py_INCREF(a[6]);
        return a[6];
    });
}

// (pooled, params, B, luts, scale, offset, workspace, stream) -> (luts, scale, offset)
PyObject *build_luts(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return usual([&]() -> PyObject * {
        if (n != 8) throw NotUsual();
        const bool pooled = truth(a[0]);
        const at::Tensor &B = tensor(a[2]);
        const Rows rb = rows_of(B);
        if (own_D(a[1]) != rb.rows) throw NotUsual();
        const maddness_params p = params_of(a[1], rb.rows);
        const int32_t M = narrow(rb.cols);
        const float *B_p = pointer<float>(a[2], at::kFloat);
        void *stream = stream_of(a[7]);
        const auto bytes = at::TensorOptions().dtype(at::kByte).device(B.device()), floats = bytes.dtype(at::kFloat);
        const at::Tensor luts = a[3] == Py_None ? at::empty({p.C, 16, M}, bytes) : tensor(a[3]);
        const at::Tensor scale = a[4] == Py_None ? at::empty({M}, floats) : tensor(a[4]);
        const at::Tensor offset = a[5] == Py_None ? at::empty({M}, floats) : tensor(a[5]);
        const at::Tensor work = a[6] == Py_None ? at::empty({(int64_t)maddness_build_luts_workspace(p.D, p.C, M)}, bytes) : tensor(a[6]);
        if (luts.scalar_type() != at::kByte || scale.scalar_type() != at::kFloat || offset.scalar_type() != at::kFloat ||
            work.scalar_type() != at::kByte)
            throw NotUsual();
        uint8_t *luts_p = static_cast<uint8_t *>(luts.data_ptr());
        float *scale_p = static_cast<float *>(scale.data_ptr()), *offset_p = static_cast<float *>(offset.data_ptr());
        void *work_p = work.data_ptr();
        const size_t work_bytes = (size_t)work.numel();
        int rc;
        Py_BEGIN_ALLOW_THREADS
        rc = (pooled ? maddness_build_luts_pooled : maddness_build_luts)(&p, B_p, M, rb.ld, luts_p, scale_p, offset_p, work_p, work_bytes,
                                                                         stream);
        Py_END_ALLOW_THREADS
        if (rc != MADDNESS_OK) return int_status(rc);
        PyObject *three[3];
        for (int k = 0; k < 3; ++k) {
            if (a[3 + k] == Py_None) {
                three[k] = THPVariable_Wrap(k == 0 ? luts : k == 1 ? scale : offset);
            } else {
                Py_INCREF(a[3 + k]);
                three[k] = a[3 + k];
            }
        }
        PyObject *tuple = PyTuple_New(3);
        for (int k = 0; k < 3; ++k) PyTuple_SET_ITEM(tuple, k, three[k]);
        return tuple;
    });
}

// Tensors are read by the layout of the torch, and objects by that of the Python, that this was built with: with others it is an
// ImportError, also where every symbol is found.
bool built_for_these()
{
    PyObject *torch = PyImport_ImportModule("torch");
    PyObject *version = torch ? PyObject_GetAttrString(torch, "__version__") : nullptr;
    const char *have = version ? PyUnicode_AsUTF8(version) : nullptr;
    char python[32];
    std::snprintf(python, sizeof python, "%d.%d.", PY_MAJOR_VERSION, PY_MINOR_VERSION);
    const bool same = have && std::strcmp(have, MADDNESS_TORCH_VERSION) == 0 && std::strncmp(Py_GetVersion(), python, std::strlen(python)) == 0;
    if (!same && !PyErr_Occurred())
        PyErr_Format(PyExc_ImportError, "built for torch %s and Python %s, this is torch %s and Python %s", MADDNESS_TORCH_VERSION, PY_VERSION,
                     have, Py_GetVersion());
    Py_XDECREF(version);
    Py_XDECREF(torch);
    return same;
}

PyMethodDef methods[] = {
    {"encode_scan", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(encode_scan)), METH_FASTCALL, nullptr},
    {"encode", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(encode)), METH_FASTCALL, nullptr},
    {"scan", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(scan)), METH_FASTCALL, nullptr},
    {"build_luts", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(build_luts)), METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr},
};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "maddness_binding", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit_maddness_binding()
{
    s_split_dims = PyUnicode_InternFromString("split_dims");
    s_thresholds = PyUnicode_InternFromString("thresholds");
    s_prototypes = PyUnicode_InternFromString("prototypes");
    s_C = PyUnicode_InternFromString("C");
    s_D = PyUnicode_InternFromString("D");
    s_cuda_stream = PyUnicode_InternFromString("cuda_stream");
    if (!built_for_these()) return nullptr;
    PyObject *torch_c = PyImport_ImportModule("torch._C");
    if (!torch_c) return nullptr;
    get_stream = PyObject_GetAttrString(torch_c, "_cuda_getCurrentRawStream");
    get_device = PyObject_GetAttrString(torch_c, "_cuda_getDevice");
    Py_DECREF(torch_c);
    if (!get_stream || !get_device) return nullptr;
    return PyModule_Create(&module);
}
