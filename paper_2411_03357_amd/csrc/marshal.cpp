// Argument marshalling of the batch calls for the Python binding: the common case (descriptor arrays
// that already are contiguous numpy arrays of the right type, device memory as CUDA tensors or
// addresses) in one native step.  A call on a few chunks takes the GPU under 10 us, and converting
// nine arguments in Python took as long.  Anything unusual is left to the Python code: the
// functions return None then, having done nothing.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <stdint.h>

namespace {

// names looked up on every call
PyObject *s_is_cuda, *s_is_contiguous, *s_data_ptr, *s_handle;

// the C entry points, by address
typedef int (*encrypt_fn)(void*, size_t, const void*, uint32_t, const void*, const void*,
                          const void*, const void*, const void*, void*, void*);
typedef int (*decrypt_fn)(void*, size_t, const void*, uint32_t, const void*, const void*,
                          const void*, const void*, const void*, const void*, void*, void*);
encrypt_fn g_encrypt;
decrypt_fn g_decrypt;

// A one-dimensional contiguous buffer of n unsigned items of `size` bytes; None is NULL.
class Array {
  public:
    ~Array() {
        if (held_) PyBuffer_Release(&view_);
    }
    bool take(PyObject* o, Py_ssize_t n, Py_ssize_t size) {
        if (o == Py_None) return true;
        if (PyObject_GetBuffer(o, &view_, PyBUF_FORMAT | PyBUF_ND | PyBUF_C_CONTIGUOUS) != 0) {
            PyErr_Clear();
            return false;
        }
        held_ = true;
        const char* f = view_.format;
        if (f == nullptr || f[0] == '\0' || f[1] != '\0') return false;
        const bool unsigned_int = f[0] == 'I' || f[0] == 'L' || f[0] == 'Q';
        ptr_ = view_.buf;
        return unsigned_int && view_.itemsize == size && view_.ndim == 1 &&
               (n < 0 || view_.shape[0] == n);
    }
    const void* ptr() const { return ptr_; }
    Py_ssize_t count() const { return held_ ? view_.shape[0] : -1; }

  private:
    Py_buffer view_;
    bool held_ = false;
    const void* ptr_ = nullptr;
};

// device address of an int, of None (NULL) or of a contiguous CUDA tensor
bool device_address(PyObject* o, void** out) {
    if (o == Py_None) {
        *out = nullptr;
        return true;
    }
    PyObject* value = nullptr;
    if (PyLong_CheckExact(o)) {
        Py_INCREF(o);
        value = o;
    } else {
        PyObject* cuda = PyObject_GetAttr(o, s_is_cuda);
        const bool on_gpu = cuda == Py_True;
        Py_XDECREF(cuda);
        if (on_gpu) {
            PyObject* contiguous = PyObject_CallMethodNoArgs(o, s_is_contiguous);
            if (contiguous == Py_True) value = PyObject_CallMethodNoArgs(o, s_data_ptr);
            Py_XDECREF(contiguous);
        }
    }
    bool ok = false;
    if (value != nullptr) {
        *out = PyLong_AsVoidPtr(value);
        ok = PyErr_Occurred() == nullptr;
        Py_DECREF(value);
    }
    PyErr_Clear();
    return ok;
}

// (key, ivs, iv_bytes, aad, aad_len, src, length, dst, tags[, ok], stream) -> status or None
PyObject* batch(PyObject* const* args, Py_ssize_t nargs, bool decrypt) {
    if (nargs != (decrypt ? 11 : 10)) {
        PyErr_SetString(PyExc_TypeError, "wrong number of arguments");
        return nullptr;
    }
    void *key, *ivs, *tags, *ok = nullptr, *stream;
    PyObject* handle = PyObject_GetAttr(args[0], s_handle);
    if (handle == nullptr || !PyLong_CheckExact(handle)) {
        PyErr_Clear();
        Py_XDECREF(handle);
        Py_RETURN_NONE;
    }
    key = PyLong_AsVoidPtr(handle);
    Py_DECREF(handle);
    const long iv_bytes = PyLong_AsLong(args[2]);
    if (PyErr_Occurred() || iv_bytes < 0 || iv_bytes > 0x7FFFFFFF) {
        PyErr_Clear();
        Py_RETURN_NONE;
    }
    Array len, src, dst, aad, aad_len;
    if (args[6] == Py_None || !len.take(args[6], -1, 8)) Py_RETURN_NONE;
    const Py_ssize_t n = len.count();
    if (!src.take(args[5], n, 8) || !dst.take(args[7], n, 8) || !aad.take(args[3], n, 8) ||
        !aad_len.take(args[4], n, 4) || !device_address(args[1], &ivs) ||
        !device_address(args[8], &tags) || (decrypt && !device_address(args[9], &ok)) ||
        !device_address(args[nargs - 1], &stream))
        Py_RETURN_NONE;
    int status;
    Py_BEGIN_ALLOW_THREADS
    status = decrypt ? g_decrypt(key, (size_t)n, ivs, (uint32_t)iv_bytes, aad.ptr(), aad_len.ptr(),
                                 src.ptr(), len.ptr(), dst.ptr(), tags, ok, stream)
                     : g_encrypt(key, (size_t)n, ivs, (uint32_t)iv_bytes, aad.ptr(), aad_len.ptr(),
                                 src.ptr(), len.ptr(), dst.ptr(), tags, stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(status);
}

PyObject* encrypt_batch(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
    return batch(args, nargs, false);
}
PyObject* decrypt_verify_batch(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
    return batch(args, nargs, true);
}

// bind(address of pgcm_encrypt_batch_iv, address of pgcm_decrypt_verify_batch_iv)
PyObject* bind(PyObject*, PyObject* args) {
    PyObject *e, *d;
    if (!PyArg_ParseTuple(args, "OO", &e, &d)) return nullptr;
    g_encrypt = reinterpret_cast<encrypt_fn>(PyLong_AsVoidPtr(e));
    g_decrypt = reinterpret_cast<decrypt_fn>(PyLong_AsVoidPtr(d));
    if (PyErr_Occurred()) return nullptr;
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"bind", bind, METH_VARARGS, nullptr},
    {"encrypt_batch", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(encrypt_batch)),
     METH_FASTCALL, nullptr},
    {"decrypt_verify_batch",
     reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(decrypt_verify_batch)),
     METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods,
                      nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal(void) {
    s_is_cuda = PyUnicode_InternFromString("is_cuda");
    s_is_contiguous = PyUnicode_InternFromString("is_contiguous");
    s_data_ptr = PyUnicode_InternFromString("data_ptr");
    s_handle = PyUnicode_InternFromString("_h");
    if (!s_is_cuda || !s_is_contiguous || !s_data_ptr || !s_handle) return nullptr;
    return PyModule_Create(&module);
}
