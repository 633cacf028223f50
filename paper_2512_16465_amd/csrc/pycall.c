/* The three gemm_run entry points of the Python binding as vector calls: the arguments go from Python integers and floats straight to the
 * C ABI.  Through ctypes a call whose kernel is shorter than the host's part takes 8.1 us (1x4096x4096 with the weight stored N x K, 832x512x768:
 * 8.07 and 8.32), so 6.6 to 6.9.  The semantics are those of the ctypes functions in binding.py, which take every call that is not made of plain ints, floats and an epilogue (and
 * the first one, which loads the library): their conversions, errors and messages stay the reference. */
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <stdint.h>

typedef int (*run_fn)(void*, int64_t, int64_t, int64_t, int, int, int, float, const void*, int64_t, const void*, int64_t, float, void*,
                      int64_t, const void*, void*);
typedef int (*batched_fn)(void*, int64_t, int64_t, int64_t, int64_t, int, int, int, float, const void*, int64_t, int64_t, const void*,
                          int64_t, int64_t, float, void*, int64_t, int64_t, const void*, void*);

#define MAX_ARGS 22

/* one letter per argument: p pointer, q 64-bit integer, i int, f float, e epilogue, c check */
typedef struct {
    const char* name;
    const char* kinds;
    int required;
    const char* names[MAX_ARGS];
    PyObject* interned[MAX_ARGS];
} entry_t;

static entry_t entries[3] = {
    {"gemm_run", "pqqqiiifpqpqfpqepc", 15,
     {"handle", "M", "N", "K", "transA", "transB", "dtype", "alpha", "A", "lda", "B", "ldb", "beta", "C", "ldc", "epilogue", "stream", "check"}, {0}},
    {"gemm_run_noalloc", "pqqqiiifpqpqfpqepc", 15,
     {"handle", "M", "N", "K", "transA", "transB", "dtype", "alpha", "A", "lda", "B", "ldb", "beta", "C", "ldc", "epilogue", "stream", "check"}, {0}},
    {"gemm_run_batched", "pqqqqiiifpqqpqqfpqqepc", 19,
     {"handle", "batch", "M", "N", "K", "transA", "transB", "dtype", "alpha", "A", "lda", "strideA", "B", "ldb", "strideB", "beta", "C", "ldc",
      "strideC", "epilogue", "stream", "check"}, {0}},
};

static PyObject *binding_dict, *key_lib, *error_class, *slow[3], *addresses_of, *bound_lib;
static PyTypeObject* epilogue_type;
static void* address[3];

/* 0 when `binding._lib` is the library whose addresses are held */
static int library_changed(void) {
    PyObject* lib = PyDict_GetItemWithError(binding_dict, key_lib);
    return lib == NULL || lib == Py_None || lib != bound_lib;
}

static PyObject* take_slow(int which, PyObject* const* args, Py_ssize_t nargs, PyObject* kwnames) {
    PyObject* result = PyObject_Vectorcall(slow[which], args, (size_t)nargs, kwnames);
    if (result && library_changed()) {
        PyObject* lib = PyDict_GetItemWithError(binding_dict, key_lib);
        if (lib && lib != Py_None) {
            PyObject* t = PyObject_CallFunctionObjArgs(addresses_of, lib, NULL);
            if (!t || !PyTuple_Check(t) || PyTuple_GET_SIZE(t) != 3) { Py_XDECREF(t); Py_DECREF(result); return NULL; }
            for (int i = 0; i < 3; ++i) address[i] = PyLong_AsVoidPtr(PyTuple_GET_ITEM(t, i));
            Py_DECREF(t);
            if (PyErr_Occurred()) { Py_DECREF(result); return NULL; }
            Py_INCREF(lib);
            Py_XSETREF(bound_lib, lib);
        }
    }
    return result;
}

static PyObject* call(int which, PyObject* const* args, Py_ssize_t nargs, PyObject* kwnames) {
    const entry_t* e = &entries[which];
    PyObject* arg[MAX_ARGS];
    const int count = (int)strlen(e->kinds);
    if (nargs > count || library_changed()) return take_slow(which, args, nargs, kwnames);
    for (int i = 0; i < count; ++i) arg[i] = i < nargs ? args[i] : NULL;
    if (kwnames) {
        const Py_ssize_t n = PyTuple_GET_SIZE(kwnames);
        for (Py_ssize_t k = 0; k < n; ++k) {
            int at = -1;
            for (int i = 0; i < count && at < 0; ++i)
                if (PyTuple_GET_ITEM(kwnames, k) == e->interned[i]) at = i;
            if (at < 0 || arg[at]) return take_slow(which, args, nargs, kwnames);      /* (unknown, twice, or not interned) */
            arg[at] = args[nargs + k];
        }
    }
    union { int64_t q; void* p; int i; float f; } v[MAX_ARGS];
    Py_buffer view;
    const void* epilogue = NULL;
    int check = 1, held = 0;
    for (int i = 0; i < count; ++i) {
        PyObject* o = arg[i];
        if (!o) {
            if (i < e->required) return take_slow(which, args, nargs, kwnames);
            v[i].p = NULL;
            continue;
        }
        switch (e->kinds[i]) {
            case 'p':
                if (o == Py_None) v[i].p = NULL;
                else if (PyLong_CheckExact(o)) v[i].p = (void*)(uintptr_t)PyLong_AsUnsignedLongLongMask(o);
                else goto other;
                break;
            case 'q':
                if (!PyLong_CheckExact(o)) goto other;
                v[i].q = (int64_t)PyLong_AsUnsignedLongLongMask(o);
                break;
            case 'i':
                if (!PyLong_CheckExact(o)) goto other;
                v[i].i = (int)PyLong_AsUnsignedLongMask(o);
                break;
            case 'f':
                if (!PyFloat_CheckExact(o)) goto other;
                v[i].f = (float)PyFloat_AS_DOUBLE(o);
                break;
            case 'e':
                if (o == Py_None) break;
                if (Py_TYPE(o) != epilogue_type || held) goto other;
                if (PyObject_GetBuffer(o, &view, PyBUF_SIMPLE) != 0) { PyErr_Clear(); goto other; }
                held = 1;
                epilogue = view.buf;
                break;
            default:
                check = PyObject_IsTrue(o);
                if (check < 0) goto other;
        }
    }
    int status;
    Py_BEGIN_ALLOW_THREADS
    if (which == 2) {
        status = ((batched_fn)address[2])(v[0].p, v[1].q, v[2].q, v[3].q, v[4].q, v[5].i, v[6].i, v[7].i, v[8].f, v[9].p, v[10].q, v[11].q,
                                          v[12].p, v[13].q, v[14].q, v[15].f, v[16].p, v[17].q, v[18].q, epilogue, v[20].p);
    } else {
        status = ((run_fn)address[which])(v[0].p, v[1].q, v[2].q, v[3].q, v[4].i, v[5].i, v[6].i, v[7].f, v[8].p, v[9].q, v[10].p, v[11].q,
                                          v[12].f, v[13].p, v[14].q, epilogue, v[16].p);
    }
    Py_END_ALLOW_THREADS
    if (held) PyBuffer_Release(&view);
    if (check && status != 0) {
        PyObject* error = PyObject_CallFunction(error_class, "is", status, e->name);
        if (error) {
            PyErr_SetObject(error_class, error);
            Py_DECREF(error);
        }
        return NULL;
    }
    return PyLong_FromLong(status);
other:
    if (held) PyBuffer_Release(&view);
    PyErr_Clear();
    return take_slow(which, args, nargs, kwnames);
}

static PyObject* run(PyObject* self, PyObject* const* args, Py_ssize_t nargs, PyObject* kwnames) { (void)self; return call(0, args, nargs, kwnames); }
static PyObject* noalloc(PyObject* self, PyObject* const* args, Py_ssize_t nargs, PyObject* kwnames) { (void)self; return call(1, args, nargs, kwnames); }
static PyObject* batched(PyObject* self, PyObject* const* args, Py_ssize_t nargs, PyObject* kwnames) { (void)self; return call(2, args, nargs, kwnames); }

/* setup(binding.__dict__, gemm_epilogue_t, GemmError, (the three ctypes functions), lib -> the three addresses) */
static PyObject* setup(PyObject* self, PyObject* args) {
    (void)self;
    PyObject *dict, *type, *error, *functions, *addresses;
    if (!PyArg_ParseTuple(args, "O!O!OO!O", &PyDict_Type, &dict, &PyType_Type, &type, &error, &PyTuple_Type, &functions, &addresses)) return NULL;
    if (PyTuple_GET_SIZE(functions) != 3) { PyErr_SetString(PyExc_TypeError, "setup"); return NULL; }
    Py_INCREF(dict); Py_INCREF(type); Py_INCREF(error); Py_INCREF(addresses);
    binding_dict = dict; epilogue_type = (PyTypeObject*)type; error_class = error; addresses_of = addresses;
    key_lib = PyUnicode_InternFromString("_lib");
    for (int i = 0; i < 3; ++i) {
        slow[i] = PyTuple_GET_ITEM(functions, i);
        Py_INCREF(slow[i]);
        for (size_t k = 0; k < strlen(entries[i].kinds); ++k) entries[i].interned[k] = PyUnicode_InternFromString(entries[i].names[k]);
    }
    Py_RETURN_NONE;
}

static PyMethodDef methods[] = {
    {"gemm_run", (PyCFunction)(void (*)(void))run, METH_FASTCALL | METH_KEYWORDS,
     "gemm_run(handle, M, N, K, transA, transB, dtype, alpha, A, lda, B, ldb, beta, C, ldc, epilogue=None, stream=0, check=True)\n--\n\n"
     "A, B, C, epilogue.bias are device addresses (e.g. tensor.data_ptr()); stream is a hipStream_t as an integer.  Returns the status; "
     "raises GemmError unless check is False."},
    {"gemm_run_noalloc", (PyCFunction)(void (*)(void))noalloc, METH_FASTCALL | METH_KEYWORDS,
     "gemm_run_noalloc(handle, M, N, K, transA, transB, dtype, alpha, A, lda, B, ldb, beta, C, ldc, epilogue=None, stream=0, check=True)\n--\n\n"
     "gemm_run with the split-K scratch in the library's static device buffer: allocates nothing."},
    {"gemm_run_batched", (PyCFunction)(void (*)(void))batched, METH_FASTCALL | METH_KEYWORDS,
     "gemm_run_batched(handle, batch, M, N, K, transA, transB, dtype, alpha, A, lda, strideA, B, ldb, strideB, beta, C, ldc, strideC, "
     "epilogue=None, stream=0, check=True)\n--\n\n"
     "`batch` products of one shape; matrix b of each operand starts b * stride elements after the first one."},
    {"setup", setup, METH_VARARGS, NULL},
    {NULL, NULL, 0, NULL},
};

static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_pycall", NULL, -1, methods, NULL, NULL, NULL, NULL};

PyMODINIT_FUNC PyInit__pycall(void) { return PyModule_Create(&module); }
