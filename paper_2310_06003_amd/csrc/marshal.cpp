// CPython extension: argument marshalling for the device calls, which a training program makes every step.
//
// What bounds a small step is the host (one launch over 2^18 elements: the GPU works 3.4 us).  ctypes makes an array object
// per call for the contribution pointers and a conversion object per argument: a step of one launch 5.9 us, of two 9.7; with
// this extension 4.9 and 8.9.  Here the usual call - positional arguments, plain ints, a list or tuple of addresses - is read straight into C
// variables.  Anything else (keywords, None, numpy integers, ctypes objects, wrong types, a closed plan) goes to the
// ctypes function of the same name, unchanged, which accepts or refuses it as ever.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <dlfcn.h>

#include <climits>
#include <cstdint>
#include <cstring>

#include "paro.h"

namespace {

PyObject *g_plan_type, *g_handle_type, *g_adam_type, *g_check;      // the binding's classes, and its check of a status code
PyObject *g_handle_name;

// One argument of a call.
union Arg {
    void *ptr;
    int64_t num;
};
struct Args {
    Arg a[14];
    const void *contrib[PARO_MAX_RANKS];
    paro_adam_t hp;
};

// Copies `bytes` from an object that lies in memory as its C type does.
bool copy_out(PyObject *o, void *to, size_t bytes) {
    Py_buffer view;
    if (PyObject_GetBuffer(o, &view, PyBUF_SIMPLE) != 0) {
        PyErr_Clear();
        return false;
    }
    const bool fits = view.len == (Py_ssize_t)bytes;
    if (fits) std::memcpy(to, view.buf, bytes);
    PyBuffer_Release(&view);
    return fits;
}

bool address(PyObject *o, void **to) {
    if (!PyLong_CheckExact(o)) return false;
    const unsigned long long x = PyLong_AsUnsignedLongLong(o);
    if (x == (unsigned long long)-1 && PyErr_Occurred()) {
        PyErr_Clear();
        return false;
    }
    *to = reinterpret_cast<void *>((uintptr_t)x);
    return true;
}

bool number(PyObject *o, int64_t lo, int64_t hi, int64_t *to) {
    if (!PyLong_CheckExact(o)) return false;
    int overflow;
    const long long x = PyLong_AsLongLongAndOverflow(o, &overflow);
    if (overflow || x < lo || x > hi) return false;
    *to = x;
    return true;
}

bool addresses(PyObject *o, const void **to) {
    const bool list = PyList_CheckExact(o);
    if (!list && !PyTuple_CheckExact(o)) return false;
    const Py_ssize_t n = list ? PyList_GET_SIZE(o) : PyTuple_GET_SIZE(o);
    if (n > PARO_MAX_RANKS) return false;
    for (Py_ssize_t i = 0; i < n; ++i) {
        void *p;
        if (!address(list ? PyList_GET_ITEM(o, i) : PyTuple_GET_ITEM(o, i), &p)) return false;
        to[i] = p;
    }
    for (Py_ssize_t i = n; i < PARO_MAX_RANKS; ++i) to[i] = nullptr;     // a list too short for its plan is refused by the library
    return true;
}

bool plan_of(PyObject *o, void **to) {
    if ((PyObject *)Py_TYPE(o) != g_plan_type) return false;
    PyObject *handle = PyObject_GetAttr(o, g_handle_name);
    if (!handle) {
        PyErr_Clear();
        return false;
    }
    const bool ok = (PyObject *)Py_TYPE(handle) == g_handle_type && copy_out(handle, to, sizeof(void *)) && *to;
    Py_DECREF(handle);
    return ok;
}

// kinds: P plan, i int, n int64_t, c contribution (or buffer) addresses, h hyper-parameters, p address
bool parse(const char *kinds, PyObject *const *args, Py_ssize_t n, Args *out) {
    for (Py_ssize_t k = 0; kinds[k]; ++k) {
        Arg *a = &out->a[k];
        a->ptr = nullptr;
        if (k >= n) continue;                               // left out: the trailing arguments default to 0
        PyObject *o = args[k];
        bool ok = false;
        switch (kinds[k]) {
            case 'P': ok = plan_of(o, &a->ptr); break;
            case 'i': ok = number(o, INT_MIN, INT_MAX, &a->num); break;
            case 'n': ok = number(o, INT64_MIN, INT64_MAX, &a->num); break;
            case 'c': ok = addresses(o, out->contrib); break;
            case 'h': ok = (PyObject *)Py_TYPE(o) == g_adam_type && copy_out(o, &out->hp, sizeof(out->hp)); break;
            case 'p': ok = address(o, &a->ptr); break;
        }
        if (!ok) return false;
    }
    return true;
}

// The calls.  fn: the function's address in the library that the binding has loaded.
template <class T>
T *at(const Arg &a) {
    return static_cast<T *>(a.ptr);
}
int64_t call_reduce(void *fn, Args &x) {
    return reinterpret_cast<decltype(&paro_reduce_shard)>(fn)(at<paro_plan_t>(x.a[0]), (int)x.a[1].num, x.contrib, (int)x.a[3].num,
                                                              at<float>(x.a[4]), at<double>(x.a[5]), x.a[6].ptr);
}
int64_t call_adam(void *fn, Args &x) {
    return reinterpret_cast<decltype(&paro_adam_shard)>(fn)(at<paro_plan_t>(x.a[0]), (int)x.a[1].num, &x.hp, at<float>(x.a[3]),
                                                            at<double>(x.a[4]), at<float>(x.a[5]), at<float>(x.a[6]),
                                                            at<float>(x.a[7]), at<uint16_t>(x.a[8]), x.a[9].ptr);
}
int64_t call_pack(void *fn, Args &x) {
    return reinterpret_cast<decltype(&paro_pack_params)>(fn)(at<paro_plan_t>(x.a[0]), (int)x.a[1].num, at<float>(x.a[2]),
                                                             at<uint16_t>(x.a[3]), x.a[4].ptr);
}
int64_t call_step(void *fn, Args &x) {
    return reinterpret_cast<decltype(&paro_step_fused)>(fn)(at<paro_plan_t>(x.a[0]), (int)x.a[1].num, x.contrib, (int)x.a[3].num, &x.hp,
                                                            at<float>(x.a[5]), at<double>(x.a[6]), at<float>(x.a[7]),
                                                            at<float>(x.a[8]), at<float>(x.a[9]), at<uint16_t>(x.a[10]), x.a[11].ptr);
}
int64_t call_static(void *fn, Args &x) {
    return reinterpret_cast<decltype(&paro_step_fused_static)>(fn)(at<paro_plan_t>(x.a[0]), (int)x.a[1].num, x.contrib, &x.hp,
                                                                   at<float>(x.a[4]), at<double>(x.a[5]), at<float>(x.a[6]),
                                                                   at<float>(x.a[7]), at<float>(x.a[8]), at<uint16_t>(x.a[9]),
                                                                   x.a[10].ptr);
}
int64_t call_hop(void *fn, Args &x) {
    return reinterpret_cast<decltype(&paro_ring_hop)>(fn)(at<paro_plan_t>(x.a[0]), x.a[1].ptr, (int)x.a[2].num, x.a[3].ptr,
                                                          (int)x.a[4].num, at<float>(x.a[5]), x.a[6].num, x.a[7].ptr);
}
int64_t call_collective(void *fn, Args &x) {
    return reinterpret_cast<decltype(&paro_collective_step)>(fn)(at<paro_plan_t>(x.a[0]), (int)x.a[1].num, (int)x.a[2].num,
                                                                 (int)x.a[3].num, (int)x.a[4].num, (int)x.a[5].num, (int)x.a[6].num,
                                                                 const_cast<void *const *>(x.contrib), x.a[8].ptr);
}

struct Call {
    const char *name, *kinds, *doc;
    int least;                        // arguments without a default
    int64_t (*call)(void *, Args &);
    bool counts;                      // returns a number
};
constexpr Call CALLS[] = {
    {"paro_reduce_shard", "Picippp",
     "paro_reduce_shard(plan, rank, contrib, layout, grad_out, sumsq_out, stream=0)\n--\n\n", 6, call_reduce, false},
    {"paro_adam_shard", "Pihppppppp",
     "paro_adam_shard(plan, rank, hp, grad, total_sumsq, p, m, v, dst_base=0, stream=0)\n--\n\n", 8, call_adam, false},
    {"paro_pack_params", "Pippp", "paro_pack_params(plan, rank, p, dst_base, stream=0)\n--\n\n", 4, call_pack, false},
    {"paro_step_fused", "Picihppppppp",
     "paro_step_fused(plan, rank, contrib, layout, hp, grad_scratch, sumsq_scratch, p, m, v, dst_base, stream=0)\n--\n\n", 11, call_step, false},
    {"paro_step_fused_static", "Pichppppppp",
     "paro_step_fused_static(plan, rank, contrib, hp, grad_scratch, sumsq_scratch, p, m, v, dst_base, stream=0)\n--\n\n", 10, call_static, false},
    {"paro_ring_hop", "Ppipipnp", "paro_ring_hop(plan, partial_in, in_dtype, local, local_dtype, out, n, stream=0)\n--\n\n", 7, call_hop, false},
    {"paro_collective_step", "Piiiiiicp", "paro_collective_step(plan, rank, sched, collective, phase, ring, step, bufs, stream=0)\n--\n\n", 8,
     call_collective, true},
};
constexpr int N_CALLS = sizeof(CALLS) / sizeof(CALLS[0]);
void *g_fn[N_CALLS];
PyObject *g_slow[N_CALLS + 1];        // the ctypes functions; the last is make_adam's Python form

PyObject *slow(int which, PyObject *const *args, Py_ssize_t n, PyObject *kwnames) {
    return PyObject_Vectorcall(g_slow[which], args, (size_t)n, kwnames);
}

template <int I>
PyObject *fast(PyObject *, PyObject *const *args, Py_ssize_t n, PyObject *kwnames) {
    constexpr Call c = CALLS[I];
    Args x;
    const bool usual = (!kwnames || PyTuple_GET_SIZE(kwnames) == 0) && n >= c.least && n <= (Py_ssize_t)std::strlen(c.kinds);
    if (!usual || !parse(c.kinds, args, n, &x)) return slow(I, args, n, kwnames);
    int64_t rc;
    Py_BEGIN_ALLOW_THREADS
    rc = c.call(g_fn[I], x);
    Py_END_ALLOW_THREADS
    if (rc < 0) return PyObject_CallFunction(g_check, "L", (long long)rc);      // raises
    if (c.counts) return PyLong_FromLongLong(rc);
    Py_RETURN_NONE;
}

// make_adam(*, lr, ...): the fields in paro_adam_t's order
const char *const FIELDS[] = {"lr", "beta1", "beta2", "eps", "weight_decay", "grad_scale", "max_norm", "step", "adamw", "skip_nonfinite"};
constexpr int N_FIELDS = 10, N_FLOATS = 7, STEP = 7, REQUIRED = 6;
PyObject *g_fields[N_FIELDS];

PyObject *make_adam(PyObject *, PyObject *const *args, Py_ssize_t n, PyObject *kwnames) {
    paro_adam_t hp;
    std::memset(&hp, 0, sizeof(hp));
    hp.step = 1;
    hp.adamw = 1;
    float *const floats[N_FLOATS] = {&hp.lr, &hp.beta1, &hp.beta2, &hp.eps, &hp.weight_decay, &hp.grad_scale, &hp.max_norm};
    const Py_ssize_t n_kw = kwnames ? PyTuple_GET_SIZE(kwnames) : 0;
    unsigned seen = 0;
    bool usual = n == 0;
    for (Py_ssize_t k = 0; usual && k < n_kw; ++k) {
        PyObject *name = PyTuple_GET_ITEM(kwnames, k), *o = args[k];
        int f = 0;
        while (f < N_FIELDS && name != g_fields[f]) ++f;                 // names in a program's text are interned
        if (f == N_FIELDS) {
            usual = false;
        } else if (f < N_FLOATS) {
            if (PyFloat_CheckExact(o)) *floats[f] = (float)PyFloat_AS_DOUBLE(o);
            else usual = false;
        } else if (f == STEP) {
            int64_t step;
            usual = number(o, INT_MIN, INT_MAX, &step);
            if (usual) hp.step = (int32_t)step;
        } else {
            usual = o == Py_True || o == Py_False;
            (f == STEP + 1 ? hp.adamw : hp.skip_nonfinite) = o == Py_True;
        }
        seen |= 1u << f;
    }
    if (!usual || (seen & ((1u << REQUIRED) - 1)) != (1u << REQUIRED) - 1) return slow(N_CALLS, args, n, kwnames);
    PyObject *out = PyObject_CallNoArgs(g_adam_type);
    if (!out) return nullptr;
    Py_buffer view;
    if (PyObject_GetBuffer(out, &view, PyBUF_WRITABLE) != 0) {
        Py_DECREF(out);
        return nullptr;
    }
    std::memcpy(view.buf, &hp, sizeof(hp));                              // setup() has checked the size
    PyBuffer_Release(&view);
    return out;
}

PyMethodDef g_defs[N_CALLS + 1];

template <int I>
void define() {
    if constexpr (I < N_CALLS) {
        g_defs[I] = {CALLS[I].name, (PyCFunction)(void (*)())fast<I>, METH_FASTCALL | METH_KEYWORDS, CALLS[I].doc};
        define<I + 1>();
    }
}

// setup(module, handle): the forms of the calls below for the binding `module` that holds their ctypes forms, by name.
// handle: the library as the binding has loaded it - not linked to, so that there is one of it.
PyObject *setup(PyObject *, PyObject *args) {
    PyObject *module;
    unsigned long long handle;
    if (!PyArg_ParseTuple(args, "OK", &module, &handle)) return nullptr;
    for (int k = 0; k < N_CALLS; ++k) {
        g_fn[k] = dlsym(reinterpret_cast<void *>((uintptr_t)handle), CALLS[k].name);
        if (!g_fn[k]) {
            PyErr_Format(PyExc_ImportError, "the library does not export %s", CALLS[k].name);
            return nullptr;
        }
    }
    PyObject *types[] = {PyObject_GetAttrString(module, "Plan"), PyObject_GetAttrString(module, "c_void_p"),
                         PyObject_GetAttrString(module, "paro_adam_t"), PyObject_GetAttrString(module, "_check")};
    for (PyObject *t : types)
        if (!t) return nullptr;
    PyObject *hp = PyObject_CallNoArgs(types[2]), *out = PyDict_New(), *doc_name = PyUnicode_FromString("paper_2310_06003_amd");
    paro_adam_t probe;
    if (!hp || !out || !doc_name) return nullptr;
    const bool fits = copy_out(hp, &probe, sizeof(probe));
    Py_DECREF(hp);
    if (!fits) {
        PyErr_SetString(PyExc_RuntimeError, "paro_adam_t has another size here than in paro.h");
        return nullptr;
    }
    define<0>();
    g_defs[N_CALLS] = {"make_adam", (PyCFunction)(void (*)())make_adam, METH_FASTCALL | METH_KEYWORDS,
                       "make_adam(*, lr, beta1, beta2, eps, weight_decay, grad_scale, max_norm=0.0, step=1, adamw=True, "
                       "skip_nonfinite=False)\n--\n\n"};
    for (int k = 0; k < N_FIELDS; ++k)
        if (!(g_fields[k] = PyUnicode_InternFromString(FIELDS[k]))) return nullptr;
    if (!(g_handle_name = PyUnicode_InternFromString("handle"))) return nullptr;
    for (int k = 0; k <= N_CALLS; ++k) {
        if (!(g_slow[k] = PyObject_GetAttrString(module, g_defs[k].ml_name))) return nullptr;
        PyObject *f = PyCFunction_NewEx(&g_defs[k], nullptr, doc_name);
        if (!f || PyDict_SetItemString(out, g_defs[k].ml_name, f) != 0) return nullptr;
        Py_DECREF(f);
    }
    Py_DECREF(doc_name);
    g_handle_type = types[1];
    g_adam_type = types[2];
    g_check = types[3];
    g_plan_type = types[0];
    return out;
}

PyMethodDef g_module_defs[] = {{"setup", setup, METH_VARARGS, nullptr}, {nullptr, nullptr, 0, nullptr}};
PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, g_module_defs, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal() { return PyModule_Create(&g_module); }
