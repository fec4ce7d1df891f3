// Python's way into the run-time entry points of libflexiq, as a native extension module.
//
// A call of a small layer is bound by its host side: of the 7.0 us of a 64 x 256 -> 256 layer with a new output tensor 2.4 are the
// launch, 1.7 torch.empty() from Python and 2 the marshalling in binding.py (argument handling, tensor checks, the ctypes structure and
// call).  Here the arguments are taken as the interpreter hands them over (vectorcall), tensors are looked at and made through the C++
// interface.  Only the ordinary call is served: exact torch tensors that pass the checks of binding.py, plain numbers, layers of this
// process.  Anything else, wrong arguments included, goes to the function of binding.py that a Call wraps, which answers it as before.
#include <Python.h>
#include <structmember.h>

#include <ATen/ATen.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "flexiq.h"

namespace {

// ---- a layer's handle: the base of binding.Layer, whose sizes are ordinary attributes
struct Handle {
    PyObject_HEAD
    unsigned long long ptr;   // flexiq_layer *; 0 once freed
    uint64_t version;         // of the instance's dictionary when the sizes were read; 0: not read
    long N, C, R, S;
};

PyMemberDef handle_members[] = {{"_ptr", T_ULONGLONG, offsetof(Handle, ptr), 0, nullptr}, {nullptr, 0, 0, 0, nullptr}};

PyTypeObject handle_type = {PyVarObject_HEAD_INIT(nullptr, 0)};

// ---- the entry points, found in the library that binding.load() opened; null before
struct Entry {
    decltype(&flexiq_mixed_gemm) gemm;
    decltype(&flexiq_mixed_gemm_fp6) gemm_fp6;
    decltype(&flexiq_mixed_gemm_packed4) gemm_packed4;
    decltype(&flexiq_mixed_conv_implicit) conv;
    decltype(&flexiq_lower_fp6) lower_fp6;
    decltype(&flexiq_lower_packed4) lower_packed4;
    decltype(&flexiq_quantize_act) quantize_act;
    decltype(&flexiq_permute_channels) permute;
    decltype(&flexiq_dynamic_positions) positions;
    decltype(&flexiq_fp6_channels) fp6_channels;
    decltype(&flexiq_fp6_bytes) fp6_bytes;
    decltype(&flexiq_layer_info) layer_info;
} entry;
bool ready = false;
PyObject *check = nullptr;   // binding._check(status): raises

constexpr int kMost = 12;
struct Call;
typedef PyObject *(*Body)(PyObject *const *a);   // a: the parameters in order, null where not given; null without an error set: not served
struct Kind {
    const char *name;
    Body body;
    const char *params[kMost + 1];
    PyObject *names[kMost];   // interned
    int count;
};

struct Call {
    PyObject_HEAD
    vectorcallfunc vectorcall;
    PyObject *dict;
    PyObject *weak;       // list of weak references
    PyObject *fallback;
    const Kind *kind;
};

// ---- arguments
PyObject *size_names[4];   // interned
inline flexiq_layer *raw(const Handle *h) { return reinterpret_cast<flexiq_layer *>(h->ptr); }
inline Handle *handle(PyObject *o)   // null: not a layer of this process, or freed
{
    if (!o || !PyObject_TypeCheck(o, &handle_type)) return nullptr;
    Handle *h = reinterpret_cast<Handle *>(o);
    return h->ptr ? h : nullptr;
}
// ... with its sizes, which are looked up when something in the instance's dictionary has changed (at every call 0.01 to 0.02 us of 0.19 without
// the launch and a new output); null too where they are no plain integers
inline const Handle *layer(PyObject *o)
{
    Handle *h = handle(o);
    PyObject **const dict = h ? _PyObject_GetDictPtr(o) : nullptr;
    if (!dict || !*dict) return nullptr;
#if PY_VERSION_HEX < 0x030c0000   // (later ones have no such number to rely on)
    const uint64_t version = reinterpret_cast<PyDictObject *>(*dict)->ma_version_tag;
    if (h->version == version) return h;
#else
    const uint64_t version = 0;
#endif
    long *const to[4] = {&h->N, &h->C, &h->R, &h->S};
    h->version = 0;
    for (int k = 0; k < 4; ++k) {
        PyObject *v = PyDict_GetItem(*dict, size_names[k]);
        int over = 1;
        if (v && PyLong_CheckExact(v)) *to[k] = PyLong_AsLongAndOverflow(v, &over);
        if (over) return nullptr;
    }
    h->version = version;
    return h;
}
inline bool given(PyObject *o) { return o && o != Py_None; }
inline const at::Tensor *tensor(PyObject *o) { return o && THPVariable_CheckExact(o) ? &THPVariable_Unpack(o) : nullptr; }
inline bool flag(PyObject *o, bool *v)   // True, False or not given
{
    *v = o == Py_True;
    return !o || o == Py_True || o == Py_False;
}
inline bool number(PyObject *o, float *v)
{
    if (PyFloat_CheckExact(o)) *v = (float)PyFloat_AS_DOUBLE(o);
    else return false;
    return true;
}
inline bool integer(PyObject *o, int *v)
{
    if (!o || !PyLong_CheckExact(o)) return false;
    int over = 0;
    const long w = PyLong_AsLongAndOverflow(o, &over);
    *v = (int)w;
    return !over && w >= 0 && w < (1 << 20);
}
// int8, on a GPU, contiguous, `dim` dimensions (0: any), the last of them the layer's input channels
inline const at::Tensor *codes(PyObject *o, const Handle *h, int dim)
{
    const at::Tensor *t = tensor(o);
    if (!t || !t->is_cuda() || t->scalar_type() != at::kChar || !t->is_contiguous()) return nullptr;
    const int64_t d = t->dim();
    return d > 0 && (dim == 0 || d == dim) && t->size(d - 1) == h->C ? t : nullptr;
}
inline void *stream() { return c10::hip::getCurrentHIPStream().stream(); }

PyObject *failed(int status)
{
    PyObject *r = PyObject_CallFunction(check, "i", status);
    Py_XDECREF(r);
    if (!PyErr_Occurred()) PyErr_SetString(PyExc_RuntimeError, "flexiq: a call failed");
    return nullptr;
}

// ---- outputs of a GEMM or convolution: acc, y, q, out_scale, bufs, lower_for and scan_for are a[at] .. a[at + 6] (scan: whether the last exists)
struct Outs {
    flexiq_out o = {};
    PyObject *obj[3] = {nullptr, nullptr, nullptr};   // owned
    ~Outs()
    {
        for (PyObject *p : obj) Py_XDECREF(p);
    }
    bool read(PyObject *const *a, int at, bool scan, at::IntArrayRef shape, const at::Tensor &like)
    {
        static const char *const keys[3] = {"acc", "y", "q"};
        static const at::ScalarType types[3] = {at::kInt, at::kFloat, at::kChar};
        static PyObject *names[3] = {PyUnicode_InternFromString(keys[0]), PyUnicode_InternFromString(keys[1]), PyUnicode_InternFromString(keys[2])};
        bool want[3];
        for (int k = 0; k < 3; ++k)
            if (!flag(a[at + k], &want[k])) return false;
        o.out_scale = 1.0f;
        if (a[at + 3] && !number(a[at + 3], &o.out_scale)) return false;
        PyObject *bufs = given(a[at + 4]) ? a[at + 4] : nullptr;
        if (bufs && !PyDict_CheckExact(bufs)) return false;
        for (int k = 0; k < 2; ++k) {
            PyObject *l = k == 0 ? a[at + 5] : scan ? a[at + 6] : nullptr;
            if (!given(l)) continue;
            const Handle *h = handle(l);
            if (!h) return false;
            if (k == 0) o.lower_for = raw(h);
            else o.scan_for = raw(h);
        }
        for (int k = 0; k < 3; ++k) {   // (nothing is allocated for a call that is not served)
            if (!want[k] || !bufs) continue;
            PyObject *b = PyDict_GetItem(bufs, names[k]);
            if (!b) continue;
            if (!tensor(b)) return false;
            Py_INCREF(b);
            obj[k] = b;
        }
        void *data[3] = {nullptr, nullptr, nullptr};
        for (int k = 0; k < 3; ++k) {
            if (!want[k]) continue;
            if (!obj[k]) obj[k] = THPVariable_Wrap(at::empty(shape, like.options().dtype(types[k])));
            data[k] = THPVariable_Unpack(obj[k]).data_ptr();
        }
        o.acc = (int32_t *)data[0];
        o.y = (float *)data[1];
        o.q = (int8_t *)data[2];
        return true;
    }
    PyObject *result()
    {
        PyObject *d = PyDict_New();
        if (!d) return nullptr;
        static PyObject *names[3] = {PyUnicode_InternFromString("acc"), PyUnicode_InternFromString("y"), PyUnicode_InternFromString("q")};
        for (int k = 0; k < 3; ++k)
            if (PyDict_SetItem(d, names[k], obj[k] ? obj[k] : Py_None) < 0) {
                Py_DECREF(d);
                return nullptr;
            }
        return d;
    }
};

template <class F> inline int launch(F f)   // (other threads run meanwhile, as they do during a ctypes call)
{
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = f();
    Py_END_ALLOW_THREADS
    return rc;
}

PyObject *gemm(PyObject *const *a)
{
    const Handle *h = layer(a[0]);
    const at::Tensor *x = h ? codes(a[1], h, 2) : nullptr;
    if (!x) return nullptr;
    const at::Tensor *x4 = nullptr;
    if (given(a[9]) && !(x4 = tensor(a[9]))) return nullptr;
    const int64_t M = x->size(0);
    Outs o;
    if (!o.read(a, 2, true, {M, h->N}, *x)) return nullptr;
    if (x4) o.o.x4 = (uint8_t *)x4->data_ptr();
    const int8_t *px = (const int8_t *)x->data_ptr();
    void *s = stream();
    const int rc = launch([&] { return entry.gemm(raw(h), px, M, &o.o, s); });
    return rc ? failed(rc) : o.result();
}

PyObject *gemm_fp6(PyObject *const *a)
{
    const Handle *h = layer(a[0]);
    const at::Tensor *x = h ? codes(a[1], h, 2) : nullptr;
    if (!x || !a[2]) return nullptr;
    const at::Tensor *x6 = nullptr, *x6_out = nullptr;
    if (a[2] != Py_None && !(x6 = tensor(a[2]))) return nullptr;
    if (given(a[9]) && !(x6_out = tensor(a[9]))) return nullptr;
    const int64_t M = x->size(0);
    Outs o;
    if (!o.read(a, 3, false, {M, h->N}, *x)) return nullptr;
    if (x6_out) o.o.x6 = (uint8_t *)x6_out->data_ptr();
    const int8_t *px = (const int8_t *)x->data_ptr();
    const uint8_t *p6 = x6 ? (const uint8_t *)x6->data_ptr() : nullptr;
    void *s = stream();
    const int rc = launch([&] { return entry.gemm_fp6(raw(h), px, p6, M, &o.o, s); });
    return rc ? failed(rc) : o.result();
}

PyObject *gemm_packed4(PyObject *const *a)
{
    const Handle *h = layer(a[0]);
    const at::Tensor *x = h ? codes(a[1], h, 2) : nullptr, *x4 = x ? tensor(a[2]) : nullptr, *x4_out = nullptr;
    if (!x4) return nullptr;
    if (given(a[9]) && !(x4_out = tensor(a[9]))) return nullptr;
    const int64_t M = x->size(0);
    Outs o;
    if (!o.read(a, 3, false, {M, h->N}, *x)) return nullptr;
    if (x4_out) o.o.x4 = (uint8_t *)x4_out->data_ptr();
    const int8_t *px = (const int8_t *)x->data_ptr();
    const uint8_t *p4 = (const uint8_t *)x4->data_ptr();
    void *s = stream();
    const int rc = launch([&] { return entry.gemm_packed4(raw(h), px, p4, M, &o.o, s); });
    return rc ? failed(rc) : o.result();
}

PyObject *conv(PyObject *const *a)
{
    const Handle *h = layer(a[0]);
    const at::Tensor *x = h ? codes(a[1], h, 4) : nullptr;
    int stride, pad;
    if (!x || !integer(a[2], &stride) || !integer(a[3], &pad) || stride == 0) return nullptr;
    const int64_t B = x->size(0), H = x->size(1), W = x->size(2);
    if (B > INT32_MAX || H > INT32_MAX || W > INT32_MAX || H + 2 * pad < h->R || W + 2 * pad < h->S) return nullptr;
    const int64_t Ho = (H + 2 * pad - h->R) / stride + 1, Wo = (W + 2 * pad - h->S) / stride + 1;
    Outs o;
    if (!o.read(a, 4, true, {B, Ho, Wo, h->N}, *x)) return nullptr;
    const int8_t *px = (const int8_t *)x->data_ptr();
    void *s = stream();
    const int rc = launch([&] { return entry.conv(raw(h), px, (int32_t)B, (int32_t)H, (int32_t)W, stride, pad, &o.o, s); });
    return rc ? failed(rc) : o.result();
}

PyObject *lower_fp6(PyObject *const *a)
{
    const Handle *h = layer(a[0]);
    const at::Tensor *x = h ? codes(a[1], h, 2) : nullptr;
    if (!x) return nullptr;
    const at::Tensor *given6 = nullptr;
    if (given(a[2]) && !(given6 = tensor(a[2]))) return nullptr;
    if (a[3] && a[3] != Py_None && a[3] != Py_True && a[3] != Py_False) return nullptr;
    const int64_t M = x->size(0), bytes = entry.fp6_bytes(raw(h), M);
    int32_t k6 = 0, k4 = 0;
    if (bytes < 0 || entry.fp6_channels(raw(h), &k6) || entry.layer_info(raw(h), nullptr, nullptr, nullptr, nullptr, nullptr, &k4)) return nullptr;
    const bool low = given(a[3]) ? a[3] == Py_True : k6 < k4;
    at::Tensor x6 = given6 ? *given6 : at::empty({std::max<int64_t>(bytes, 16)}, x->options().dtype(at::kByte)), xlow;
    if (low) xlow = at::empty_like(*x);
    const int8_t *px = (const int8_t *)x->data_ptr();
    uint8_t *p6 = (uint8_t *)x6.data_ptr();
    int8_t *pl = low ? (int8_t *)xlow.data_ptr() : nullptr;
    void *s = stream();
    const int rc = launch([&] { return entry.lower_fp6(raw(h), px, M, p6, pl, s); });
    if (rc) return failed(rc);
    PyObject *first = a[2], *second = a[1];
    if (given6) Py_INCREF(first);
    else first = THPVariable_Wrap(std::move(x6));
    if (low) second = THPVariable_Wrap(std::move(xlow));
    else Py_INCREF(second);
    PyObject *r = PyTuple_Pack(2, first, second);
    Py_XDECREF(first);
    Py_XDECREF(second);
    return r;
}

PyObject *lower_packed4(PyObject *const *a)
{
    const Handle *h = layer(a[0]);
    const at::Tensor *x = h ? codes(a[1], h, 2) : nullptr;
    if (!x) return nullptr;
    const at::Tensor *given4 = nullptr;
    if (given(a[2]) && !(given4 = tensor(a[2]))) return nullptr;
    const int64_t M = x->size(0);
    at::Tensor x4 = given4 ? *given4 : at::empty({std::max<int64_t>(M, 1), h->C / 2}, x->options().dtype(at::kByte));
    const int8_t *px = (const int8_t *)x->data_ptr();
    uint8_t *p4 = (uint8_t *)x4.data_ptr();
    void *s = stream();
    const int rc = launch([&] { return entry.lower_packed4(raw(h), px, M, p4, s); });
    if (rc) return failed(rc);
    if (!given4) return THPVariable_Wrap(std::move(x4));
    Py_INCREF(a[2]);
    return a[2];
}

PyObject *quantize_act(PyObject *const *a)
{
    const at::Tensor *x = tensor(a[0]);
    float scale;
    if (!x || !x->is_cuda() || x->scalar_type() != at::kFloat || !x->is_contiguous() || !a[1] || !number(a[1], &scale)) return nullptr;
    const at::Tensor *given_q = nullptr;
    if (given(a[2]) && !(given_q = tensor(a[2]))) return nullptr;
    at::Tensor q = given_q ? *given_q : at::empty(x->sizes(), x->options().dtype(at::kChar));
    const float *px = (const float *)x->data_ptr();
    int8_t *pq = (int8_t *)q.data_ptr();
    const int64_t n = x->numel();
    void *s = stream();
    const int rc = launch([&] { return entry.quantize_act(px, pq, n, scale, s); });
    if (rc) return failed(rc);
    if (!given_q) return THPVariable_Wrap(std::move(q));
    Py_INCREF(a[2]);
    return a[2];
}

PyObject *permute(PyObject *const *a)
{
    const Handle *h = layer(a[0]);
    const at::Tensor *x = h ? tensor(a[1]) : nullptr;
    if (!x || !x->is_cuda() || x->scalar_type() != at::kChar || !x->is_contiguous() || h->C <= 0) return nullptr;
    at::Tensor to = at::empty_like(*x);
    const int8_t *px = (const int8_t *)x->data_ptr();
    int8_t *pt = (int8_t *)to.data_ptr();
    const int64_t rows = x->numel() / h->C;
    void *s = stream();
    const int rc = launch([&] { return entry.permute(raw(h), px, pt, rows, s); });
    return rc ? failed(rc) : THPVariable_Wrap(std::move(to));
}

PyObject *positions(PyObject *const *a)
{
    const Handle *h = layer(a[0]);
    const at::Tensor *x = h ? codes(a[1], h, 0) : nullptr;
    if (!x || h->C <= 0) return nullptr;
    const int8_t *px = (const int8_t *)x->data_ptr();
    const int64_t rows = x->numel() / h->C;
    void *s = stream();
    const int rc = launch([&] { return entry.positions(raw(h), px, rows, s); });
    if (rc) return failed(rc);
    Py_RETURN_NONE;
}

Kind kinds[] = {
    {"flexiq_mixed_gemm", gemm, {"layer", "X", "acc", "y", "q", "out_scale", "bufs", "lower_for", "scan_for", "x4_out"}},
    {"flexiq_mixed_gemm_fp6", gemm_fp6, {"layer", "X", "x6", "acc", "y", "q", "out_scale", "bufs", "lower_for", "x6_out"}},
    {"flexiq_mixed_gemm_packed4", gemm_packed4, {"layer", "X", "x4", "acc", "y", "q", "out_scale", "bufs", "lower_for", "x4_out"}},
    {"flexiq_mixed_conv_implicit", conv, {"layer", "X", "stride", "pad", "acc", "y", "q", "out_scale", "bufs", "lower_for", "scan_for"}},
    {"flexiq_lower_fp6", lower_fp6, {"layer", "X", "x6", "need_xlow"}},
    {"flexiq_lower_packed4", lower_packed4, {"layer", "X", "x4"}},
    {"flexiq_quantize_act", quantize_act, {"x", "scale", "out"}},
    {"flexiq_permute_channels", permute, {"layer", "src"}},
    {"flexiq_dynamic_positions", positions, {"layer", "X"}},
};

PyObject *call(PyObject *self, PyObject *const *args, size_t nargsf, PyObject *kwnames)
{
    Call *c = reinterpret_cast<Call *>(self);
    const Kind &k = *c->kind;
    const Py_ssize_t n = PyVectorcall_NARGS(nargsf), nk = kwnames ? PyTuple_GET_SIZE(kwnames) : 0;
    bool ok = ready && n <= k.count;
    PyObject *a[kMost] = {};
    if (ok) {
        for (Py_ssize_t i = 0; i < n; ++i) a[i] = args[i];
        for (Py_ssize_t j = 0; j < nk && ok; ++j) {
            PyObject *name = PyTuple_GET_ITEM(kwnames, j);   // (a call site's names are interned)
            int at = 0;
            while (at < k.count && k.names[at] != name) ++at;
            if (at == k.count || a[at]) ok = false;
            else a[at] = args[n + j];
        }
    }
    if (ok) {
        HANDLE_TH_ERRORS
        PyObject *r = k.body(a);
        if (r || PyErr_Occurred()) return r;
        END_HANDLE_TH_ERRORS
    }
    return PyObject_Vectorcall(c->fallback, args, nargsf, kwnames);
}

void call_dealloc(PyObject *self)
{
    Call *c = reinterpret_cast<Call *>(self);
    PyObject_GC_UnTrack(self);
    if (c->weak) PyObject_ClearWeakRefs(self);
    Py_CLEAR(c->dict);
    Py_CLEAR(c->fallback);
    Py_TYPE(self)->tp_free(self);
}
int call_traverse(PyObject *self, visitproc visit, void *arg)
{
    Call *c = reinterpret_cast<Call *>(self);
    Py_VISIT(c->dict);
    Py_VISIT(c->fallback);
    return 0;
}
int call_clear(PyObject *self)
{
    Call *c = reinterpret_cast<Call *>(self);
    Py_CLEAR(c->dict);
    return 0;
}

// ---- what else a program does with a function: it is one for isinstance() and the inspect module (as it is for a program that asks
// whether something is one before it looks at its defaults or code), binds as a method, and is copied and pickled by its name
PyObject *call_class(PyObject *, void *)
{
    Py_INCREF(&PyFunction_Type);
    return reinterpret_cast<PyObject *>(&PyFunction_Type);
}
PyObject *call_getattro(PyObject *self, PyObject *name)
{
    PyObject *v = PyObject_GenericGetAttr(self, name);
    if (v || !PyErr_ExceptionMatches(PyExc_AttributeError)) return v;
    PyErr_Clear();
    return PyObject_GetAttr(reinterpret_cast<Call *>(self)->fallback, name);
}
PyObject *call_bind(PyObject *self, PyObject *object, PyObject *)
{
    if (object && object != Py_None) return PyMethod_New(self, object);
    Py_INCREF(self);
    return self;
}
PyObject *call_reduce(PyObject *self, PyObject *) { return PyObject_GetAttrString(self, "__qualname__"); }

PyMethodDef call_methods[] = {{"__reduce__", call_reduce, METH_NOARGS, nullptr}, {nullptr, nullptr, 0, nullptr}};
PyGetSetDef call_getset[] = {{"__dict__", PyObject_GenericGetDict, PyObject_GenericSetDict, nullptr, nullptr},
                             {"__class__", call_class, nullptr, nullptr, nullptr},
                             {nullptr, nullptr, nullptr, nullptr, nullptr}};
PyTypeObject call_type = {PyVarObject_HEAD_INIT(nullptr, 0)};

// wrap(function): a Call of the entry point of that name which hands what it does not serve to the function
PyObject *wrap(PyObject *, PyObject *function)
{
    PyObject *name = PyObject_GetAttrString(function, "__name__");
    const char *text = name ? PyUnicode_AsUTF8(name) : nullptr;
    const Kind *kind = nullptr;
    for (const Kind &k : kinds)
        if (text && !strcmp(k.name, text)) kind = &k;
    Py_XDECREF(name);
    if (!kind) {
        if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "no entry point of that name");
        return nullptr;
    }
    Call *c = PyObject_GC_New(Call, &call_type);
    if (!c) return nullptr;
    c->vectorcall = call;
    c->dict = nullptr;
    c->weak = nullptr;
    Py_INCREF(function);
    c->fallback = function;
    c->kind = kind;
    PyObject_GC_Track(reinterpret_cast<PyObject *>(c));
    return reinterpret_cast<PyObject *>(c);
}

// connect(addresses, check): the addresses of the entry points by name; an empty dict: none (the library is not loaded)
PyObject *connect(PyObject *, PyObject *args)
{
    PyObject *d, *f;
    if (!PyArg_ParseTuple(args, "O!O", &PyDict_Type, &d, &f)) return nullptr;
    ready = false;
    if (PyDict_Size(d) == 0) Py_RETURN_NONE;
    bool ok = true;
    auto get = [&](const char *name, auto *to) {
        PyObject *v = PyDict_GetItemString(d, name);
        const unsigned long long p = v ? PyLong_AsUnsignedLongLong(v) : 0;
        if (!p || PyErr_Occurred()) ok = false;
        *reinterpret_cast<unsigned long long *>(to) = p;
    };
    get("flexiq_mixed_gemm", &entry.gemm);
    get("flexiq_mixed_gemm_fp6", &entry.gemm_fp6);
    get("flexiq_mixed_gemm_packed4", &entry.gemm_packed4);
    get("flexiq_mixed_conv_implicit", &entry.conv);
    get("flexiq_lower_fp6", &entry.lower_fp6);
    get("flexiq_lower_packed4", &entry.lower_packed4);
    get("flexiq_quantize_act", &entry.quantize_act);
    get("flexiq_permute_channels", &entry.permute);
    get("flexiq_dynamic_positions", &entry.positions);
    get("flexiq_fp6_channels", &entry.fp6_channels);
    get("flexiq_fp6_bytes", &entry.fp6_bytes);
    get("flexiq_layer_info", &entry.layer_info);
    if (!ok) {
        if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "an entry point is missing");
        return nullptr;
    }
    Py_INCREF(f);
    Py_XDECREF(check);
    check = f;
    ready = true;
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {{"wrap", wrap, METH_O, nullptr}, {"connect", connect, METH_VARARGS, nullptr}, {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_calls", nullptr, -1, methods};

}  // namespace

PyMODINIT_FUNC PyInit__calls()
{
    handle_type.tp_name = "_calls.Handle";
    handle_type.tp_basicsize = sizeof(Handle);
    handle_type.tp_flags = Py_TPFLAGS_DEFAULT | Py_TPFLAGS_BASETYPE;
    handle_type.tp_members = handle_members;
    handle_type.tp_new = PyType_GenericNew;
    call_type.tp_name = "_calls.Call";
    call_type.tp_basicsize = sizeof(Call);
    call_type.tp_flags = Py_TPFLAGS_DEFAULT | Py_TPFLAGS_HAVE_VECTORCALL | Py_TPFLAGS_HAVE_GC;
    call_type.tp_vectorcall_offset = offsetof(Call, vectorcall);
    call_type.tp_call = PyVectorcall_Call;
    call_type.tp_dictoffset = offsetof(Call, dict);
    call_type.tp_weaklistoffset = offsetof(Call, weak);
    call_type.tp_methods = call_methods;
    call_type.tp_getset = call_getset;
    call_type.tp_descr_get = call_bind;
    call_type.tp_dealloc = call_dealloc;
    call_type.tp_traverse = call_traverse;
    call_type.tp_clear = call_clear;
    call_type.tp_getattro = call_getattro;
    call_type.tp_setattro = PyObject_GenericSetAttr;
    if (PyType_Ready(&handle_type) < 0 || PyType_Ready(&call_type) < 0) return nullptr;
    const char *const sizes[4] = {"N", "C", "R", "S"};
    for (int k = 0; k < 4; ++k) size_names[k] = PyUnicode_InternFromString(sizes[k]);
    for (Kind &k : kinds) {
        k.count = 0;
        while (k.params[k.count]) {
            k.names[k.count] = PyUnicode_InternFromString(k.params[k.count]);
            ++k.count;
        }
    }
    PyObject *m = PyModule_Create(&module);
    if (!m) return nullptr;
    if (PyModule_AddStringConstant(m, "built_for", BUILT_FOR) < 0) return nullptr;   // torch.__version__
    Py_INCREF(&handle_type);
    if (PyModule_AddObject(m, "Handle", reinterpret_cast<PyObject *>(&handle_type)) < 0) return nullptr;
    return m;
}
