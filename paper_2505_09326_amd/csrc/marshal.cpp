// The binding's fast way into libsphattn.so: checks, outputs, workspace and launch of a call in one step, as a CPython
// extension on torch's C++ headers.  No arithmetic, no kernels.
//
// The smallest calls are bound by what the host does before the launch, and a training step's two halves run on two threads
// that wake each other, where the interpreter runs at half its speed.  In Python, with ctypes, a forward call took 8.8 us of host
// time, 3.8 with this, of which the launch is 3 (1 x 256 x 64 in fp32 8.7 -> 6.4 us a call), a backward call 22 and 11 (a training step of 8
// heads on 2 of 1500 x 64 with counts 137 -> 89).
//
// A function here does a call only if everything about it is as it has to be: exactly torch's tensor type, with storage, the
// shapes, element types and device that the entry point's header states, contiguous, no function or dispatch mode in force.  For anything
// else, and for whatever throws on the way (no memory for an output), it returns None, having launched nothing, and the binding's Python does the call and finds out what is wrong.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/PythonTorchFunctionTLS.h>
#include <ATen/ops/empty.h>
#include <ATen/ops/empty_like.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <array>
#include <climits>
#include <exception>

#include "../../include/sphattn.h"

namespace {

struct EntryPoints {
    decltype(&sphattn_cross_fwd) cross = nullptr;
    decltype(&sphattn_cross_splitkv_fwd) cross_cut = nullptr;
    decltype(&sphattn_cross_splitkv_workspace_bytes) cross_bytes = nullptr;
    decltype(&sphattn_grn_bwd) bwd = nullptr;
    decltype(&sphattn_grn_bwd_split) bwd_cut = nullptr;
    decltype(&sphattn_bwd_workspace_bytes) bwd_bytes = nullptr;
    decltype(&sphattn_fp8_grn_fwd) fp8 = nullptr;
} entry;
PyObject* raise_on = nullptr;                      // the binding's function that raises for an error code

// The interpreter's lock is given back while torch allocates and the library launches.
struct Unlocked {
    PyThreadState* state = PyEval_SaveThread();
    ~Unlocked() { PyEval_RestoreThread(state); }
};

// Workspace sizes by shape and device (and by the function asked): the library's choice of slices takes a few microseconds.  Per thread,
// one shape per place.
class SizeTable {
public:
    template <typename Ask>
    size_t get(const std::array<int64_t, 9>& key, Ask ask)
    {
        uint64_t h = 0;
        for (const int64_t k : key) h = (h ^ (uint64_t)k) * 0x9e3779b97f4a7c15ull;
        Place& place = places_[h >> 59];
        if (!place.known || place.key != key) place = Place{key, ask(), true};
        return place.bytes;
    }
private:
    struct Place { std::array<int64_t, 9> key; size_t bytes; bool known = false; };
    Place places_[32];
};
thread_local SizeTable sizes;

const at::Tensor* tensor(PyObject* o)
{
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor& t = THPVariable_Unpack(o);
    return t.defined() && t.has_storage() ? &t : nullptr;
}

bool fits(const at::Tensor& t, at::IntArrayRef shape, at::ScalarType type, at::Device device)
{
    return t.scalar_type() == type && t.device() == device && t.layout() == at::kStrided && t.sizes() == shape && t.is_contiguous();
}

bool is_e4m3(const at::Tensor& t) { return t.scalar_type() == at::kFloat8_e4m3fn || t.scalar_type() == at::kByte; }

void* data(const at::Tensor& t) { return t.data_ptr(); }
void* data(const at::Tensor* t) { return t ? t->data_ptr() : nullptr; }

// Q [B,H,Nq,d]; K, V [B,H_kv,Nk,d]
struct Shape {
    int64_t B, H, Nq, d, H_kv, Nk;
    bool read(const at::Tensor& Q, const at::Tensor& K, bool same_n, bool same_h)
    {
        if (Q.dim() != 4 || K.dim() != 4 || !Q.is_cuda()) return false;
        B = Q.size(0), H = Q.size(1), Nq = Q.size(2), d = Q.size(3), H_kv = K.size(1), Nk = K.size(2);
        const int64_t most = INT_MAX;
        return K.size(0) == B && K.size(3) == d && H_kv > 0 && H % H_kv == 0 && (!same_n || Nk == Nq) && (!same_h || H_kv == H) &&
               B <= most && H <= most && Nq <= most && Nk <= most && d <= most;
    }
};

void* stream_of(const at::Tensor& t) { return c10::hip::getCurrentHIPStream(t.get_device()).stream(); }

at::Tensor workspace(size_t bytes, const at::Tensor& like)
{
    if (bytes == 0) return {};
    try {
        return at::empty({(int64_t)bytes}, like.options().dtype(at::kByte));
    } catch (const c10::OutOfMemoryError&) {
        return {};                                 // the uncut launches need none
    }
}

// An optional tensor argument: `there` and its tensor, or false for something that is neither None nor a tensor.
bool optional(PyObject* o, const at::Tensor*& t)
{
    t = nullptr;
    return o == Py_None || (t = tensor(o)) != nullptr;
}

PyObject* wrapped(at::Tensor&& t)
{
    try {
        return THPVariable_Wrap(std::move(t));
    } catch (const std::exception& e) {
        if (!PyErr_Occurred()) PyErr_SetString(PyExc_RuntimeError, e.what());
        return nullptr;
    }
}

PyObject* raised(int rc)
{
    PyObject* none = PyObject_CallFunction(raise_on, "i", rc);
    if (none != nullptr) {                         // (it always raises)
        Py_DECREF(none);
        PyErr_SetString(PyExc_RuntimeError, "sphattn error");
    }
    return nullptr;
}

bool arguments(Py_ssize_t n, Py_ssize_t want)
{
    if (n == want) return true;
    PyErr_Format(PyExc_TypeError, "%zd arguments, not %zd", want, n);
    return false;
}

// (A dispatch mode makes its own tensors for what is allocated here: Python checks those as it does a caller's.)
bool ready() { return entry.cross != nullptr && !at::impl::torch_function_mode_enabled() && !c10::impl::TorchDispatchModeTLS::any_modes_set(); }

// forward(Q, K, V, mult, Z, code, same_n, same_h, want_z) -> O, with want_z (O, Z)
PyObject* forward(PyObject*, PyObject* const* args, Py_ssize_t n)
{
    if (!arguments(n, 9)) return nullptr;
    const at::Tensor *Q = tensor(args[0]), *K = tensor(args[1]), *V = tensor(args[2]), *mult, *Z;
    const long code = PyLong_AsLong(args[5]);
    if (code == -1 && PyErr_Occurred()) return nullptr;
    if (!Q || !K || !V || !optional(args[3], mult) || !optional(args[4], Z) || !ready()) Py_RETURN_NONE;
    at::Tensor O, own_z;
    int rc = 0;
    try {
        Shape s;
        if (!s.read(*Q, *K, args[6] == Py_True, args[7] == Py_True)) Py_RETURN_NONE;
        const at::Device device = Q->device();
        const at::ScalarType vo = code == SPHATTN_F32 ? at::kFloat : code == SPHATTN_F16 ? at::kHalf : at::kBFloat16;
        if (code == SPHATTN_FP8QK_BF16V) {
            if (!is_e4m3(*Q) || !is_e4m3(*K)) Py_RETURN_NONE;
        } else if ((code != SPHATTN_F32 && code != SPHATTN_F16 && code != SPHATTN_BF16) || Q->scalar_type() != vo || K->scalar_type() != vo) {
            Py_RETURN_NONE;
        }
        const int64_t kv[4] = {s.B, s.H_kv, s.Nk, s.d}, counts[2] = {s.B, s.Nk}, rows[3] = {s.B, s.H, s.Nq};
        if (!Q->is_contiguous() || Q->layout() != at::kStrided || !fits(*K, kv, K->scalar_type(), device) || !fits(*V, kv, vo, device) ||
            (mult && !fits(*mult, counts, at::kFloat, device)) || (Z && !fits(*Z, rows, at::kFloat, device)))
            Py_RETURN_NONE;
        const Unlocked unlocked;
        O = Q->scalar_type() == vo ? at::empty_like(*Q) : at::empty(Q->sizes(), Q->options().dtype(vo));
        if (args[8] == Py_True) {
            own_z = at::empty(rows, Q->options().dtype(at::kFloat));
            Z = &own_z;
        }
        const size_t bytes = sizes.get({(int64_t)entry.cross_bytes, Q->get_device(), s.B, s.H, s.H_kv, s.Nq, s.Nk, s.d, code}, [&] {
            return entry.cross_bytes((int)s.B, (int)s.H, (int)s.H_kv, (int)s.Nq, (int)s.Nk, (int)s.d, (int)code);
        });
        const at::Tensor ws = workspace(bytes, *Q);
        auto launch = [&](auto call, auto... rest) {
            return call(data(*Q), data(*K), data(*V), (const float*)data(mult), data(O), (float*)data(Z), (int)s.B, (int)s.H, (int)s.H_kv, (int)s.Nq,
                        (int)s.Nk, (int)s.d, (int)code, rest..., stream_of(*Q));
        };
        rc = ws.defined() ? launch(entry.cross_cut, data(ws), bytes) : launch(entry.cross);
    } catch (...) {
        PyErr_Clear();
        Py_RETURN_NONE;
    }
    if (rc != 0) return raised(rc);
    if (!own_z.defined()) return wrapped(std::move(O));
    PyObject *o = wrapped(std::move(O)), *z = o ? wrapped(std::move(own_z)) : nullptr;
    PyObject* both = z ? PyTuple_Pack(2, o, z) : nullptr;
    Py_XDECREF(o);
    Py_XDECREF(z);
    return both;
}

// backward(Q, K, V, mult, O, dO, Z, code, same_h) -> (dQ, dK, dV)
PyObject* backward(PyObject*, PyObject* const* args, Py_ssize_t n)
{
    if (!arguments(n, 9)) return nullptr;
    const at::Tensor *Q = tensor(args[0]), *K = tensor(args[1]), *V = tensor(args[2]), *O = tensor(args[4]), *dO = tensor(args[5]), *Z = tensor(args[6]), *mult;
    const long code = PyLong_AsLong(args[7]);
    if (code == -1 && PyErr_Occurred()) return nullptr;
    if (!Q || !K || !V || !O || !dO || !Z || !optional(args[3], mult) || (code != SPHATTN_BF16 && code != SPHATTN_F16) || !ready()) Py_RETURN_NONE;
    at::Tensor d[3];
    int rc = 0;
    try {
        Shape s;
        if (!s.read(*Q, *K, true, args[8] == Py_True)) Py_RETURN_NONE;
        const at::Device device = Q->device();
        const at::ScalarType t16 = code == SPHATTN_F16 ? at::kHalf : at::kBFloat16;
        const int64_t q[4] = {s.B, s.H, s.Nq, s.d}, kv[4] = {s.B, s.H_kv, s.Nk, s.d}, counts[2] = {s.B, s.Nk}, rows[3] = {s.B, s.H, s.Nq};
        if (!fits(*Q, q, t16, device) || !fits(*K, kv, t16, device) || !fits(*V, kv, t16, device) || !fits(*O, q, t16, device) || !fits(*dO, q, t16, device) ||
            !fits(*Z, rows, at::kFloat, device) || (mult && !fits(*mult, counts, at::kFloat, device)))
            Py_RETURN_NONE;
        const Unlocked unlocked;
        d[0] = at::empty_like(*Q);
        d[1] = at::empty_like(*K);
        d[2] = at::empty_like(*V);
        if (!fits(d[0], q, t16, device) || !fits(d[1], kv, t16, device) || !fits(d[2], kv, t16, device)) throw 0;
        const at::Tensor delta = at::empty({2, s.B, s.H, s.Nq}, Q->options().dtype(at::kFloat));
        const size_t bytes = sizes.get({(int64_t)entry.bwd_bytes, Q->get_device(), s.B, s.H, s.H_kv, s.Nq, s.Nk, s.d, code}, [&] {
            return entry.bwd_bytes((int)s.B, (int)s.H, (int)s.H_kv, (int)s.Nq, (int)s.d, (int)code);
        });
        const at::Tensor ws = workspace(bytes, *Q);
        auto launch = [&](auto call, auto... rest) {
            return call(data(*Q), data(*K), data(*V), (const float*)data(mult), data(*O), data(*dO), (const float*)data(*Z), data(d[0]), data(d[1]), data(d[2]),
                        (float*)data(delta), (int)s.B, (int)s.H, (int)s.H_kv, (int)s.Nq, (int)s.d, (int)code, rest..., stream_of(*Q));
        };
        rc = ws.defined() ? launch(entry.bwd_cut, data(ws), bytes) : launch(entry.bwd);
    } catch (...) {
        PyErr_Clear();
        Py_RETURN_NONE;
    }
    if (rc != 0) return raised(rc);
    PyObject* out = PyTuple_New(3);
    for (int i = 0; out != nullptr && i < 3; ++i) {
        PyObject* o = wrapped(std::move(d[i]));
        if (o == nullptr) Py_CLEAR(out);
        else PyTuple_SET_ITEM(out, i, o);
    }
    return out;
}

// fp8_forward(Q, K, V, mult, workspace) -> O
PyObject* fp8_forward(PyObject*, PyObject* const* args, Py_ssize_t n)
{
    if (!arguments(n, 5)) return nullptr;
    const at::Tensor *Q = tensor(args[0]), *K = tensor(args[1]), *V = tensor(args[2]), *ws = tensor(args[4]), *mult;
    if (!Q || !K || !V || !ws || !optional(args[3], mult) || !ready()) Py_RETURN_NONE;
    at::Tensor O;
    int rc = 0;
    try {
        Shape s;
        if (!s.read(*Q, *K, true, false) || !is_e4m3(*Q) || !is_e4m3(*K) || !is_e4m3(*V)) Py_RETURN_NONE;
        const at::Device device = Q->device();
        const int64_t kv[4] = {s.B, s.H_kv, s.Nk, s.d}, counts[2] = {s.B, s.Nk};
        if (!Q->is_contiguous() || Q->layout() != at::kStrided || !fits(*K, kv, K->scalar_type(), device) || !fits(*V, kv, V->scalar_type(), device) ||
            (mult && !fits(*mult, counts, at::kFloat, device)) || ws->dim() != 1 || !fits(*ws, ws->sizes(), ws->scalar_type(), device))
            Py_RETURN_NONE;
        const Unlocked unlocked;
        O = at::empty(Q->sizes(), Q->options().dtype(at::kBFloat16));
        rc = entry.fp8(data(*Q), data(*K), data(*V), (const float*)data(mult), data(O), data(*ws), ws->nbytes(), (int)s.B, (int)s.H, (int)s.H_kv,
                       (int)s.Nq, (int)s.d, stream_of(*Q));
    } catch (...) {
        PyErr_Clear();
        Py_RETURN_NONE;
    }
    if (rc != 0) return raised(rc);
    return wrapped(std::move(O));
}

// bind(raise_on, addresses of the entry points in the order of EntryPoints)
PyObject* bind(PyObject*, PyObject* args)
{
    PyObject* handler;
    unsigned long long a[7];
    if (!PyArg_ParseTuple(args, "OKKKKKKK", &handler, &a[0], &a[1], &a[2], &a[3], &a[4], &a[5], &a[6])) return nullptr;
    Py_INCREF(handler);
    Py_XDECREF(raise_on);
    raise_on = handler;
    entry.cross = (decltype(entry.cross))a[0];
    entry.cross_cut = (decltype(entry.cross_cut))a[1];
    entry.cross_bytes = (decltype(entry.cross_bytes))a[2];
    entry.bwd = (decltype(entry.bwd))a[3];
    entry.bwd_cut = (decltype(entry.bwd_cut))a[4];
    entry.bwd_bytes = (decltype(entry.bwd_bytes))a[5];
    entry.fp8 = (decltype(entry.fp8))a[6];
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {{"forward", (PyCFunction)(void*)forward, METH_FASTCALL, nullptr},
                         {"backward", (PyCFunction)(void*)backward, METH_FASTCALL, nullptr},
                         {"fp8_forward", (PyCFunction)(void*)fp8_forward, METH_FASTCALL, nullptr},
                         {"bind", bind, METH_VARARGS, nullptr},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", "Checks, outputs, workspace and launch of a call (see marshal.cpp).", -1, methods};

}  // namespace

PyMODINIT_FUNC PyInit__marshal()
{
    PyObject* m = PyModule_Create(&module);
    // the torch whose headers this was compiled with (its tensors' layout), for the binding to compare
    if (m != nullptr && PyModule_AddStringConstant(m, "built_for", MARSHAL_TORCH) != 0) Py_CLEAR(m);
    return m;
}
