// The call path of the layer's smallest calls, pq_linear and pq_linear2 with the caller's own output and workspace, in native code:
// argument checks, pointers and the current stream.  A decoded token's kernel takes 4.0 us (1 x 4096 -> 4096), the call through
// Python attributes and ctypes 5.5 us of host time, of which 3.5 are ctypes and the launch; here the whole call takes 3.4 us
// (1 x 4096 -> 4096, eager, weights in turn: 5.95 -> 4.33 us a call).
//
// Only the plain case is taken: exact Tensor objects, contiguous, of the types and shapes that the binding asks for.  For anything else
// the functions return -1 and have done nothing, and the Python path decides (and words the error).
#include <Python.h>

#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>

namespace {

using Linear = int (*)(const void*, const void*, const float*, float, int32_t, int64_t, int64_t, int64_t, void*, void*, size_t, void*);
using Linear2 = int (*)(const void*, const void*, const float*, int64_t, void*, const void*, const float*, int64_t, void*, float, int32_t,
                        int64_t, int64_t, void*, size_t, void*);
Linear g_linear = nullptr;
Linear2 g_linear2 = nullptr;

// a tensor that the library reads: on the GPU, contiguous, of this type
bool operand(PyObject* o, at::ScalarType type, const at::Tensor** t)
{
    if (!THPVariable_CheckExact(o)) return false;
    *t = &THPVariable_Unpack(o);
    return (*t)->is_cuda() && (*t)->scalar_type() == type && (*t)->is_contiguous();
}

// the caller's fp16 output, with room for M x N values
bool result(PyObject* o, int64_t M, int64_t N, const at::Tensor** t) { return operand(o, at::kHalf, t) && (*t)->numel() >= M * N; }

// the caller's workspace, of any type (the library compares its elements, taken as bytes, with what it needs)
bool workspace(PyObject* o, const at::Tensor** t)
{
    if (!THPVariable_CheckExact(o)) return false;
    *t = &THPVariable_Unpack(o);
    return (*t)->is_cuda() && (*t)->is_contiguous();
}

bool number(PyObject* step, PyObject* block, double* s, long* h)
{
    if (!PyFloat_Check(step) || !PyLong_Check(block)) return false;
    *s = PyFloat_AS_DOUBLE(step);
    *h = PyLong_AsLong(block);
    if (*h == -1 && PyErr_Occurred()) {
        PyErr_Clear();
        return false;
    }
    return *h >= INT32_MIN && *h <= INT32_MAX;
}

// weights of K input channels and their steps
bool matrix(PyObject* w, PyObject* sw, int64_t K, const at::Tensor** wt, const at::Tensor** st)
{
    return operand(w, at::kByte, wt) && operand(sw, at::kFloat, st) && (*wt)->dim() == 2 && (*wt)->size(1) * 2 == K &&
           (*st)->numel() == (*wt)->size(0);
}

void* stream() { return c10::hip::getCurrentHIPStream().stream(); }

// (x, wq, w_scale, act_scale, had_block, out, workspace) -> status, or -1
PyObject* linear(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    try {
        const at::Tensor *x, *w, *s, *out, *ws;
        double step;
        long h;
        if (n == 7 && g_linear && operand(a[0], at::kHalf, &x) && x->dim() == 2 && matrix(a[1], a[2], x->size(1), &w, &s) &&
            number(a[3], a[4], &step, &h) && result(a[5], x->size(0), w->size(0), &out) && workspace(a[6], &ws)) {
            const void *xp = x->data_ptr(), *wp = w->data_ptr();
            const float* sp = static_cast<const float*>(s->data_ptr());
            void *op = out->data_ptr(), *wsp = ws->data_ptr(), *st = stream();
            const int64_t M = x->size(0), K = x->size(1), N = w->size(0);
            const size_t bytes = (size_t)ws->numel();
            int rc;
            Py_BEGIN_ALLOW_THREADS
            rc = g_linear(xp, wp, sp, (float)step, (int32_t)h, M, N, K, op, wsp, bytes, st);
            Py_END_ALLOW_THREADS
            return PyLong_FromLong(rc);
        }
    } catch (...) {        // (a tensor without memory of its own: the Python path reports it)
    }
    return PyLong_FromLong(-1);
}

// (x, wq_a, w_scale_a, wq_b, w_scale_b, act_scale, had_block, out_a, out_b, workspace) -> status, or -1
PyObject* linear2(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    try {
        const at::Tensor *x, *wa, *sa, *wb, *sb, *oa, *ob, *ws;
        double step;
        long h;
        if (n == 10 && g_linear2 && operand(a[0], at::kHalf, &x) && x->dim() == 2 && matrix(a[1], a[2], x->size(1), &wa, &sa) &&
            matrix(a[3], a[4], x->size(1), &wb, &sb) && number(a[5], a[6], &step, &h) &&
            result(a[7], x->size(0), wa->size(0), &oa) && result(a[8], x->size(0), wb->size(0), &ob) && workspace(a[9], &ws)) {
            const void *xp = x->data_ptr(), *wap = wa->data_ptr(), *wbp = wb->data_ptr();
            const float *sap = static_cast<const float*>(sa->data_ptr()), *sbp = static_cast<const float*>(sb->data_ptr());
            void *oap = oa->data_ptr(), *obp = ob->data_ptr(), *wsp = ws->data_ptr(), *st = stream();
            const int64_t M = x->size(0), K = x->size(1), Na = wa->size(0), Nb = wb->size(0);
            const size_t bytes = (size_t)ws->numel();
            int rc;
            Py_BEGIN_ALLOW_THREADS
            rc = g_linear2(xp, wap, sap, Na, oap, wbp, sbp, Nb, obp, (float)step, (int32_t)h, M, K, wsp, bytes, st);
            Py_END_ALLOW_THREADS
            return PyLong_FromLong(rc);
        }
    } catch (...) {
    }
    return PyLong_FromLong(-1);
}

// (address of pq_linear, address of pq_linear2): the library that the binding has loaded
PyObject* bind(PyObject*, PyObject* args)
{
    unsigned long long l, l2;
    if (!PyArg_ParseTuple(args, "KK", &l, &l2)) return nullptr;
    g_linear = reinterpret_cast<Linear>(static_cast<uintptr_t>(l));
    g_linear2 = reinterpret_cast<Linear2>(static_cast<uintptr_t>(l2));
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {{"bind", bind, METH_VARARGS, nullptr},
                         {"linear", reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(linear)), METH_FASTCALL, nullptr},
                         {"linear2", reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(linear2)), METH_FASTCALL, nullptr},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_pq_call", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__pq_call(void) { return PyModule_Create(&module); }
