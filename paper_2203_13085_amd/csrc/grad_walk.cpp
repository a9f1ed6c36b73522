// A walk over a list of torch parameters' gradients in native code: p.grad costs 95 ns from Python, and an optimizer
// over K replicas asks for hundreds of them twice an iteration (632 tensors: 60 us to see that none is
// missing, 60 more to gather them).  Host code only; nothing is kept between calls.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <c10/core/impl/COW.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/csrc/autograd/variable.h>

namespace {

enum State : long { PLAIN = 0, OTHER = 1, MISSING = 2 };

// A gradient that its buffer stands for entirely: dense, contiguous, of the parameter's own size, type and device, with
// a buffer of its own (a lazy clone's is shared until one side writes), and without anything that an operation on it would
// have to record or hand on (autograd history, forward-mode tangents, transforms, subclasses in C++ or in Python).
bool plain(const at::Tensor &p, const at::Tensor &g)
{
    const c10::TensorImpl *impl = g.unsafeGetTensorImpl();
    static const c10::DispatchKeySet wrapped({c10::DispatchKey::FuncTorchBatched, c10::DispatchKey::FuncTorchGradWrapper,
                                              c10::DispatchKey::Functionalize, c10::DispatchKey::Batched,
                                              c10::DispatchKey::Conjugate, c10::DispatchKey::Negative,
                                              c10::DispatchKey::ZeroTensor});
    const PyObject *seen = impl->pyobj_slot()->load_pyobj();       // none: Python has never seen it, so it is no subclass there
    return (!seen || (PyObject *)Py_TYPE(seen) == THPVariableClass) && !impl->is_python_dispatch() && !impl->key_set().has_any(wrapped) && g.layout() == c10::kStrided &&
           !g.is_inference() && !g.requires_grad() && !g._fw_grad(0).defined() && g.scalar_type() == p.scalar_type() &&
           g.device() == p.device() && g.numel() == p.numel() && g.is_contiguous() &&
           !c10::impl::cow::is_cow_data_ptr(g.storage().data_ptr());
}

// A buffer of n 64-bit values, or nothing for None; false with an exception set where it is neither.
struct Column {
    Py_buffer view{};
    const uint64_t *at = nullptr;
    bool take(PyObject *o, Py_ssize_t n, const char *what)
    {
        if (o == Py_None) return true;
        if (PyObject_GetBuffer(o, &view, PyBUF_SIMPLE) != 0) return false;
        at = static_cast<const uint64_t *>(view.buf);
        if (view.len == n * (Py_ssize_t)sizeof(uint64_t)) return true;
        PyErr_SetString(PyExc_ValueError, what);
        return false;
    }
    ~Column()
    {
        if (view.obj) PyBuffer_Release(&view);
    }
};

// state(params, type, addresses or None, touch, sizes = None) -> PLAIN, OTHER or MISSING (some gradient is None).
// PLAIN: every entry of `params` is exactly a `type` and has a gradient; with addresses also: it is plain, at its address, and
// with sizes as many bytes long as was bound there (a parameter may have been cut down together with its gradient).
// touch: if PLAIN, the gradients' version counters go up by one, as after an operation in place.
PyObject *state(PyObject *, PyObject *args)
{
    PyObject *params, *type, *addresses, *sizes = Py_None;
    int touch;
    if (!PyArg_ParseTuple(args, "O!OOp|O", &PyList_Type, &params, &type, &addresses, &touch, &sizes)) return nullptr;
    const Py_ssize_t n = PyList_GET_SIZE(params);
    Column address, size;
    if (!address.take(addresses, n, "one address for every parameter") || !size.take(sizes, n, "one size for every parameter"))
        return nullptr;
    long found = PLAIN;
    try {
        for (Py_ssize_t i = 0; i < n && found != MISSING; ++i) {
            PyObject *o = PyList_GET_ITEM(params, i);
            if ((PyObject *)Py_TYPE(o) != type || !THPVariable_Check(o)) {
                found = OTHER;
                break;
            }
            const at::Tensor &p = THPVariable_Unpack(o);
            const at::Tensor &g = p.grad();
            if (!g.defined()) found = MISSING;
            else if (address.at && found == PLAIN &&
                     !(plain(p, g) && (uint64_t)(uintptr_t)g.const_data_ptr() == address.at[i] &&
                       (!size.at || (uint64_t)g.nbytes() == size.at[i])))
                found = OTHER;
        }
        if (found == PLAIN && touch)
            for (Py_ssize_t i = 0; i < n; ++i)
                torch::autograd::impl::bump_version(THPVariable_Unpack(PyList_GET_ITEM(params, i)).grad());
    } catch (const std::exception &e) {
        PyErr_SetString(PyExc_RuntimeError, e.what());
        return nullptr;
    }
    return PyLong_FromLong(found);
}

PyMethodDef methods[] = {{"state", state, METH_VARARGS, "What a list of parameters' gradients are: 0 plain, 1 other, 2 one is missing."},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_grad_walk", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

} // namespace

PyMODINIT_FUNC PyInit__grad_walk()
{
    PyObject *m = PyModule_Create(&module);
    if (m && PyModule_AddStringConstant(m, "torch_version", LASGD_TORCH_VERSION) != 0) Py_CLEAR(m);
    return m;
}
