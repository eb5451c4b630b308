// The device-side calls of the Python binding, for plain tensors: the same checks, pointers and stream as
// binding.py, without the interpreter.  A call with anything out of the ordinary (a tensor subclass, a wrong
// type or size, a tensor without storage) returns kNotHere before anything was done: binding.py then takes it,
// and says what is wrong.
//
// A small tensor's call is host time, nearly all of it the launches, about 3 us each: compressing in one kernel 3.2 us where the host
// is fast, of which 0.1 are the wrapper's in binding.py, and 5.1 where it is slow, in two there 7.7.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/ATen.h>
#include <torch/csrc/autograd/python_variable.h>

#include "accept.h"

namespace {

constexpr long kNotHere = -1;
PyObject* g_get_device = nullptr;  // torch._C._cuda_getDevice, torch._C._cuda_getCurrentRawStream
PyObject* g_get_stream = nullptr;

// accept_desc inside the binding's ctypes structure, for the length of a call.
struct DescView {
  Py_buffer view{};
  bool held = false;
  const accept_desc* get(PyObject* o) {
    if (PyObject_GetBuffer(o, &view, PyBUF_SIMPLE) != 0) {
      PyErr_Clear();
      return nullptr;
    }
    held = true;
    return view.len == Py_ssize_t(sizeof(accept_desc)) ? static_cast<const accept_desc*>(view.buf) : nullptr;
  }
  ~DescView() {
    if (held) PyBuffer_Release(&view);
  }
};

bool current_stream(void** stream) {
  PyObject* device = PyObject_CallNoArgs(g_get_device);
  PyObject* raw = device ? PyObject_CallOneArg(g_get_stream, device) : nullptr;
  Py_XDECREF(device);
  if (raw) *stream = PyLong_AsVoidPtr(raw);
  Py_XDECREF(raw);
  if (!PyErr_Occurred()) return true;
  PyErr_Clear();
  return false;
}

const at::Tensor* plain_tensor(PyObject* o) { return THPVariable_CheckExact(o) ? &THPVariable_Unpack(o) : nullptr; }

bool fits(const at::Tensor* t, size_t bytes) {
  return t && t->is_cuda() && size_t(t->numel()) * t->element_size() >= bytes && t->is_contiguous();
}
bool fits(const at::Tensor* t, int dtype, int64_t elems) {
  return t && t->scalar_type() == (dtype == ACCEPT_BF16 ? at::kBFloat16 : at::kFloat) && t->is_cuda() &&
         t->numel() >= elems && t->is_contiguous();
}

// compress(desc, x, alpha_prev or None, header, payload, workspace, first) -> status or kNotHere
PyObject* compress(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
  if (nargs != 7) return PyLong_FromLong(kNotHere);
  try {
    DescView dv;
    const accept_desc* d = dv.get(args[0]);
    size_t hb = 0, pb = 0, wb = 0;
    if (!d || accept_packed_size(d, &hb, &pb) != ACCEPT_OK || accept_workspace_size(d, &wb) != ACCEPT_OK)
      return PyLong_FromLong(kNotHere);
    const bool first = args[6] == Py_True;
    const bool alpha_used = d->scheme == ACCEPT_MBQ && !first;
    const at::Tensor *x = plain_tensor(args[1]), *alpha = args[2] == Py_None ? nullptr : plain_tensor(args[2]);
    const at::Tensor *header = plain_tensor(args[3]), *payload = plain_tensor(args[4]), *ws = plain_tensor(args[5]);
    void* stream = nullptr;
    if (!fits(x, d->in_dtype, d->n * d->m) || !fits(header, hb) || !fits(payload, pb) || !fits(ws, wb) ||
        (alpha_used && !fits(alpha, ACCEPT_F32, d->bits)) || (!alpha && args[2] != Py_None) || !current_stream(&stream))
      return PyLong_FromLong(kNotHere);
    const void* xp = x->data_ptr();
    const float* ap = alpha ? static_cast<const float*>(alpha->data_ptr()) : nullptr;
    void *hp = header->data_ptr(), *pp = payload->data_ptr(), *wp = ws->data_ptr();
    accept_status st;
    Py_BEGIN_ALLOW_THREADS
    st = first ? accept_mbq_compress_first(d, xp, hp, pp, wp, stream) : accept_compress(d, xp, ap, hp, pp, wp, stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(st);
  } catch (const std::exception&) {  // a tensor that has no storage, for one
    return PyLong_FromLong(kNotHere);
  }
}

// Other Python threads run on while this lives.
struct Unlocked {
  PyThreadState* state = PyEval_SaveThread();
  ~Unlocked() { PyEval_RestoreThread(state); }
};

// decompress(desc, header, payload, out or None) -> status, or where there was no `out` the tensor made for it, or kNotHere
PyObject* decompress(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
  if (nargs != 4) return PyLong_FromLong(kNotHere);
  try {
    DescView dv;
    const accept_desc* d = dv.get(args[0]);
    size_t hb = 0, pb = 0;
    if (!d || accept_packed_size(d, &hb, &pb) != ACCEPT_OK) return PyLong_FromLong(kNotHere);
    const at::Tensor *header = plain_tensor(args[1]), *payload = plain_tensor(args[2]);
    const bool make = args[3] == Py_None;
    const at::Tensor* out = make ? nullptr : plain_tensor(args[3]);
    void* stream = nullptr;
    if (!fits(header, hb) || !fits(payload, pb) || (!make && !fits(out, d->out_dtype, d->n * d->m)) || !current_stream(&stream))
      return PyLong_FromLong(kNotHere);
    at::Tensor made;
    if (make) {
      const Unlocked unlocked;  // as in torch.empty: memory that has to be made or freed first waits for the device, and with it for what other threads do for it
      made = at::empty({d->n * d->m}, payload->options().dtype(d->out_dtype == ACCEPT_BF16 ? at::kBFloat16 : at::kFloat));
      out = &made;
    }
    const void *hp = header->data_ptr(), *pp = payload->data_ptr();
    void* op = out->data_ptr();
    accept_status st;
    Py_BEGIN_ALLOW_THREADS
    st = accept_decompress(d, hp, pp, op, stream);
    Py_END_ALLOW_THREADS
    return make && st == ACCEPT_OK ? THPVariable_Wrap(made) : PyLong_FromLong(st);
  } catch (const std::exception&) {
    return PyLong_FromLong(kNotHere);
  }
}

PyMethodDef methods[] = {
    {"compress", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(compress)), METH_FASTCALL, nullptr},
    {"decompress", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(decompress)), METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module_def = {PyModuleDef_HEAD_INIT, "_native", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native(void) {
  PyObject* torch_c = PyImport_ImportModule("torch._C");
  if (!torch_c) return nullptr;
  g_get_device = PyObject_GetAttrString(torch_c, "_cuda_getDevice");
  g_get_stream = PyObject_GetAttrString(torch_c, "_cuda_getCurrentRawStream");
  Py_DECREF(torch_c);
  if (!g_get_device || !g_get_stream) return nullptr;
  return PyModule_Create(&module_def);
}
