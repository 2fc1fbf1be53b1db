// binding.cpp -- the calls on torch tensors without Python between them.
//
// fwd, bwd and the drop-in layer take 10-11 us of host time per call through
// ctypes (checks, allocations, the stream, argument conversion; the launch
// itself takes 3), which bounds every tensor below a few million elements, and
// a Python autograd function adds a hand-over of the interpreter lock to the
// backward.  Here the same steps run in C++.
//
// Each entry handles the plain case only: exact torch tensors on one GPU, dense,
// contiguous, of the right types and sizes, outside of tracing, dispatch and
// function modes, functorch transforms and forward-mode AD.  For everything
// else it returns None before it has done anything, and the caller takes the
// general Python path, which also raises what a wrong argument raises.
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/function.h>
#include <torch/csrc/autograd/functions/utils.h>
#include <torch/csrc/autograd/python_cpp_function.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/csrc/autograd/saved_variable.h>
#include <torch/csrc/dynamo/compiled_autograd.h>
#include <torch/csrc/jit/frontend/tracer.h>
#include <torch/csrc/utils/object_ptr.h>
#include <torch/csrc/utils/pybind.h>

#include <ATen/ATen.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <ATen/SequenceNumber.h>
#include <ATen/hip/impl/HIPStreamMasqueradingAsCUDA.h>
#include <ATen/record_function.h>
#include <c10/core/DeviceGuard.h>
#include <c10/core/impl/LocalDispatchKeySet.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>

#include <algorithm>
#include <cstring>
#include <mutex>
#include <string>
#include <typeinfo>
#include <vector>

#include "fewbit.h"

namespace {

using torch::autograd::variable_list;

// The general backward of the package, (table bytes, grad, codes) -> grad_in,
// and its exception class, (status, where); set once at import.
PyObject* general_bwd = nullptr;
PyObject* error_class = nullptr;

// Storage type of the C ABI, or -1.
int storage_type(const at::Tensor& t) {
  switch (t.scalar_type()) {
    case at::kFloat: return FEWBIT_F32;
    case at::kHalf: return FEWBIT_F16;
    case at::kBFloat16: return FEWBIT_BF16;
    default: return -1;
  }
}

// Nothing watches or rewrites tensor operations on this thread.
bool plain_mode() {
  return !c10::impl::TorchDispatchModeTLS::any_modes_set() && !at::impl::torch_function_mode_enabled() &&
         !torch::jit::tracer::isTracing() &&
         !c10::impl::tls_is_dispatch_key_included(c10::DispatchKey::FuncTorchDynamicLayerFrontMode) &&
         !c10::impl::tls_is_dispatch_key_included(c10::DispatchKey::PythonTLSSnapshot);
}

// An ordinary dense device tensor, not a wrapper and not a lazy view.
bool plain(const at::Tensor& t) {
  constexpr c10::DispatchKeySet kOdd({c10::DispatchKey::Python, c10::DispatchKey::FuncTorchGradWrapper,
                                      c10::DispatchKey::FuncTorchBatched, c10::DispatchKey::Functionalize,
                                      c10::DispatchKey::ZeroTensor, c10::DispatchKey::Conjugate,
                                      c10::DispatchKey::Negative});
  return t.is_cuda() && t.layout() == at::kStrided && !t.key_set().has_any(kOdd);
}

const at::Tensor* plain_tensor(PyObject* o) {
  if (!THPVariable_CheckExact(o)) return nullptr;
  const at::Tensor& t = THPVariable_Unpack(o);
  return plain(t) && t.is_contiguous() ? &t : nullptr;
}

bool like(const at::Tensor& t, const at::Tensor& ref) {
  return t.device() == ref.device() && t.scalar_type() == ref.scalar_type() && t.numel() == ref.numel();
}

bool codes_fit(const at::Tensor& codes, const at::Tensor& ref, int bits) {
  return codes.device() == ref.device() && codes.scalar_type() == at::kInt &&
         codes.numel() >= fewbit_packed_words(ref.numel(), bits);
}

// The table, copied out of the ctypes structure; false if o is not one.
bool table_of(PyObject* o, fewbit_table* t) {
  Py_buffer b;
  if (PyObject_GetBuffer(o, &b, PyBUF_SIMPLE) != 0) {
    PyErr_Clear();
    return false;
  }
  const bool ok = b.len == static_cast<Py_ssize_t>(sizeof *t);
  if (ok) std::memcpy(t, b.buf, sizeof *t);
  PyBuffer_Release(&b);
  return ok && t->bits >= 1 && t->bits <= 4;
}

void* stream_of(const at::Tensor& t) {
  return c10::hip::getCurrentHIPStreamMasqueradingAsCUDA(t.device().index()).stream();
}

at::Tensor new_codes(const at::Tensor& x, int bits) {
  const int64_t words = std::max<int64_t>(fewbit_packed_words(x.numel(), bits), 1);
  return at::empty({words}, at::TensorOptions().dtype(at::kInt).device(x.device()));
}

int run_fwd(const fewbit_table& t, const at::Tensor& x, const at::Tensor& y, const at::Tensor& codes) {
  return fewbit_fwd(&t, storage_type(x), x.data_ptr(), y.data_ptr(), static_cast<uint32_t*>(codes.data_ptr()),
                    x.numel(), stream_of(x));
}

int run_bwd(const fewbit_table& t, const at::Tensor& g, const at::Tensor& codes, const at::Tensor& gin) {
  return fewbit_bwd(&t, storage_type(g), g.data_ptr(), static_cast<const uint32_t*>(codes.data_ptr()),
                    gin.data_ptr(), g.numel(), stream_of(g));
}

// ---------------------------------------------------------------- direct calls
// fwd(table, x, y or None, codes or None) -> (y, codes), a status, or None
PyObject* fwd(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
  HANDLE_TH_ERRORS
  fewbit_table t;
  if (nargs != 4 || !table_of(args[0], &t) || !plain_mode()) Py_RETURN_NONE;
  const at::Tensor* x = plain_tensor(args[1]);
  if (!x || storage_type(*x) < 0) Py_RETURN_NONE;
  const bool own_y = args[2] == Py_None, own_codes = args[3] == Py_None;
  at::Tensor y, codes;
  if (!own_y) {
    const at::Tensor* p = plain_tensor(args[2]);
    if (!p || !like(*p, *x)) Py_RETURN_NONE;
    y = *p;
  }
  if (!own_codes) {
    const at::Tensor* p = plain_tensor(args[3]);
    if (!p || !codes_fit(*p, *x, t.bits)) Py_RETURN_NONE;
    codes = *p;
  }
  int rc;
  {
    pybind11::gil_scoped_release no_gil;
    at::AutoDispatchBelowADInplaceOrView below;
    const c10::DeviceGuard guard(x->device());
    if (own_y) y = at::empty_like(*x);
    if (own_codes) codes = new_codes(*x, t.bits);
    rc = run_fwd(t, *x, y, codes);
  }
  if (rc != FEWBIT_OK) return PyLong_FromLong(rc);
  PyObject* oy = own_y ? THPVariable_Wrap(y) : Py_NewRef(args[2]);
  PyObject* oc = own_codes ? THPVariable_Wrap(codes) : Py_NewRef(args[3]);
  PyObject* r = oy && oc ? PyTuple_Pack(2, oy, oc) : nullptr;
  Py_XDECREF(oy);
  Py_XDECREF(oc);
  return r;
  END_HANDLE_TH_ERRORS
}

// bwd(table, grad_out, codes, grad_in or None) -> grad_in, a status, or None
PyObject* bwd(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
  HANDLE_TH_ERRORS
  fewbit_table t;
  if (nargs != 4 || !table_of(args[0], &t) || !plain_mode()) Py_RETURN_NONE;
  const at::Tensor* g = plain_tensor(args[1]);
  if (!g || storage_type(*g) < 0) Py_RETURN_NONE;
  const at::Tensor* codes = plain_tensor(args[2]);
  if (!codes || !codes_fit(*codes, *g, t.bits)) Py_RETURN_NONE;
  const bool own = args[3] == Py_None;
  at::Tensor gin;
  if (!own) {
    const at::Tensor* p = plain_tensor(args[3]);
    if (!p || !like(*p, *g)) Py_RETURN_NONE;
    gin = *p;
  }
  int rc;
  {
    pybind11::gil_scoped_release no_gil;
    at::AutoDispatchBelowADInplaceOrView below;
    const c10::DeviceGuard guard(g->device());
    if (own) gin = at::empty_like(*g);
    rc = run_bwd(t, *g, *codes, gin);
  }
  if (rc != FEWBIT_OK) return PyLong_FromLong(rc);
  return own ? THPVariable_Wrap(gin) : Py_NewRef(args[3]);
  END_HANDLE_TH_ERRORS
}

// ---------------------------------------------------------------- autograd
[[noreturn]] void throw_python() {
  python_error e;
  e.persist();
  throw e;
}

// The gradient of one call of the layer.
at::Tensor layer_grad(const fewbit_table& t, const at::Tensor& grad, const at::Tensor& codes) {
  const at::Tensor g = grad.contiguous();
  if (plain_mode() && plain(g) && storage_type(g) >= 0 && plain(codes) && codes.is_contiguous() &&
      codes_fit(codes, g, t.bits)) {
    at::AutoDispatchBelowADInplaceOrView below;
    const c10::DeviceGuard guard(g.device());
    at::Tensor gin = at::empty_like(g);
    const int rc = run_bwd(t, g, codes, gin);
    if (rc == FEWBIT_OK) return gin;
    pybind11::gil_scoped_acquire gil;
    if (PyObject* e = PyObject_CallFunction(error_class, "is", rc, "fewbit_bwd")) {
      PyErr_SetObject(error_class, e);
      Py_DECREF(e);
    }
    throw_python();
  }
  // codes that a hook has moved or replaced, a gradient of another kind
  pybind11::gil_scoped_acquire gil;
  THPObjectPtr og(THPVariable_Wrap(g)), oc(THPVariable_Wrap(codes));
  THPObjectPtr ot(PyBytes_FromStringAndSize(reinterpret_cast<const char*>(&t), sizeof t));
  if (!og || !oc || !ot) throw_python();
  THPObjectPtr r(PyObject_CallFunctionObjArgs(general_bwd, ot.get(), og.get(), oc.get(), nullptr));
  if (!r) throw_python();
  return THPVariable_Unpack(r.get());
}

// The table's bytes as text ('a' .. 'p', two letters a byte) and back:
// compiled autograd takes a call's constants as values of its own types.
std::string text_of(const fewbit_table& t) {
  const auto* b = reinterpret_cast<const unsigned char*>(&t);
  std::string s;
  s.reserve(2 * sizeof t);
  for (size_t i = 0; i < sizeof t; ++i) {
    s += static_cast<char>('a' + (b[i] >> 4));
    s += static_cast<char>('a' + (b[i] & 15));
  }
  return s;
}

fewbit_table table_of_text(const std::string& s) {
  fewbit_table t;
  TORCH_CHECK(s.size() == 2 * sizeof t, "not a table");
  auto* b = reinterpret_cast<unsigned char*>(&t);
  for (size_t i = 0; i < sizeof t; ++i)
    b[i] = static_cast<unsigned char>(((s[2 * i] - 'a') << 4) | (s[2 * i + 1] - 'a'));
  return t;
}

// The layer's node: saves the packed codes alone (saved-tensor hooks see them)
// and a copy of the table.
struct FewBitNode : public torch::autograd::Node {
  torch::autograd::SavedVariable codes_;
  fewbit_table table_;

  std::string name() const override { return "FewBitActivationBackward"; }
  at::Tensor codes() {
    std::lock_guard<std::mutex> lock(mutex_);
    return codes_.unpack();
  }
  void release_variables() override {
    std::lock_guard<std::mutex> lock(mutex_);
    codes_.reset_data();
  }

  variable_list apply(variable_list&& grads) override {
    const at::Tensor saved = codes();
    if (!task_should_compute_output(0)) return {at::Tensor()};
    return {layer_grad(table_, grads[0].defined() ? grads[0] : input_metadata(0).zeros_like(), saved)};
  }

  // Compiled autograd: the codes are an input of the compiled graph, the table
  // one of its constants, and the gradient an opaque call in it (as a Python
  // function's backward is), never traced through.
  void compiled_args(torch::dynamo::autograd::CompiledNodeArgs& args) const override {
    args.collect(codes_, /*is_output=*/false);
    args.collect(text_of(table_));
  }

  variable_list apply_with_saved(const variable_list& grads, torch::dynamo::autograd::SwapSavedVariables& saved) override {
    namespace ca = torch::dynamo::autograd;
    using Outputs = std::vector<std::optional<torch::autograd::InputMetadata>>;
    saved.before(codes_);
    ca::PackedArgs args;
    args.pack(codes_.unpack());
    args.pack(text_of(table_));
    const auto& compiler = ca::getPyCompilerInterface();
    const std::string fn = compiler->bind_function(
        saved.get_py_compiler(), name(),
        [](const variable_list& g, const std::vector<c10::IValue>& a) -> variable_list {
          if (!g[0].defined()) return {at::Tensor()};
          return {layer_grad(table_of_text(a[1].toStringRef()), g[0], a[0].toTensor())};
        },
        {at::TensorType::get(), at::StringType::get()}, /*is_custom_function=*/true, /*is_traceable=*/false);
    variable_list out = compiler->call_function(saved.get_py_compiler(), "apply_functional", fn, grads, args.vec(),
                                                ca::IValuePacker<Outputs>::pack(ca::get_input_metadata(next_edges())));
    saved.after(codes_);
    return out;
  }
};

// grad_fn.saved_tensors, as a Python function's has it
PyObject* saved_tensors(PyObject* self, void*) {
  HANDLE_TH_ERRORS
  auto* node = static_cast<FewBitNode*>(reinterpret_cast<torch::autograd::THPCppFunction*>(self)->cdata.get());
  at::Tensor codes;
  {
    pybind11::gil_scoped_release no_gil;
    codes = node->codes();
  }
  THPObjectPtr oc(THPVariable_Wrap(codes));
  return oc ? PyTuple_Pack(1, oc.get()) : nullptr;
  END_HANDLE_TH_ERRORS
}

using namespace torch::autograd;      // the properties macro names its getters without it
PyTypeObject node_type;
PyGetSetDef node_properties[] = {THP_FUNCTION_DEFAULT_PROPERTIES,
                                 {"saved_tensors", saved_tensors, nullptr, nullptr, nullptr},
                                 {nullptr, nullptr, nullptr, nullptr, nullptr}};

// activation(table, x) -> y with its history, a status, or None
PyObject* activation(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
  HANDLE_TH_ERRORS
  fewbit_table t;
  if (nargs != 2 || !table_of(args[0], &t) || !plain_mode()) Py_RETURN_NONE;
  const at::Tensor* x = plain_tensor(args[1]);
  if (!x || storage_type(*x) < 0 || x->is_inference() || x->_fw_grad(0).defined()) Py_RETURN_NONE;
  at::Tensor y;
  int rc;
  {
    pybind11::gil_scoped_release no_gil;
    // the profiler's range of the call, as a Python function has it
    RECORD_FUNCTION("FewBitActivation", std::vector<c10::IValue>{*x}, static_cast<int64_t>(at::sequence_number::peek()));
    const c10::DeviceGuard device(x->device());
    at::Tensor codes;
    {
      at::AutoDispatchBelowADInplaceOrView below;
      y = at::empty_like(*x);
      codes = new_codes(*x, t.bits);
      rc = run_fwd(t, *x, y, codes);
    }
    if (rc == FEWBIT_OK && at::GradMode::is_enabled() && x->requires_grad()) {
      std::shared_ptr<FewBitNode> node(new FewBitNode(), torch::autograd::deleteNode);
      node->set_next_edges(torch::autograd::collect_next_edges(*x));
      node->codes_ = torch::autograd::SavedVariable(codes, false);
      node->table_ = t;
      torch::autograd::set_history(y, node);
    }
  }
  return rc == FEWBIT_OK ? THPVariable_Wrap(y) : PyLong_FromLong(rc);
  END_HANDLE_TH_ERRORS
}

// set_general(bwd of table bytes, error class)
PyObject* set_general(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
  if (nargs != 2) {
    PyErr_SetString(PyExc_TypeError, "set_general takes two arguments");
    return nullptr;
  }
  Py_XDECREF(general_bwd);
  Py_XDECREF(error_class);
  general_bwd = Py_NewRef(args[0]);
  error_class = Py_NewRef(args[1]);
  Py_RETURN_NONE;
}

template <PyObject* (*F)(PyObject*, PyObject* const*, Py_ssize_t)>
PyMethodDef method(const char* name) {
  return {name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(F)), METH_FASTCALL, nullptr};
}

PyMethodDef methods[] = {method<fwd>("fwd"), method<bwd>("bwd"), method<activation>("activation"),
                         method<set_general>("set_general"), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module_def = {PyModuleDef_HEAD_INIT, "_native", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native(void) {
  HANDLE_TH_ERRORS
  torch::autograd::_initFunctionPyTypeObject(node_type, "FewBitActivationBackward", node_properties, nullptr);
  torch::autograd::registerCppFunction(typeid(FewBitNode), &node_type);
  return PyModule_Create(&module_def);
  END_HANDLE_TH_ERRORS
}
