// Python extension `_marshal`: the argument checks of the binding's compute calls and the calls themselves.
//
// In Python a call's checks, shape look-ups and ctypes conversions take 8 us beside 2 us for each launch, more than the
// kernels of a small layer take.  Here they are reads of the tensors' C++ objects, a few tenths of a microsecond.
//
// Every function takes the positional arguments of its namesake in the binding, with a descriptor's plan in the place of the
// descriptor, and returns the status of the C entry point -- or None, without having called it, whenever something is not
// plainly in order: a tensor that is absent, of another type, shape or layout, of a Python subclass or without storage
// (tracing, functional transforms), a number or a stream that does not convert.  The binding then runs its own checks,
// which raise what they always raised or accept the argument.  Nothing is kept from one call for the next; a plan holds
// the descriptor and its shapes, which never change.  The GIL is released around the call, as ctypes does.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include "mi355conv.h"
#include "mi355ip.h"
#include "mi355pg.h"

namespace {

const char kTarget[] __attribute__((used)) = MARSHAL_TARGET;  // looked up in the built file, before it is loaded

struct Shape {
  int dims;
  int64_t d[4];
};

struct Plan {
  void* desc;
  Shape x, w, y, b;  // input, weights, output (and their gradients), bias
};

const char kConv[] = "mi355conv.conv_plan", kIp[] = "mi355conv.ip_plan";

void delete_plan(PyObject* capsule) { delete static_cast<Plan*>(PyCapsule_GetPointer(capsule, PyCapsule_GetName(capsule))); }

const Plan* plan_of(PyObject* o, const char* kind) {
  return PyCapsule_IsValid(o, kind) ? static_cast<const Plan*>(PyCapsule_GetPointer(o, kind)) : nullptr;
}

// A plain contiguous device tensor of the type and shape: its address (null if it is empty).
bool tensor(PyObject* o, at::ScalarType type, const Shape& s, void** out) {
  if (!THPVariable_CheckExact(o)) return false;
  const at::Tensor& t = THPVariable_Unpack(o);
  if (!t.defined() || !t.has_storage() || !t.is_cuda() || t.layout() != at::kStrided || t.scalar_type() != type) return false;
  if (!t.is_contiguous() || t.dim() != s.dims) return false;
  for (int i = 0; i < s.dims; ++i)
    if (t.size(i) != s.d[i]) return false;
  *out = t.data_ptr();
  return true;
}

bool optional_tensor(PyObject* o, at::ScalarType type, const Shape& s, void** out) {
  *out = nullptr;
  return o == Py_None || tensor(o, type, s, out);
}

bool workspace(PyObject* o, void** out, size_t* bytes) {
  *out = nullptr;
  *bytes = 0;
  if (o == Py_None) return true;
  if (!THPVariable_CheckExact(o)) return false;
  const at::Tensor& t = THPVariable_Unpack(o);
  if (!t.defined() || !t.has_storage() || !t.is_cuda() || t.layout() != at::kStrided || !t.is_contiguous()) return false;
  *out = t.data_ptr();
  *bytes = (size_t)t.numel() * t.element_size();
  return true;
}

bool stream(PyObject* o, void** out) {
  if (o == Py_None) {
    *out = c10::hip::getCurrentHIPStream().stream();
    return true;
  }
  PyObject* h = PyObject_GetAttrString(o, "cuda_stream");
  if (h) {
    if (PyLong_CheckExact(h)) *out = PyLong_AsVoidPtr(h);
    const bool ok = PyLong_CheckExact(h) && !PyErr_Occurred();
    Py_DECREF(h);
    if (ok) return true;
  }
  PyErr_Clear();
  return false;
}

bool number(PyObject* o, double* out) {
  if (!PyFloat_CheckExact(o) && !PyLong_CheckExact(o)) return false;
  *out = PyFloat_AsDouble(o);
  if (!PyErr_Occurred()) return true;
  PyErr_Clear();
  return false;
}

bool length(PyObject* o, int64_t* out) {
  if (!THPVariable_CheckExact(o)) return false;
  *out = THPVariable_Unpack(o).numel();
  return *out < ((int64_t)1 << 31);
}

template <typename Call>
PyObject* released(Call&& call) {
  int status;
  Py_BEGIN_ALLOW_THREADS
  status = call();
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(status);
}

// Runs `body` (which returns null for "not plainly in order") on `count` arguments; no C++ exception leaves.
template <typename Body>
PyObject* guarded(Py_ssize_t given, Py_ssize_t count, Body&& body) {
  if (given == count) {
    try {
      if (PyObject* r = body()) return r;
    } catch (...) {
    }
  }
  if (PyErr_Occurred()) PyErr_Clear();
  Py_RETURN_NONE;
}

typedef PyObject* const* Args;
constexpr at::ScalarType kInt = at::kInt;

template <typename T>
struct Conv;
template <>
struct Conv<float> {
  static constexpr at::ScalarType type = at::kFloat;
  static constexpr auto forward = &conv_forward;
  static constexpr auto backward_data = &conv_backward_data;
  static constexpr auto backward_filter = &conv_backward_filter;
  static constexpr auto backward_bias = &conv_backward_bias;
};
template <>
struct Conv<double> {
  static constexpr at::ScalarType type = at::kDouble;
  static constexpr auto forward = &conv_forward_f64;
  static constexpr auto backward_data = &conv_backward_data_f64;
  static constexpr auto backward_filter = &conv_backward_filter_f64;
  static constexpr auto backward_bias = &conv_backward_bias_f64;
};

template <typename T>
PyObject* py_conv_forward(PyObject*, Args a, Py_ssize_t n) {  // plan, x, w, bias, y, ws, stream
  return guarded(n, 7, [&]() -> PyObject* {
    const Plan* p = plan_of(a[0], kConv);
    void *x, *w, *b, *y, *ws, *s;
    size_t bytes;
    if (!p || !tensor(a[1], Conv<T>::type, p->x, &x) || !tensor(a[2], Conv<T>::type, p->w, &w) ||
        !optional_tensor(a[3], Conv<T>::type, p->b, &b) || !tensor(a[4], Conv<T>::type, p->y, &y) || !workspace(a[5], &ws, &bytes) ||
        !stream(a[6], &s))
      return nullptr;
    return released([&] {
      return Conv<T>::forward(static_cast<const conv_desc_t*>(p->desc), static_cast<T*>(x), static_cast<T*>(w), static_cast<T*>(b),
                              static_cast<T*>(y), ws, bytes, s);
    });
  });
}

template <typename T>
PyObject* py_conv_backward_data(PyObject*, Args a, Py_ssize_t n) {  // plan, w, dy, dx, ws, stream
  return guarded(n, 6, [&]() -> PyObject* {
    const Plan* p = plan_of(a[0], kConv);
    void *w, *dy, *dx, *ws, *s;
    size_t bytes;
    if (!p || !tensor(a[1], Conv<T>::type, p->w, &w) || !tensor(a[2], Conv<T>::type, p->y, &dy) ||
        !tensor(a[3], Conv<T>::type, p->x, &dx) || !workspace(a[4], &ws, &bytes) || !stream(a[5], &s))
      return nullptr;
    return released([&] {
      return Conv<T>::backward_data(static_cast<const conv_desc_t*>(p->desc), static_cast<T*>(w), static_cast<T*>(dy),
                                    static_cast<T*>(dx), ws, bytes, s);
    });
  });
}

template <typename T>
PyObject* py_conv_backward_filter(PyObject*, Args a, Py_ssize_t n) {  // plan, x, dy, dw, beta, ws, stream
  return guarded(n, 7, [&]() -> PyObject* {
    const Plan* p = plan_of(a[0], kConv);
    void *x, *dy, *dw, *ws, *s;
    size_t bytes;
    double beta;
    if (!p || !tensor(a[1], Conv<T>::type, p->x, &x) || !tensor(a[2], Conv<T>::type, p->y, &dy) ||
        !tensor(a[3], Conv<T>::type, p->w, &dw) || !number(a[4], &beta) || !workspace(a[5], &ws, &bytes) || !stream(a[6], &s))
      return nullptr;
    return released([&] {
      return Conv<T>::backward_filter(static_cast<const conv_desc_t*>(p->desc), static_cast<T*>(x), static_cast<T*>(dy),
                                      static_cast<T*>(dw), (T)beta, ws, bytes, s);
    });
  });
}

template <typename T>
PyObject* py_conv_backward_bias(PyObject*, Args a, Py_ssize_t n) {  // plan, dy, db, beta, ws, stream
  return guarded(n, 6, [&]() -> PyObject* {
    const Plan* p = plan_of(a[0], kConv);
    void *dy, *db, *ws, *s;
    size_t bytes;
    double beta;
    if (!p || !tensor(a[1], Conv<T>::type, p->y, &dy) || !tensor(a[2], Conv<T>::type, p->b, &db) || !number(a[3], &beta) ||
        !workspace(a[4], &ws, &bytes) || !stream(a[5], &s))
      return nullptr;
    return released([&] {
      return Conv<T>::backward_bias(static_cast<const conv_desc_t*>(p->desc), static_cast<T*>(dy), static_cast<T*>(db), (T)beta, ws,
                                    bytes, s);
    });
  });
}

PyObject* py_conv_backward_filter_bias(PyObject*, Args a, Py_ssize_t n) {  // plan, x, dy, dw, db, beta, ws, stream
  return guarded(n, 8, [&]() -> PyObject* {
    const Plan* p = plan_of(a[0], kConv);
    void *x, *dy, *dw, *db, *ws, *s;
    size_t bytes;
    double beta;
    if (!p || !tensor(a[1], at::kFloat, p->x, &x) || !tensor(a[2], at::kFloat, p->y, &dy) || !tensor(a[3], at::kFloat, p->w, &dw) ||
        !tensor(a[4], at::kFloat, p->b, &db) || !number(a[5], &beta) || !workspace(a[6], &ws, &bytes) || !stream(a[7], &s))
      return nullptr;
    return released([&] {
      return conv_backward_filter_bias(static_cast<const conv_desc_t*>(p->desc), static_cast<float*>(x), static_cast<float*>(dy),
                                       static_cast<float*>(dw), static_cast<float*>(db), (float)beta, ws, bytes, s);
    });
  });
}

PyObject* py_ip_forward(PyObject*, Args a, Py_ssize_t n) {  // plan, x, w, bias, y, ws, stream
  return guarded(n, 7, [&]() -> PyObject* {
    const Plan* p = plan_of(a[0], kIp);
    void *x, *w, *b, *y, *ws, *s;
    size_t bytes;
    if (!p || !tensor(a[1], at::kFloat, p->x, &x) || !tensor(a[2], at::kFloat, p->w, &w) || !optional_tensor(a[3], at::kFloat, p->b, &b) ||
        !tensor(a[4], at::kFloat, p->y, &y) || !workspace(a[5], &ws, &bytes) || !stream(a[6], &s))
      return nullptr;
    return released([&] {
      return ip_forward(static_cast<const ip_desc_t*>(p->desc), static_cast<float*>(x), static_cast<float*>(w), static_cast<float*>(b),
                        static_cast<float*>(y), ws, bytes, s);
    });
  });
}

PyObject* py_ip_relu_backward(PyObject*, Args a, Py_ssize_t n) {  // plan, y, dy, dz, stream
  return guarded(n, 5, [&]() -> PyObject* {
    const Plan* p = plan_of(a[0], kIp);
    void *y, *dy, *dz, *s;
    if (!p || !optional_tensor(a[1], at::kFloat, p->y, &y) || !tensor(a[2], at::kFloat, p->y, &dy) ||
        !tensor(a[3], at::kFloat, p->y, &dz) || !stream(a[4], &s))
      return nullptr;
    return released([&] {
      return ip_relu_backward(static_cast<const ip_desc_t*>(p->desc), static_cast<float*>(y), static_cast<float*>(dy),
                              static_cast<float*>(dz), s);
    });
  });
}

PyObject* py_ip_backward_data(PyObject*, Args a, Py_ssize_t n) {  // plan, w, dz, dx, ws, stream
  return guarded(n, 6, [&]() -> PyObject* {
    const Plan* p = plan_of(a[0], kIp);
    void *w, *dz, *dx, *ws, *s;
    size_t bytes;
    if (!p || !tensor(a[1], at::kFloat, p->w, &w) || !tensor(a[2], at::kFloat, p->y, &dz) || !tensor(a[3], at::kFloat, p->x, &dx) ||
        !workspace(a[4], &ws, &bytes) || !stream(a[5], &s))
      return nullptr;
    return released([&] {
      return ip_backward_data(static_cast<const ip_desc_t*>(p->desc), static_cast<float*>(w), static_cast<float*>(dz),
                              static_cast<float*>(dx), ws, bytes, s);
    });
  });
}

PyObject* py_ip_backward_filter(PyObject*, Args a, Py_ssize_t n) {  // plan, x, dz, dw, beta, ws, stream
  return guarded(n, 7, [&]() -> PyObject* {
    const Plan* p = plan_of(a[0], kIp);
    void *x, *dz, *dw, *ws, *s;
    size_t bytes;
    double beta;
    if (!p || !tensor(a[1], at::kFloat, p->x, &x) || !tensor(a[2], at::kFloat, p->y, &dz) || !tensor(a[3], at::kFloat, p->w, &dw) ||
        !number(a[4], &beta) || !workspace(a[5], &ws, &bytes) || !stream(a[6], &s))
      return nullptr;
    return released([&] {
      return ip_backward_filter(static_cast<const ip_desc_t*>(p->desc), static_cast<float*>(x), static_cast<float*>(dz),
                                static_cast<float*>(dw), (float)beta, ws, bytes, s);
    });
  });
}

PyObject* py_ip_backward_bias(PyObject*, Args a, Py_ssize_t n) {  // plan, dz, db, beta, ws, stream
  return guarded(n, 6, [&]() -> PyObject* {
    const Plan* p = plan_of(a[0], kIp);
    void *dz, *db, *ws, *s;
    size_t bytes;
    double beta;
    if (!p || !tensor(a[1], at::kFloat, p->y, &dz) || !tensor(a[2], at::kFloat, p->b, &db) || !number(a[3], &beta) ||
        !workspace(a[4], &ws, &bytes) || !stream(a[5], &s))
      return nullptr;
    return released([&] {
      return ip_backward_bias(static_cast<const ip_desc_t*>(p->desc), static_cast<float*>(dz), static_cast<float*>(db), (float)beta, ws,
                              bytes, s);
    });
  });
}

PyObject* py_pg_sigmoid_sample_action(PyObject*, Args a, Py_ssize_t n) {  // aprob, random, action, stream
  return guarded(n, 4, [&]() -> PyObject* {
    void *aprob, *random, *action, *s;
    int64_t steps;
    if (!length(a[0], &steps)) return nullptr;
    const Shape row = {1, {steps}};
    if (!tensor(a[0], at::kFloat, row, &aprob) || !tensor(a[1], at::kFloat, row, &random) || !tensor(a[2], kInt, row, &action) ||
        !stream(a[3], &s))
      return nullptr;
    return released([&] {
      return pg_sigmoid_sample_action(static_cast<float*>(aprob), static_cast<float*>(random), static_cast<int32_t*>(action),
                                      (int32_t)steps, s);
    });
  });
}

PyObject* py_pg_discount_rewards(PyObject*, Args a, Py_ssize_t n) {  // reward, episode_offsets, gamma, discounted, stream
  return guarded(n, 5, [&]() -> PyObject* {
    void *reward, *offsets, *discounted, *s;
    int64_t steps, ends;
    double gamma;
    if (!length(a[0], &steps) || !length(a[1], &ends)) return nullptr;
    const Shape row = {1, {steps}}, bounds = {1, {ends}};
    if (!tensor(a[0], at::kFloat, row, &reward) || !tensor(a[1], kInt, bounds, &offsets) || !number(a[2], &gamma) ||
        !tensor(a[3], at::kFloat, row, &discounted) || !stream(a[4], &s))
      return nullptr;
    return released([&] {
      return pg_discount_rewards(static_cast<float*>(reward), static_cast<int32_t*>(offsets), (int32_t)(ends - 1), (int32_t)steps,
                                 (float)gamma, static_cast<float*>(discounted), s);
    });
  });
}

PyObject* py_pg_sigmoid_bottom_diff(PyObject*, Args a, Py_ssize_t n) {  // aprob, action, discounted, dlogps, bottom_diff, stream
  return guarded(n, 6, [&]() -> PyObject* {
    void *aprob, *action, *discounted, *dlogps, *diff, *s;
    int64_t steps;
    if (!length(a[0], &steps)) return nullptr;
    const Shape row = {1, {steps}};
    if (!tensor(a[0], at::kFloat, row, &aprob) || !tensor(a[1], kInt, row, &action) || !optional_tensor(a[2], at::kFloat, row, &discounted) ||
        !optional_tensor(a[3], at::kFloat, row, &dlogps) || !tensor(a[4], at::kFloat, row, &diff) || !stream(a[5], &s))
      return nullptr;
    return released([&] {
      return pg_sigmoid_bottom_diff(static_cast<float*>(aprob), static_cast<int32_t*>(action), static_cast<float*>(discounted),
                                    static_cast<float*>(dlogps), static_cast<float*>(diff), (int32_t)steps, s);
    });
  });
}

PyObject* py_pg_softmax_bottom_diff(PyObject*, Args a, Py_ssize_t n) {  // logits, action, discounted, probs, bottom_diff, stream
  return guarded(n, 6, [&]() -> PyObject* {
    if (!THPVariable_CheckExact(a[0])) return nullptr;
    const at::Tensor& t = THPVariable_Unpack(a[0]);
    if (t.dim() != 2 || t.size(0) >= ((int64_t)1 << 31) || t.size(1) >= ((int64_t)1 << 31)) return nullptr;
    const Shape all = {2, {t.size(0), t.size(1)}}, row = {1, {t.size(0)}};
    void *logits, *action, *discounted, *probs, *diff, *s;
    if (!tensor(a[0], at::kFloat, all, &logits) || !tensor(a[1], kInt, row, &action) || !optional_tensor(a[2], at::kFloat, row, &discounted) ||
        !optional_tensor(a[3], at::kFloat, all, &probs) || !tensor(a[4], at::kFloat, all, &diff) || !stream(a[5], &s))
      return nullptr;
    return released([&] {
      return pg_softmax_bottom_diff(static_cast<float*>(logits), static_cast<int32_t*>(action), static_cast<float*>(discounted),
                                    static_cast<float*>(probs), static_cast<float*>(diff), (int32_t)all.d[0], (int32_t)all.d[1], s);
    });
  });
}

PyObject* new_plan(const Plan& p, const char* kind) {
  Plan* own = new (std::nothrow) Plan(p);
  if (!own) return PyErr_NoMemory();
  PyObject* c = PyCapsule_New(own, kind, &delete_plan);
  if (!c) delete own;
  return c;
}

PyObject* py_conv_plan(PyObject*, PyObject* args) {  // handle, (n, c, h, w), (num_output, c/group, kh, kw), (n, num_output, oh, ow)
  unsigned long long handle;
  Plan p = {};
  p.x.dims = p.w.dims = p.y.dims = 4;
  p.b.dims = 1;
  if (!PyArg_ParseTuple(args, "K(LLLL)(LLLL)(LLLL)", &handle, p.x.d, p.x.d + 1, p.x.d + 2, p.x.d + 3, p.w.d, p.w.d + 1, p.w.d + 2,
                        p.w.d + 3, p.y.d, p.y.d + 1, p.y.d + 2, p.y.d + 3))
    return nullptr;
  p.desc = reinterpret_cast<void*>(handle);
  p.b.d[0] = p.w.d[0];
  return new_plan(p, kConv);
}

PyObject* py_ip_plan(PyObject*, PyObject* args) {  // handle, m, k, num_output
  unsigned long long handle;
  long long m, k, o;
  if (!PyArg_ParseTuple(args, "KLLL", &handle, &m, &k, &o)) return nullptr;
  return new_plan(Plan{reinterpret_cast<void*>(handle), {2, {m, k}}, {2, {o, k}}, {2, {m, o}}, {1, {o}}}, kIp);
}

#define FAST(name, fn) {name, (PyCFunction)(void (*)(void))(PyObject * (*)(PyObject*, Args, Py_ssize_t)) & fn, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    {"conv_plan", py_conv_plan, METH_VARARGS, nullptr},
    {"ip_plan", py_ip_plan, METH_VARARGS, nullptr},
    FAST("conv_forward", py_conv_forward<float>),
    FAST("conv_forward_f64", py_conv_forward<double>),
    FAST("conv_backward_data", py_conv_backward_data<float>),
    FAST("conv_backward_data_f64", py_conv_backward_data<double>),
    FAST("conv_backward_filter", py_conv_backward_filter<float>),
    FAST("conv_backward_filter_f64", py_conv_backward_filter<double>),
    FAST("conv_backward_bias", py_conv_backward_bias<float>),
    FAST("conv_backward_bias_f64", py_conv_backward_bias<double>),
    FAST("conv_backward_filter_bias", py_conv_backward_filter_bias),
    FAST("ip_forward", py_ip_forward),
    FAST("ip_relu_backward", py_ip_relu_backward),
    FAST("ip_backward_data", py_ip_backward_data),
    FAST("ip_backward_filter", py_ip_backward_filter),
    FAST("ip_backward_bias", py_ip_backward_bias),
    FAST("pg_sigmoid_sample_action", py_pg_sigmoid_sample_action),
    FAST("pg_discount_rewards", py_pg_discount_rewards),
    FAST("pg_sigmoid_bottom_diff", py_pg_sigmoid_bottom_diff),
    FAST("pg_softmax_bottom_diff", py_pg_softmax_bottom_diff),
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal() { return PyModule_Create(&module); }
