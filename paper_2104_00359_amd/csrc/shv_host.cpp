// The host side of the differentiable shading operations (ops.py): device
// memory, layout and the library calls of one forward or backward pass in one
// call from Python.  The autograd functions stay Python's; what they did per
// pass in two dozen Python-level tensor operations is here.  Per pass (300
// receivers, 16 spheres, 4 bands, when the GPU waits for the host): forward 47
// -> 22 us, backward 102 -> 85, of which 59 are what an autograd pass that does
// nothing takes.
//
// The library's entry points arrive as addresses (bind), so the library that
// the Python binding loaded is the one that runs.
#include <Python.h>

#include <ATen/ATen.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <string>
#include <vector>

#include "shv_soa.h"
#include "shvis.h"

namespace {

struct Api {
  decltype(&shv_last_error) last_error;
  decltype(&shv_status_string) status_string;
  decltype(&shv_render_saved_floats) render_saved_floats;
  decltype(&sh_render_forward) render_forward;
  decltype(&sh_render_backward) render_backward;
  decltype(&shv_saved_floats) saved_floats;
  decltype(&sh_visibility_forward) visibility_forward;
  decltype(&sh_visibility_backward) visibility_backward;
  decltype(&sh_shade_channels) shade_channels;
  decltype(&sh_shade_channels_backward) shade_channels_backward;
  decltype(&shv_internal_soa) soa;
};
constexpr int kApi = sizeof(Api) / sizeof(void*);
Api api;

// The interpreter lock, given up for a scope.
struct Unlocked {
  PyThreadState* state = PyEval_SaveThread();
  ~Unlocked() { PyEval_RestoreThread(state); }
};

void check(shv_status st, const char* what) {
  if (st == SHV_OK) return;
  throw std::runtime_error(std::string(what) + ": " + api.status_string(st) + " (" + std::to_string((int)st) +
                           "): " + api.last_error());
}

const at::Tensor& tensor(PyObject* o) {
  if (!THPVariable_Check(o)) throw std::runtime_error("expected a tensor");
  return THPVariable_Unpack(o);
}
void* pointer(PyObject* o) { return PyLong_AsVoidPtr(o); }
float* data(const at::Tensor& t) { return t.defined() ? static_cast<float*>(t.data_ptr()) : nullptr; }

at::Tensor f32(const at::Tensor& x) {
  at::Tensor d = x.detach();
  if (d.scalar_type() != at::kFloat) d = d.to(at::kFloat);
  return d.contiguous();
}
at::Tensor soa(const at::Tensor& x) {  // [P, C] -> [C, P]
  at::Tensor d = x.detach();
  if (d.scalar_type() != at::kFloat) d = d.to(at::kFloat);
  return d.t().contiguous();
}
at::Tensor empty(at::IntArrayRef size, const at::Tensor& like) {
  return at::empty(size, at::TensorOptions().dtype(at::kFloat).device(like.device()));
}

// Positions and normals, [P, 3] each, as [3, P]: in one launch where both are
// plain FP32 rows.  Always copies: the caller may write to its tensors before
// the backward pass.
std::pair<at::Tensor, at::Tensor> soa2(const at::Tensor& a, const at::Tensor& b, void* stream) {
  const int64_t P = a.size(0);
  if (P > 0 && a.scalar_type() == at::kFloat && b.scalar_type() == at::kFloat && a.is_contiguous() &&
      b.is_contiguous() && !a.is_neg() && !b.is_neg()) {
    at::Tensor x = empty({3, P}, a), y = empty({3, P}, a);
    check(api.soa(data(a), data(b), P, data(x), data(y), (hipStream_t)stream), "layout");
    return {x, y};
  }
  return {soa(a), soa(b)};
}

bool fits(PyObject* o, std::initializer_list<int64_t> shape, const at::Device& dev) {
  if (!THPVariable_Check(o)) return false;
  const at::Tensor& t = THPVariable_Unpack(o);
  if (!at::isFloatingType(t.scalar_type()) || t.dim() != (int64_t)shape.size() || t.device() != dev) return false;
  int64_t d = 0;
  for (int64_t w : shape)
    if (t.size(d++) != w) return false;
  return true;
}

PyObject* py_bind(PyObject*, PyObject* const* args, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  if (n != kApi) throw std::runtime_error("bind: wrong number of entry points");
  void** slot = reinterpret_cast<void**>(&api);
  for (Py_ssize_t i = 0; i < n; ++i) slot[i] = pointer(args[i]);
  if (PyErr_Occurred()) return nullptr;
  Py_RETURN_NONE;
  END_HANDLE_TH_ERRORS
}

// inputs_ok(points, normals, albedo, spheres, light, N): whether the
// inputs of shade_sh (light of one dimension) or shade_sh_channels (two) have the types, shapes
// and one HIP device that the operations ask for.
PyObject* py_inputs_ok(PyObject*, PyObject* const* a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  if (n != 6) throw std::runtime_error("inputs_ok: six arguments");
  const long long N = PyLong_AsLongLong(a[5]);
  if (PyErr_Occurred()) return nullptr;
  if (!THPVariable_Check(a[0]) || !THPVariable_Check(a[3]) || !THPVariable_Check(a[4])) Py_RETURN_FALSE;
  const at::Tensor &p = THPVariable_Unpack(a[0]), &s = THPVariable_Unpack(a[3]), &l = THPVariable_Unpack(a[4]);
  if (!p.device().is_cuda() || p.dim() != 2 || s.dim() != 2 || l.dim() < 1 || l.dim() > 2) Py_RETURN_FALSE;
  const int64_t P = p.size(0), S = s.size(0);
  const at::Device dev = p.device();
  bool ok = fits(a[0], {P, 3}, dev) && fits(a[1], {P, 3}, dev) && fits(a[3], {S, 4}, dev);
  if (l.dim() == 1) ok = ok && fits(a[2], {P}, dev) && fits(a[4], {N}, dev);
  else ok = ok && fits(a[2], {P, l.size(0)}, dev) && fits(a[4], {l.size(0), N}, dev);
  if (ok) Py_RETURN_TRUE;
  Py_RETURN_FALSE;
  END_HANDLE_TH_ERRORS
}

PyObject* tuple(const std::vector<at::Tensor>& ts) {  // undefined tensors as None
  PyObject* r = PyTuple_New((Py_ssize_t)ts.size());
  if (!r) return nullptr;
  for (size_t i = 0; i < ts.size(); ++i) {
    PyObject* o = ts[i].defined() ? THPVariable_Wrap(ts[i]) : Py_NewRef(Py_None);
    if (!o) {
      Py_DECREF(r);
      return nullptr;
    }
    PyTuple_SET_ITEM(r, (Py_ssize_t)i, o);
  }
  return r;
}

// shade_forward(points, normals, albedo, spheres, light, params, ws, stream)
//   -> radiance, points, normals, albedo, spheres (as the library takes them), vis, saved
PyObject* py_shade_forward(PyObject*, PyObject* const* a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  if (n != 8) throw std::runtime_error("shade_forward: eight arguments");
  const at::Tensor &points = tensor(a[0]), &normals = tensor(a[1]), &albedo = tensor(a[2]), &spheres = tensor(a[3]),
                   &light = tensor(a[4]), &ws = tensor(a[6]);
  const shv_params* prm = (const shv_params*)pointer(a[5]);
  void* stream = pointer(a[7]);
  if (PyErr_Occurred()) return nullptr;
  std::vector<at::Tensor> out;
  {
    Unlocked u;
    const int64_t P = points.size(0), S = spheres.size(0), N = (int64_t)prm->n_bands * prm->n_bands;
    auto [pts, nrm] = soa2(points, normals, stream);
    at::Tensor alb = f32(albedo), sph = f32(spheres), L = f32(light);
    at::Tensor vis = empty({N, P}, points), rad = empty({P}, points);
    at::Tensor saved = empty({std::max<int64_t>(api.render_saved_floats(P, prm), 1)}, points);
    check(api.render_forward(data(pts), data(nrm), data(alb), data(sph), data(L), P, S, prm, data(vis), data(rad),
                             data(saved), saved.numel() * 4, ws.data_ptr(), ws.numel(), (hipStream_t)stream),
          "sh_render_forward");
    out = {rad, pts, nrm, alb, sph, vis, saved};
  }
  return tuple(out);
  END_HANDLE_TH_ERRORS
}

// shade_backward(grad_radiance, points, normals, albedo, spheres, vis, saved, params, ws, stream, need x 5)
//   -> gradients of points [3, P], normals [3, P], albedo, spheres, light (None where not needed)
PyObject* py_shade_backward(PyObject*, PyObject* const* a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  if (n != 15) throw std::runtime_error("shade_backward: fifteen arguments");
  const at::Tensor &grad = tensor(a[0]), &pts = tensor(a[1]), &nrm = tensor(a[2]), &alb = tensor(a[3]),
                   &sph = tensor(a[4]), &vis = tensor(a[5]), &saved = tensor(a[6]), &ws = tensor(a[8]);
  const shv_params* prm = (const shv_params*)pointer(a[7]);
  void* stream = pointer(a[9]);
  if (PyErr_Occurred()) return nullptr;
  bool need[5];
  for (int i = 0; i < 5; ++i) need[i] = a[10 + i] == Py_True;
  std::vector<at::Tensor> out;
  {
    Unlocked u;
    const int64_t P = pts.size(1), S = sph.size(0), N = (int64_t)prm->n_bands * prm->n_bands;
    const at::Tensor gB = f32(grad);
    at::Tensor gP, gN, gA, gS, gL;
    if (need[0]) gP = empty({3, P}, pts);
    if (need[1]) gN = empty({3, P}, pts);
    if (need[2]) gA = empty({P}, pts);
    if (need[3]) gS = empty({S, 4}, pts);
    if (need[4]) gL = empty({N}, pts);
    check(api.render_backward(data(gB), data(pts), data(nrm), data(alb), data(sph), P, S, prm, data(vis), data(saved),
                              saved.numel() * 4, data(gP), data(gN), data(gA), data(gS), data(gL), ws.data_ptr(),
                              ws.numel(), (hipStream_t)stream),
          "sh_render_backward");
    out = {gP.defined() ? gP.t() : gP, gN.defined() ? gN.t() : gN, gA, gS, gL};
  }
  return tuple(out);
  END_HANDLE_TH_ERRORS
}

// channels_forward(points, normals, albedo, spheres, light, params, ws, stream)
//   -> radiance [P, C], points, normals, albedo, spheres, light (as the library takes them), vis, saved
PyObject* py_channels_forward(PyObject*, PyObject* const* a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  if (n != 8) throw std::runtime_error("channels_forward: eight arguments");
  const at::Tensor &points = tensor(a[0]), &normals = tensor(a[1]), &albedo = tensor(a[2]), &spheres = tensor(a[3]),
                   &light = tensor(a[4]), &ws = tensor(a[6]);
  const shv_params* prm = (const shv_params*)pointer(a[5]);
  void* stream = pointer(a[7]);
  if (PyErr_Occurred()) return nullptr;
  std::vector<at::Tensor> out;
  {
    Unlocked u;
    const int64_t P = points.size(0), S = spheres.size(0), C = light.size(0),
                  N = (int64_t)prm->n_bands * prm->n_bands;
    auto [pts, nrm] = soa2(points, normals, stream);
    at::Tensor alb = soa(albedo), sph = f32(spheres), L = f32(light);
    at::Tensor vis = empty({N, P}, points), rad = empty({C, P}, points);
    at::Tensor saved = empty({std::max<int64_t>(api.saved_floats(P, prm), 1)}, points);
    check(api.visibility_forward(data(pts), P, data(sph), S, prm, data(vis), data(saved), saved.numel() * 4,
                                 ws.data_ptr(), ws.numel(), (hipStream_t)stream),
          "sh_visibility_forward");
    check(api.shade_channels(data(vis), data(nrm), data(alb), data(L), (int32_t)C, P, prm, data(rad), ws.data_ptr(),
                             ws.numel(), (hipStream_t)stream),
          "sh_shade_channels");
    out = {rad.t(), pts, nrm, alb, sph, L, vis, saved};
  }
  return tuple(out);
  END_HANDLE_TH_ERRORS
}

// channels_backward(grad_radiance, points, normals, albedo, spheres, light, vis, saved, params, ws, stream, need x 5)
//   -> gradients of points, normals, albedo, spheres, light (None where not needed)
PyObject* py_channels_backward(PyObject*, PyObject* const* a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  if (n != 16) throw std::runtime_error("channels_backward: sixteen arguments");
  const at::Tensor &grad = tensor(a[0]), &pts = tensor(a[1]), &nrm = tensor(a[2]), &alb = tensor(a[3]),
                   &sph = tensor(a[4]), &L = tensor(a[5]), &vis = tensor(a[6]), &saved = tensor(a[7]),
                   &ws = tensor(a[9]);
  const shv_params* prm = (const shv_params*)pointer(a[8]);
  void* stream = pointer(a[10]);
  if (PyErr_Occurred()) return nullptr;
  bool need[5];
  for (int i = 0; i < 5; ++i) need[i] = a[11 + i] == Py_True;
  std::vector<at::Tensor> out;
  {
    Unlocked u;
    const int64_t P = pts.size(1), S = sph.size(0), C = L.size(0), N = (int64_t)prm->n_bands * prm->n_bands;
    const bool need_v = need[0] || need[3];
    const at::Tensor gB = soa(grad);
    at::Tensor gV, gN, gA, gL, gP, gS;
    if (need_v) gV = empty({N, P}, pts);
    if (need[1]) gN = empty({3, P}, pts);
    if (need[2]) gA = empty({C, P}, pts);
    if (need[4]) gL = empty({C, N}, pts);
    if (need[0]) gP = empty({3, P}, pts);
    if (need[3]) gS = empty({S, 4}, pts);
    check(api.shade_channels_backward(data(gB), data(vis), data(nrm), data(alb), data(L), (int32_t)C, P, prm, data(gV),
                                      data(gN), data(gA), data(gL), ws.data_ptr(), ws.numel(), (hipStream_t)stream),
          "sh_shade_channels_backward");
    if (need_v)
      check(api.visibility_backward(data(gV), data(vis), data(pts), P, data(sph), S, prm, data(saved),
                                    saved.numel() * 4, data(gP), data(gS), ws.data_ptr(), ws.numel(),
                                    (hipStream_t)stream),
            "sh_visibility_backward");
    out = {gP.defined() ? gP.t() : gP, gN.defined() ? gN.t() : gN, gA.defined() ? gA.t() : gA, gS, gL};
  }
  return tuple(out);
  END_HANDLE_TH_ERRORS
}

#define FAST(f) (PyCFunction)(void (*)(void))(f), METH_FASTCALL
PyMethodDef methods[] = {{"bind", FAST(py_bind), nullptr},
                         {"inputs_ok", FAST(py_inputs_ok), nullptr},
                         {"shade_forward", FAST(py_shade_forward), nullptr},
                         {"shade_backward", FAST(py_shade_backward), nullptr},
                         {"channels_forward", FAST(py_channels_forward), nullptr},
                         {"channels_backward", FAST(py_channels_backward), nullptr},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_host", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__host() { return PyModule_Create(&module); }
