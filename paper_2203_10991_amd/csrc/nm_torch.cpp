// The common forms of the Python binding's hot calls on torch tensors, in C++: checks, output tensors and the call into libnm_mvue without
// the interpreter in between.  api.py asks here first.  Whatever is not the common form -- another type, layout or device, tensor
// subclasses, arguments that are errors -- comes back as None and takes api.py's own way, which also raises the exceptions.  An error
// status of the library comes back as an int.
//
// Why: a call cost the host 7.7 us of which the launch is 2.5 (three tensors made from Python 4, arguments turned by ctypes 1, the rest checks), and in the
// worker thread of a backward pass, with cold caches, half as much again.
#include <Python.h>

#include <ATen/PythonTorchFunctionTLS.h>
#include <ATen/autocast_mode.h>
#include <ATen/core/Tensor.h>
#include <ATen/ops/empty.h>
#include <c10/core/GradMode.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/core/impl/VirtualGuardImpl.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>

#include "../../include/nm_mvue.h"

namespace {

// The library's functions, by the addresses that ctypes resolved (the library is loaded once, by api.py), and the callable that gives a
// device's current stream as an int
decltype(&mvue_prune_1of2) p_prune_1of2;
decltype(&mvue_prune_2of4) p_prune_2of4;
decltype(&nm_update_gemm) p_update_gemm;
decltype(&nm_update_gemm_workspace) p_update_gemm_workspace;
decltype(&nm_linear_update) p_linear_update;
decltype(&nm_linear_update_workspace) p_linear_update_workspace;
decltype(&nm_linear_forward) p_linear_forward;
decltype(&nm_linear_input_grad) p_linear_input_grad;
PyObject *stream_of = nullptr;

struct NoGil {                                                       // as a ctypes call does: a launch may wait for the queue
    PyThreadState *state = PyEval_SaveThread();
    ~NoGil() { PyEval_RestoreThread(state); }
};

// a tensor (or parameter, no other subclass) on the GPU with memory of its own (a batch of gradients under vmap has none), or nullptr
const at::Tensor *gpu_tensor(PyObject *o)
{
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor &t = THPVariable_Unpack(o);
    return t.defined() && t.is_cuda() && t.layout() == at::kStrided && t.has_storage() ? &t : nullptr;
}
// rows of a 2-D tensor with unit column stride: the row stride, or -1
int64_t row_stride(const at::Tensor &t)
{
    if (t.dim() != 2 || (t.size(1) > 1 && t.stride(1) != 1)) return -1;
    return t.size(0) > 1 ? t.stride(0) : std::max(t.size(1), t.stride(0));
}
// ... whose rows the layer calls read as they are
int64_t layer_rows(const at::Tensor &t)
{
    if (t.dim() != 2 || t.scalar_type() != at::kBFloat16 || t.stride(1) != 1 || t.stride(0) < t.size(1) || t.stride(0) % 8 || t.stride(0) > (1 << 21) ||
        (uintptr_t)t.data_ptr() % 16)
        return -1;
    return t.size(0) > 1 ? t.stride(0) : t.size(1);
}
bool stream(const at::Tensor &t, void *&out)
{
    PyObject *device = PyLong_FromLong(t.get_device());
    if (!device) return false;
    PyObject *s = PyObject_CallOneArg(stream_of, device);
    Py_DECREF(device);
    if (!s) return false;
    out = PyLong_AsVoidPtr(s);
    Py_DECREF(s);
    return !PyErr_Occurred();
}
bool whole_number(PyObject *o) { return PyLong_Check(o) && !PyBool_Check(o); }
at::Tensor empty(at::IntArrayRef size, at::ScalarType type, const at::Tensor &like) { return at::empty(size, like.options().dtype(type).requires_grad(false)); }
PyObject *none() { Py_RETURN_NONE; }

// prune(pattern, g, seed, stream_id, mode) -> (vals, meta): MVUE 1:2 (pattern 2) or 2:4 (4) of g, outputs allocated
PyObject *prune(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    if (n != 5) return none();
    const at::Tensor *g = gpu_tensor(a[1]);
    if (!g || !whole_number(a[2]) || !whole_number(a[3]) || !PyLong_Check(a[4])) return none();
    const int64_t ld = row_stride(*g);
    const at::ScalarType type = g->scalar_type();
    if (ld < 0 || (type != at::kFloat && type != at::kBFloat16)) return none();
    const int64_t T = g->size(0), O = g->size(1), G = T / 16;
    const uint64_t seed = PyLong_AsUnsignedLongLongMask(a[2]);
    const uint32_t id = (uint32_t)PyLong_AsUnsignedLongMask(a[3]);
    const long pattern = PyLong_AsLong(a[0]), mode = PyLong_AsLong(a[4]);
    void *st;
    if (PyErr_Occurred() || !stream(*g, st)) return nullptr;
    at::Tensor vals = empty({G, O, 8}, type, *g), meta = empty({G, O}, at::kShort, *g);
    const int dt = type == at::kFloat ? NM_F32 : NM_BF16;
    void *from = g->data_ptr(), *v = vals.data_ptr();
    uint16_t *m = (uint16_t *)meta.data_ptr();
    int rc;
    {
        NoGil free;
        rc = pattern == 2 ? p_prune_1of2(from, T, O, ld, dt, seed, id, v, m, nullptr, 0, st)
                          : p_prune_2of4(from, T, O, ld, dt, seed, id, (int)mode, v, m, nullptr, 0, st);
    }
    if (rc) return PyLong_FromLong(rc);
    return Py_BuildValue("(NN)", THPVariable_Wrap(std::move(vals)), THPVariable_Wrap(std::move(meta)));
    END_HANDLE_TH_ERRORS
}

// update_gemm(vals, meta, h, bf16x3) -> dW, allocated with the workspace
PyObject *update_gemm(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    if (n != 4) return none();
    const at::Tensor *vals = gpu_tensor(a[0]), *meta = gpu_tensor(a[1]), *h = gpu_tensor(a[2]);
    if (!vals || !meta || !h || vals->dim() != 3 || vals->scalar_type() != h->scalar_type()) return none();
    const int64_t ld = row_stride(*h);
    const at::ScalarType type = h->scalar_type();
    if (ld < 0 || (type != at::kFloat && type != at::kBFloat16) || h->size(0) != vals->size(0) * 16) return none();
    const int x3 = PyObject_IsTrue(a[3]);
    const int64_t T = h->size(0), I = h->size(1), O = vals->size(1);
    const int dt = type == at::kBFloat16 ? NM_BF16 : x3 ? NM_F32_BF16X3 : NM_F32;
    void *st;
    if (x3 < 0 || !stream(*h, st)) return nullptr;
    at::Tensor dW = empty({O, I}, at::kFloat, *h), ws;
    const size_t need = p_update_gemm_workspace(T, O, I, dt);
    if (need) ws = empty({(int64_t)need}, at::kByte, *h);
    void *w = need ? ws.data_ptr() : nullptr;
    const void *v = vals->data_ptr(), *b = h->data_ptr();
    const uint16_t *m = (const uint16_t *)meta->data_ptr();
    float *to = (float *)dW.data_ptr();
    int rc;
    {
        NoGil free;
        rc = p_update_gemm(v, m, b, ld, to, std::max<int64_t>(I, 1), T, O, I, dt, 0.f, w, need, st);
    }
    if (rc) return PyLong_FromLong(rc);
    return THPVariable_Wrap(std::move(dW));
    END_HANDLE_TH_ERRORS
}

// linear_update(g, h, pattern, mode, q8, seed, stream_id, act or None, bias) -> (dW, db or None, g_out or None)
PyObject *linear_update(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    if (n != 9) return none();
    const at::Tensor *g = gpu_tensor(a[0]), *h = gpu_tensor(a[1]), *act = a[7] == Py_None ? nullptr : gpu_tensor(a[7]);
    if (!g || !h || (a[7] != Py_None && !act) || !whole_number(a[5]) || !whole_number(a[6]) || !PyLong_Check(a[2]) || !PyLong_Check(a[3])) return none();
    const int64_t ldg = layer_rows(*g), ldh = layer_rows(*h), lda = act ? layer_rows(*act) : 0;
    if (ldg < 0 || ldh < 0 || lda < 0 || h->size(0) != g->size(0) || (act && act->sizes() != g->sizes())) return none();
    const int64_t T = g->size(0), O = g->size(1), I = h->size(1);
    const int q8 = PyObject_IsTrue(a[4]), bias = PyObject_IsTrue(a[8]);
    const int pattern = (int)PyLong_AsLong(a[2]), mode = (int)PyLong_AsLong(a[3]);
    const uint64_t seed = PyLong_AsUnsignedLongLongMask(a[5]);
    const uint32_t id = (uint32_t)PyLong_AsUnsignedLongMask(a[6]);
    void *st;
    if (PyErr_Occurred() || !stream(*g, st)) return nullptr;
    const size_t need = p_linear_update_workspace(T, O, I, q8, bias);
    at::Tensor dW = empty({O, I}, at::kBFloat16, *g), db, g_out, ws = empty({(int64_t)std::max<size_t>(need, 1)}, at::kByte, *g);
    if (bias) db = empty({O}, at::kBFloat16, *g);
    if (act) g_out = empty({T, O}, at::kBFloat16, *g);
    const void *pg = g->data_ptr(), *ph = h->data_ptr(), *pa = act ? act->data_ptr() : nullptr;
    void *pw = ws.data_ptr(), *pd = dW.data_ptr(), *pb = bias ? db.data_ptr() : nullptr, *po = act ? g_out.data_ptr() : nullptr;
    int rc;
    {
        NoGil free;
        rc = p_linear_update(pg, ldg, pa, lda, ph, ldh, T, O, I, pattern, mode, q8, seed, id, po, O, pd, pb, pw, need, st);
    }
    if (rc) return PyLong_FromLong(rc);
    return Py_BuildValue("(NNN)", THPVariable_Wrap(std::move(dW)), bias ? THPVariable_Wrap(std::move(db)) : none(), act ? THPVariable_Wrap(std::move(g_out)) : none());
    END_HANDLE_TH_ERRORS
}

// ---- the dense products of a layer.  Which of them are the library's: plain bf16 tensors on the current device that the kernels read as they are, at
// sizes at which they are the faster way.  Up to DENSE_SURE multiply-adds the host's time counts, 6 us of it a call instead of 20, and the kernels take 0.77 of
// the vendor library's time in the mean (0.4 to 1.1 and one of 1.33: gemm_dense.hip).  From there to DENSE_MOST the kernels count: over 288 products
// 0.80 in the mean, and at most 1.06 but for reductions beyond DENSE_LARGE_DEEP (641 x 3520 -> 2744 29.5 us against 25.2) and for ones of DENSE_LARGE_ROUND or
// more with a few tiles of 128 x 128 more than a round of 256 (264 tiles, 5519 x 2192 -> 712: 53 against 36), which stay the vendor library's.  With a ReLU behind the
// product, up to DENSE_RELU_MOST of them and the reduction width DENSE_RELU_WIDTH: the pass over the output that is saved outweighs what the product
// may lose (a layer of 6143 x 640 -> 1320 157 us -> 126; 9143 x 1088 -> 2000 203.8 -> 202.9; alone 16384 x 2048 -> 2048 is 122 against 95 and 23).  Beyond,
// the power limit takes the gain back: 16384 x 1024 -> 4096 alone 128 us against 106 and 43, inside its layer 445-462 us against 450-456.
// A tile's reduction runs on one workgroup from end to end, 0.25 us for every 64 steps, where the vendor library splits it: 64 x 65536 -> 64 takes 269 us
// against 46, 256 x 16384 -> 256 71 against 17.  So the reduction is at most DENSE_DEEP long, or DENSE_DEEPER where there are DENSE_TILES tiles of 64 x 64
// to wait for.  Over 420 calls inside these lines one takes 0.44 of the framework's time in the mean, two 1.13 and 1.21 of it (694 x 1400 ->
// 3280: a few tiles in a second round), all others at most 1.07.
// Both are rules for calls that the host makes one by one.  Where only the kernels' time counts, in a captured graph or behind a deep queue, the forward
// kernel takes 0.9 of the vendor library's in the mean and up to 1.8 times it on few tiles, the input gradient's 0.84 and up to 1.65, and with the ReLU
// 0.65 and up to 1.35 of product and pass.  A captured step takes the same way all the same: it has to find there what the step before it, run once to
// warm up, has used, and the vendor library's first product of a process or thread cannot be captured.
// The framework's stay: autocast regions, and operators that a mode of functions or of dispatch watches.
constexpr int64_t DENSE_SURE = 5000000000, DENSE_MOST = 12000000000, DENSE_LARGE_DEEP = 3072, DENSE_LARGE_ROUND = 1024, DENSE_RELU_MOST = 20000000000, DENSE_RELU_WIDTH = 1536,
                  DENSE_DEEP = 2048, DENSE_DEEPER = 3584, DENSE_TILES = 128;

bool dense_takes(const at::Tensor &a, const at::Tensor &w, const at::Tensor *bias, bool relu, int64_t width, int64_t &rows, int64_t &ld)
{
    if (w.dim() != 2 || a.dim() < 2 || a.scalar_type() != at::kBFloat16 || w.scalar_type() != at::kBFloat16 || a.size(-1) != width) return false;
    const int64_t O = w.size(0), I = w.size(1);
    rows = width ? a.numel() / width : 0;                              // (width: the reduction axis)
    if (rows < 1 || O < 1 || I < 1 || O % 8 || I % 8 || O > (1 << 21) || I > (1 << 21) || rows > ((int64_t)1 << 34) / O || rows > ((int64_t)1 << 36) / I) return false;
    if (width > DENSE_DEEP && (width > DENSE_DEEPER || (rows + 63) / 64 * ((O * I / width + 63) / 64) < DENSE_TILES)) return false;
    const bool relu_pass = relu && I <= DENSE_RELU_WIDTH;              // (a ReLU whose pass over the output outweighs the product's time)
    if (rows * O > (relu_pass ? DENSE_RELU_MOST : DENSE_MOST) / I) return false;
    if (!relu_pass && rows * O > DENSE_SURE / I) {
        const int64_t tiles = (rows + 127) / 128 * ((O * I / width + 127) / 128);
        if (width > DENSE_LARGE_DEEP || (width >= DENSE_LARGE_ROUND && tiles > 256 && tiles <= 384)) return false;
    }
    if (a.dim() == 2) ld = rows > 1 ? a.stride(0) : width;
    else if (a.is_contiguous()) ld = width;
    else return false;
    if (a.stride(-1) != 1 || ld < width || ld % 8 || ld > (1 << 21) || !w.is_contiguous() || (uintptr_t)a.data_ptr() % 16 || (uintptr_t)w.data_ptr() % 16) return false;
    if (a.device() != w.device() || c10::impl::VirtualGuardImpl(c10::DeviceType::CUDA).getDevice() != a.device()) return false;
    if (bias && (bias->dim() != 1 || bias->size(0) != O || bias->scalar_type() != at::kBFloat16 || !bias->is_contiguous() || (uintptr_t)bias->data_ptr() % 16 ||
                 bias->device() != a.device()))
        return false;
    return !at::autocast::is_autocast_enabled(at::kCUDA) && !c10::impl::TorchDispatchModeTLS::any_modes_set() && !at::impl::torch_function_mode_enabled();
}
at::Tensor rows_like(const at::Tensor &a, int64_t width)
{
    at::DimVector size(a.sizes().begin(), a.sizes().end());
    size.back() = width;
    return empty(size, at::kBFloat16, a);
}

// linear_forward(x, weight, bias or None, relu) -> y
PyObject *linear_forward(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    if (n != 4) return none();
    const at::Tensor *x = gpu_tensor(a[0]), *w = gpu_tensor(a[1]), *b = a[2] == Py_None ? nullptr : gpu_tensor(a[2]);
    const int relu = PyObject_IsTrue(a[3]);
    int64_t T, ld;
    if (relu < 0 || !x || !w || (a[2] != Py_None && !b) || w->dim() != 2 || !dense_takes(*x, *w, b, relu, w->size(1), T, ld)) return relu < 0 ? nullptr : none();
    void *st;
    if (!stream(*x, st)) return nullptr;
    at::Tensor y = rows_like(*x, w->size(0));
    const void *px = x->data_ptr(), *pw = w->data_ptr(), *pb = b ? b->data_ptr() : nullptr;
    void *py = y.data_ptr();
    const int64_t O = w->size(0), I = w->size(1);
    int rc;
    {
        NoGil free;
        rc = p_linear_forward(px, ld, pw, pb, T, O, I, relu, py, st);
    }
    if (rc) return PyLong_FromLong(rc);
    return THPVariable_Wrap(std::move(y));
    END_HANDLE_TH_ERRORS
}

// linear_input_grad(g, weight) -> dx; not where gradients are recorded
PyObject *linear_input_grad(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    if (n != 2 || c10::GradMode::is_enabled()) return none();
    const at::Tensor *g = gpu_tensor(a[0]), *w = gpu_tensor(a[1]);
    int64_t T, ld;
    if (!g || !w || w->dim() != 2 || !dense_takes(*g, *w, nullptr, false, w->size(0), T, ld)) return none();
    void *st;
    if (!stream(*g, st)) return nullptr;
    at::Tensor dx = rows_like(*g, w->size(1));
    const void *pg = g->data_ptr(), *pw = w->data_ptr();
    void *pd = dx.data_ptr();
    const int64_t O = w->size(0), I = w->size(1);
    int rc;
    {
        NoGil free;
        rc = p_linear_input_grad(pg, ld, pw, T, O, I, pd, st);
    }
    if (rc) return PyLong_FromLong(rc);
    return THPVariable_Wrap(std::move(dx));
    END_HANDLE_TH_ERRORS
}

// bind({name: address}, stream_of)
PyObject *bind(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    if (n != 2 || !PyDict_Check(a[0])) { PyErr_SetString(PyExc_TypeError, "bind(functions, stream_of)"); return nullptr; }
    struct { const char *name; void **at; } all[] = {
        {"mvue_prune_1of2", (void **)&p_prune_1of2}, {"mvue_prune_2of4", (void **)&p_prune_2of4}, {"nm_update_gemm", (void **)&p_update_gemm},
        {"nm_update_gemm_workspace", (void **)&p_update_gemm_workspace}, {"nm_linear_update", (void **)&p_linear_update},
        {"nm_linear_update_workspace", (void **)&p_linear_update_workspace}, {"nm_linear_forward", (void **)&p_linear_forward},
        {"nm_linear_input_grad", (void **)&p_linear_input_grad}};
    for (auto &f : all) {
        PyObject *address = PyDict_GetItemString(a[0], f.name);
        if (!address) { PyErr_Format(PyExc_KeyError, "%s", f.name); return nullptr; }
        *f.at = PyLong_AsVoidPtr(address);
        if (PyErr_Occurred()) return nullptr;
    }
    Py_INCREF(a[1]);
    Py_XDECREF(stream_of);
    stream_of = a[1];
    Py_RETURN_NONE;
}

#define NM_METHOD(name) {#name, (PyCFunction)(void (*)())name, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {NM_METHOD(bind), NM_METHOD(prune), NM_METHOD(update_gemm), NM_METHOD(linear_update), NM_METHOD(linear_forward), NM_METHOD(linear_input_grad),
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module_def = {PyModuleDef_HEAD_INIT, "_nm_torch", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

extern "C" __attribute__((visibility("default"))) PyObject *PyInit__nm_torch() { return PyModule_Create(&module_def); }
