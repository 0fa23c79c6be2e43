// The calls of binding.py in native code: what a call does on the host beside its launch (checks, output tensors, the
// arguments of the C entry) took 3-4 us of Python, half of a small call.  Every function serves the plain case only (plain
// device tensors, whole-number arguments, no outputs or streams handed in) and returns None for anything else, which binding.py
// then serves, errors and all; an error code of the library comes back as an int.
#include <Python.h>
#include <ATen/ATen.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Dtype.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>
#include <vector>
#include "../../include/division.h"

namespace {

// entries of libdivision.so, which binding.py has loaded
decltype(&division_packed_bytes_3d) packed_bytes;
decltype(&division_compress_3d) compress;
decltype(&division_decompress_3d) decompress;
decltype(&division_compress_maps) compress_maps;
decltype(&division_decompress_maps) decompress_maps;
decltype(&division_relu_compress) relu_compress;
decltype(&division_relu_forward) relu_forward;
decltype(&division_dropout_forward) dropout_forward;
decltype(&division_mask_backward) mask_backward;
decltype(&division_maxpool_forward) maxpool_forward;
decltype(&division_maxpool_backward) maxpool_backward;
decltype(&division_mask_bytes) mask_bytes;

// A mode of torch that replaces or watches calls sees those of binding.py
bool plain_state() { return !c10::impl::TorchDispatchModeTLS::any_modes_set() && !at::impl::torch_function_mode_enabled(); }

// A plain device tensor with memory of its own (no subclass, no wrapper of a transform)
const at::Tensor* device_tensor(PyObject* o) {
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor& t = THPVariable_Unpack(o);
    return t.is_cuda() && t.layout() == at::kStrided && t.has_storage() ? &t : nullptr;
}
bool whole(PyObject* o, int64_t* v) {
    if (!PyLong_CheckExact(o)) return false;
    int over = 0;
    *v = PyLong_AsLongLongAndOverflow(o, &over);
    return over == 0;
}
bool whole32(PyObject* o, int* v) {
    int64_t w;
    if (!whole(o, &w) || w < INT32_MIN || w > INT32_MAX) return false;
    *v = (int)w;
    return true;
}
bool seed64(PyObject* o, uint64_t* v) {
    if (!PyLong_CheckExact(o)) return false;
    *v = PyLong_AsUnsignedLongLongMask(o);                 // seed mod 2^64, negative ones too
    return true;
}
// -1: a type that binding.py refuses
int type_of(at::ScalarType t, bool c16) {
    if (t == at::kFloat) return c16 ? DIVISION_F32_C16 : DIVISION_F32;
    return t == at::kBFloat16 && !c16 ? DIVISION_BF16 : -1;
}
struct Dims { int64_t n, c, d, h, w; };
bool dims_of(const at::Tensor& x, Dims* s) {
    const auto v = x.sizes();
    if (v.size() == 4) *s = {v[0], v[1], 1, v[2], v[3]};
    else if (v.size() == 5) *s = {v[0], v[1], v[2], v[3], v[4]};
    else return false;
    return x.numel() > 0;
}
// a shape of positive whole numbers: a tuple, torch.Size or list of 4 or 5
bool dims_of(PyObject* shape, Dims* s, std::vector<int64_t>* sizes) {
    if (!PyTuple_Check(shape) && !PyList_CheckExact(shape)) return false;
    const Py_ssize_t n = PySequence_Fast_GET_SIZE(shape);
    if (n != 4 && n != 5) return false;
    sizes->resize((size_t)n);
    for (Py_ssize_t i = 0; i < n; ++i)
        if (!whole(PySequence_Fast_GET_ITEM(shape, i), &(*sizes)[(size_t)i]) || (*sizes)[(size_t)i] <= 0) return false;
    const auto& v = *sizes;
    if (n == 4) *s = {v[0], v[1], 1, v[2], v[3]};
    else *s = {v[0], v[1], v[2], v[3], v[4]};
    return true;
}
at::Tensor make(at::IntArrayRef sizes, at::ScalarType t, c10::Device device) { return at::empty(sizes, at::TensorOptions().dtype(t).device(device)); }
size_t bytes(const at::Tensor& t) { return (size_t)(t.numel() * t.element_size()); }
void* current_stream() { return c10::hip::getCurrentHIPStream().stream(); }      // of the current device, as torch.cuda.current_stream()

PyObject* none() { Py_RETURN_NONE; }
PyObject* wrap(at::Tensor t) { return THPVariable_Wrap(std::move(t)); }
PyObject* tuple_of(std::initializer_list<at::Tensor> ts) {
    PyObject* r = PyTuple_New((Py_ssize_t)ts.size());
    if (!r) return nullptr;
    Py_ssize_t i = 0;
    for (const at::Tensor& t : ts) {
        PyObject* o = wrap(t);
        if (!o) { Py_DECREF(r); return nullptr; }
        PyTuple_SET_ITEM(r, i++, o);
    }
    return r;
}
// The output tensors and the library call without the interpreter's lock, as torch.empty and a call through ctypes take them: an
// allocation may wait for the device, other threads do not wait with it.  f touches no Python object.
template <typename F> int without_lock(F&& f) {
    struct Unlocked {
        PyThreadState* state = PyEval_SaveThread();
        ~Unlocked() { PyEval_RestoreThread(state); }        // behind exceptions too
    } unlocked;
    return f();
}

#define PLAIN(n) if (nargs != (n) || !plain_state()) return none()

// compress(x, B, b, seed, c16, dims): dims = the number of dimensions the caller's entry takes
PyObject* py_compress(PyObject*, PyObject* const* a, Py_ssize_t nargs) {
    HANDLE_TH_ERRORS
    PLAIN(6);
    const at::Tensor* x = device_tensor(a[0]);
    int B, b, nd;
    uint64_t seed;
    Dims s;
    if (!x || !whole32(a[1], &B) || !whole32(a[2], &b) || !seed64(a[3], &seed) || !PyBool_Check(a[4]) || !whole32(a[5], &nd)) return none();
    const int dt = type_of(x->scalar_type(), a[4] == Py_True);
    if (dt < 0 || x->dim() != nd || !dims_of(*x, &s) || !x->is_contiguous()) return none();
    const size_t need = packed_bytes(s.n, s.c, s.d, s.h, s.w, B, b, (division_dtype)dt);
    if (need == 0) return none();
    const void* xp = x->data_ptr();
    const c10::Device dev = x->device();
    void* st = current_stream();
    at::Tensor packed;
    const int rc = without_lock([&] {
        packed = make({(int64_t)need}, at::kByte, dev);
        return compress(xp, s.n, s.c, s.d, s.h, s.w, (division_dtype)dt, B, b, seed, packed.data_ptr(), need, st);
    });
    return rc ? PyLong_FromLong(rc) : wrap(std::move(packed));
    END_HANDLE_TH_ERRORS
}

// decompress(packed, shape, B, b, dtype, c16, dims)
PyObject* py_decompress(PyObject*, PyObject* const* a, Py_ssize_t nargs) {
    HANDLE_TH_ERRORS
    PLAIN(7);
    const at::Tensor* packed = device_tensor(a[0]);
    int B, b, nd;
    Dims s;
    std::vector<int64_t> sizes;
    if (!packed || !dims_of(a[1], &s, &sizes) || !whole32(a[2], &B) || !whole32(a[3], &b) || !THPDtype_Check(a[4]) || !PyBool_Check(a[5]) ||
        !whole32(a[6], &nd) || sizes.size() != (size_t)nd)
        return none();
    const at::ScalarType t = reinterpret_cast<THPDtype*>(a[4])->scalar_type;
    const int dt = type_of(t, a[5] == Py_True);
    // (sizes the library refuses: before a tensor of them is asked for)
    if (dt < 0 || packed_bytes(s.n, s.c, s.d, s.h, s.w, B, b, (division_dtype)dt) == 0) return none();
    const void* pk = packed->data_ptr();
    const size_t have = bytes(*packed);
    const c10::Device dev = packed->device();
    void* st = current_stream();
    at::Tensor out;
    const int rc = without_lock([&] {
        out = make(sizes, t, dev);
        return decompress(pk, have, s.n, s.c, s.d, s.h, s.w, (division_dtype)dt, B, b, out.data_ptr(), st);
    });
    return rc ? PyLong_FromLong(rc) : wrap(std::move(out));
    END_HANDLE_TH_ERRORS
}

// one value for every map, or a list or tuple of one per map
PyObject* per_map(PyObject* v, Py_ssize_t i, Py_ssize_t n) {
    if (!PyList_CheckExact(v) && !PyTuple_CheckExact(v)) return v;
    return PySequence_Fast_GET_SIZE(v) == n ? PySequence_Fast_GET_ITEM(v, i) : nullptr;
}
bool is_sequence(PyObject* v) { return PyList_CheckExact(v) || PyTuple_CheckExact(v); }
PyObject* list_of(std::vector<at::Tensor>& ts) {
    PyObject* r = PyList_New((Py_ssize_t)ts.size());
    if (!r) return nullptr;
    for (size_t i = 0; i < ts.size(); ++i) {
        PyObject* o = wrap(std::move(ts[i]));
        if (!o) { Py_DECREF(r); return nullptr; }
        PyList_SET_ITEM(r, (Py_ssize_t)i, o);
    }
    return r;
}

// compress_maps(xs, B, b, seeds, c16)
PyObject* py_compress_maps(PyObject*, PyObject* const* a, Py_ssize_t nargs) {
    HANDLE_TH_ERRORS
    PLAIN(5);
    if (!is_sequence(a[0]) || !is_sequence(a[3]) || !PyBool_Check(a[4])) return none();
    const Py_ssize_t n = PySequence_Fast_GET_SIZE(a[0]);
    if (n == 0 || PySequence_Fast_GET_SIZE(a[3]) != n) return none();
    std::vector<division_map> maps((size_t)n);
    std::vector<at::Tensor> made((size_t)n), held((size_t)n);      // held: the maps, whose list another thread may change meanwhile
    for (Py_ssize_t i = 0; i < n; ++i) {
        division_map& m = maps[(size_t)i];
        const at::Tensor* x = device_tensor(PySequence_Fast_GET_ITEM(a[0], i));
        PyObject *pB = per_map(a[1], i, n), *pb = per_map(a[2], i, n);
        Dims s;
        if (!x || !pB || !pb || !whole32(pB, &m.B) || !whole32(pb, &m.b) || !seed64(PySequence_Fast_GET_ITEM(a[3], i), &m.seed)) return none();
        const int dt = type_of(x->scalar_type(), a[4] == Py_True && x->scalar_type() == at::kFloat);
        if (dt < 0 || !dims_of(*x, &s) || !x->is_contiguous()) return none();
        m.dt = (division_dtype)dt;
        m.N = s.n; m.C = s.c; m.D = s.d; m.H = s.h; m.W = s.w;
        m.packed_bytes = packed_bytes(s.n, s.c, s.d, s.h, s.w, m.B, m.b, m.dt);
        if (m.packed_bytes == 0) return none();
        m.x = x->data_ptr();
        m.xhat = nullptr;
        held[(size_t)i] = *x;
    }
    void* st = current_stream();
    const int rc = without_lock([&] {
        for (size_t i = 0; i < maps.size(); ++i) {
            made[i] = make({(int64_t)maps[i].packed_bytes}, at::kByte, held[i].device());
            maps[i].packed = made[i].data_ptr();
        }
        return compress_maps((int)n, maps.data(), st);
    });
    return rc ? PyLong_FromLong(rc) : list_of(made);
    END_HANDLE_TH_ERRORS
}

// decompress_maps(packed, shapes, B, b, dtypes, c16)
PyObject* py_decompress_maps(PyObject*, PyObject* const* a, Py_ssize_t nargs) {
    HANDLE_TH_ERRORS
    PLAIN(6);
    if (!is_sequence(a[0]) || !is_sequence(a[1]) || !PyBool_Check(a[5])) return none();
    const Py_ssize_t n = PySequence_Fast_GET_SIZE(a[0]);
    if (n == 0 || PySequence_Fast_GET_SIZE(a[1]) != n) return none();
    std::vector<division_map> maps((size_t)n);
    std::vector<at::Tensor> made((size_t)n), held((size_t)n);
    std::vector<std::vector<int64_t>> sizes((size_t)n);
    std::vector<at::ScalarType> types((size_t)n);
    for (Py_ssize_t i = 0; i < n; ++i) {
        division_map& m = maps[(size_t)i];
        const at::Tensor* packed = device_tensor(PySequence_Fast_GET_ITEM(a[0], i));
        PyObject *pB = per_map(a[2], i, n), *pb = per_map(a[3], i, n), *pt = per_map(a[4], i, n);
        Dims s;
        if (!packed || !pB || !pb || !pt || !whole32(pB, &m.B) || !whole32(pb, &m.b) || !THPDtype_Check(pt) ||
            !dims_of(PySequence_Fast_GET_ITEM(a[1], i), &s, &sizes[(size_t)i]))
            return none();
        types[(size_t)i] = reinterpret_cast<THPDtype*>(pt)->scalar_type;
        const int dt = type_of(types[(size_t)i], a[5] == Py_True && types[(size_t)i] == at::kFloat);
        if (dt < 0) return none();
        m.dt = (division_dtype)dt;
        m.N = s.n; m.C = s.c; m.D = s.d; m.H = s.h; m.W = s.w;
        if (packed_bytes(s.n, s.c, s.d, s.h, s.w, m.B, m.b, m.dt) == 0) return none();
        m.packed = packed->data_ptr();
        m.packed_bytes = bytes(*packed);
        m.x = nullptr;
        m.seed = 0;
        held[(size_t)i] = *packed;
    }
    void* st = current_stream();
    const int rc = without_lock([&] {
        for (size_t i = 0; i < maps.size(); ++i) {
            made[i] = make(sizes[i], types[i], held[i].device());
            maps[i].xhat = made[i].data_ptr();
        }
        return decompress_maps((int)n, maps.data(), st);
    });
    return rc ? PyLong_FromLong(rc) : list_of(made);
    END_HANDLE_TH_ERRORS
}

// ---- the operators that cache a 1-bit mask

// a contiguous device tensor of an element type the operators take (0, 1), else -1
int flat_type(const at::Tensor* x) { return x && x->numel() > 0 && x->is_contiguous() ? type_of(x->scalar_type(), false) : -1; }
at::Tensor new_mask(int64_t n, const at::Tensor& x) { return make({(int64_t)(mask_bytes(n) / 4)}, at::kInt, x.device()); }
// y like x and a mask of x's elements
struct Masked { at::Tensor y, mask; };
Masked new_masked(const at::Tensor& x) { return {at::empty_like(x), new_mask(x.numel(), x)}; }

// relu_forward(x)
PyObject* py_relu_forward(PyObject*, PyObject* const* a, Py_ssize_t nargs) {
    HANDLE_TH_ERRORS
    PLAIN(1);
    const at::Tensor* x = device_tensor(a[0]);
    const int dt = flat_type(x);
    if (dt < 0) return none();
    const int64_t n = x->numel();
    const void* xp = x->data_ptr();
    void* st = current_stream();
    Masked o;
    const int rc = without_lock([&] {
        o = new_masked(*x);
        return relu_forward(xp, n, (division_dtype)dt, o.y.data_ptr(), o.mask.data_ptr(), bytes(o.mask), st);
    });
    return rc ? PyLong_FromLong(rc) : tuple_of({o.y, o.mask});
    END_HANDLE_TH_ERRORS
}

// relu_compress(x, B, b, seed, c16)
PyObject* py_relu_compress(PyObject*, PyObject* const* a, Py_ssize_t nargs) {
    HANDLE_TH_ERRORS
    PLAIN(5);
    const at::Tensor* x = device_tensor(a[0]);
    int B, b;
    uint64_t seed;
    if (flat_type(x) < 0 || x->dim() != 4 || !whole32(a[1], &B) || !whole32(a[2], &b) || !seed64(a[3], &seed) || !PyBool_Check(a[4])) return none();
    const int dt = type_of(x->scalar_type(), a[4] == Py_True);
    Dims s;
    if (dt < 0 || !dims_of(*x, &s)) return none();
    const size_t need = packed_bytes(s.n, s.c, 1, s.h, s.w, B, b, (division_dtype)dt);
    if (need == 0) return none();
    const void* xp = x->data_ptr();
    void* st = current_stream();
    Masked o;
    at::Tensor packed;
    const int rc = without_lock([&] {
        o = new_masked(*x);
        packed = make({(int64_t)need}, at::kByte, x->device());
        return relu_compress(xp, s.n, s.c, s.h, s.w, (division_dtype)dt, B, b, seed, o.y.data_ptr(), o.mask.data_ptr(), bytes(o.mask), packed.data_ptr(), need, st);
    });
    return rc ? PyLong_FromLong(rc) : tuple_of({o.y, o.mask, packed});
    END_HANDLE_TH_ERRORS
}

// dropout_forward(x, p, seed)
PyObject* py_dropout_forward(PyObject*, PyObject* const* a, Py_ssize_t nargs) {
    HANDLE_TH_ERRORS
    PLAIN(3);
    const at::Tensor* x = device_tensor(a[0]);
    const int dt = flat_type(x);
    uint64_t seed;
    if (dt < 0 || !PyFloat_CheckExact(a[1]) || !seed64(a[2], &seed)) return none();
    const float p = (float)PyFloat_AS_DOUBLE(a[1]);
    const int64_t n = x->numel();
    const void* xp = x->data_ptr();
    void* st = current_stream();
    Masked o;
    const int rc = without_lock([&] {
        o = new_masked(*x);
        return dropout_forward(xp, n, (division_dtype)dt, p, seed, o.y.data_ptr(), o.mask.data_ptr(), bytes(o.mask), st);
    });
    return rc ? PyLong_FromLong(rc) : tuple_of({o.y, o.mask});
    END_HANDLE_TH_ERRORS
}

// mask_backward(mask, grad_out)
PyObject* py_mask_backward(PyObject*, PyObject* const* a, Py_ssize_t nargs) {
    HANDLE_TH_ERRORS
    PLAIN(2);
    const at::Tensor *mask = device_tensor(a[0]), *g = device_tensor(a[1]);
    const int dt = flat_type(g);
    if (!mask || dt < 0) return none();
    const int64_t n = g->numel();
    const void *mp = mask->data_ptr(), *gp = g->data_ptr();
    const size_t mb = bytes(*mask);
    void* st = current_stream();
    at::Tensor out;
    const int rc = without_lock([&] {
        out = at::empty_like(*g);
        return mask_backward(mp, mb, gp, n, (division_dtype)dt, out.data_ptr(), st);
    });
    return rc ? PyLong_FromLong(rc) : wrap(std::move(out));
    END_HANDLE_TH_ERRORS
}

// maxpool_forward(x, k)
PyObject* py_maxpool_forward(PyObject*, PyObject* const* a, Py_ssize_t nargs) {
    HANDLE_TH_ERRORS
    PLAIN(2);
    const at::Tensor* x = device_tensor(a[0]);
    const int dt = flat_type(x);
    int k;
    Dims s;
    if (dt < 0 || x->dim() != 4 || !whole32(a[1], &k) || k < 1 || !dims_of(*x, &s)) return none();
    const void* xp = x->data_ptr();
    void* st = current_stream();
    at::Tensor y, mask;
    const int rc = without_lock([&] {
        y = make({s.n, s.c, s.h / k, s.w / k}, x->scalar_type(), x->device());
        mask = new_mask(x->numel(), *x);
        return maxpool_forward(xp, s.n, s.c, s.h, s.w, (division_dtype)dt, k, y.data_ptr(), mask.data_ptr(), bytes(mask), st);
    });
    return rc ? PyLong_FromLong(rc) : tuple_of({y, mask});
    END_HANDLE_TH_ERRORS
}

// maxpool_backward(mask, grad_out, shape, k)
PyObject* py_maxpool_backward(PyObject*, PyObject* const* a, Py_ssize_t nargs) {
    HANDLE_TH_ERRORS
    PLAIN(4);
    const at::Tensor *mask = device_tensor(a[0]), *g = device_tensor(a[1]);
    const int dt = flat_type(g);
    int k;
    Dims s;
    std::vector<int64_t> sizes;
    if (!mask || dt < 0 || !whole32(a[3], &k) || k < 1 || !dims_of(a[2], &s, &sizes) || sizes.size() != 4 || g->dim() != 4) return none();
    const auto gs = g->sizes();
    if (gs[0] != s.n || gs[1] != s.c || gs[2] != s.h / k || gs[3] != s.w / k) return none();
    const void *mp = mask->data_ptr(), *gp = g->data_ptr();
    const size_t mb = bytes(*mask);
    void* st = current_stream();
    at::Tensor out;
    const int rc = without_lock([&] {
        out = make(sizes, g->scalar_type(), g->device());
        return maxpool_backward(mp, mb, gp, s.n, s.c, s.h, s.w, (division_dtype)dt, k, out.data_ptr(), st);
    });
    return rc ? PyLong_FromLong(rc) : wrap(std::move(out));
    END_HANDLE_TH_ERRORS
}

// bind(addresses, version, map_bytes): the entries above in the order of the table, of a library of this ABI version whose descriptors
// are so large.  A ValueError where this module was built for another library.
PyObject* py_bind(PyObject*, PyObject* const* a, Py_ssize_t nargs) {
    void** at[] = {(void**)&packed_bytes, (void**)&compress, (void**)&decompress, (void**)&compress_maps, (void**)&decompress_maps,
                   (void**)&relu_compress, (void**)&relu_forward, (void**)&dropout_forward, (void**)&mask_backward,
                   (void**)&maxpool_forward, (void**)&maxpool_backward, (void**)&mask_bytes};
    constexpr Py_ssize_t n = sizeof at / sizeof at[0];
    int version = 0, map_bytes = 0;
    if (nargs != 3 || !PyList_CheckExact(a[0]) || PyList_GET_SIZE(a[0]) != n || !whole32(a[1], &version) || !whole32(a[2], &map_bytes) ||
        version != DIVISION_ABI_VERSION || map_bytes != (int)sizeof(division_map)) {
        PyErr_Format(PyExc_ValueError, "built for ABI version %d with %d entries and descriptors of %d bytes", DIVISION_ABI_VERSION, (int)n, (int)sizeof(division_map));
        return nullptr;
    }
    void* found[n];
    for (Py_ssize_t i = 0; i < n; ++i) {
        found[i] = PyLong_AsVoidPtr(PyList_GET_ITEM(a[0], i));
        if (!found[i]) { if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "a null entry"); return nullptr; }
    }
    for (Py_ssize_t i = 0; i < n; ++i) *at[i] = found[i];
    Py_RETURN_NONE;
}

#define FAST(name) {#name, (PyCFunction)(void*)py_##name, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {FAST(compress), FAST(decompress), FAST(compress_maps), FAST(decompress_maps), FAST(relu_forward), FAST(relu_compress),
                         FAST(dropout_forward), FAST(mask_backward), FAST(maxpool_forward), FAST(maxpool_backward),
                         FAST(bind), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_fastcall", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__fastcall() { return PyModule_Create(&module); }
