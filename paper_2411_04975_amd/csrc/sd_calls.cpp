// The calls of a decode step from Python: argument marshalling in native code.
//
// A step's calls take eight to thirteen tensors each.  binding.py checks every one of them (dtype, device,
// contiguity, size) and passes its address on; done in Python that is 0.7 us a tensor, 11 us a call, while the
// kernels of a small batch take 3 to 15 us: a loop that is driven from the host waited for itself.  Here the same
// checks take some 20 ns a tensor and a call 3 us with its launch.  What is not plainly right (a wrong type, a
// tensor too small, a subclass of the expected classes) is left to binding.py, which says what is
// wrong with it: the functions return None then, and have done nothing.
//
// Nothing is remembered between calls.
#include <Python.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/sd.h"

namespace {

PyObject *trees_class = nullptr;
enum { N_NODES, TOKENS, PARENTS, MATCH_LEN, SOURCE, SCORES, TREE_SCORE, USE_DRAFT, BATCH, MAX_NODES, N_NAMES };
const char *const names[N_NAMES] = {"n_nodes", "tokens", "parents", "match_len", "source", "scores", "tree_score", "use_draft", "batch", "max_nodes"};
PyObject *interned[N_NAMES];

// tensors that are more than they look like: their address is not for us to take
const c10::DispatchKeySet wrapped({c10::DispatchKey::Python, c10::DispatchKey::Functionalize, c10::DispatchKey::FuncTorchBatched,
                                   c10::DispatchKey::FuncTorchGradWrapper, c10::DispatchKey::Batched, c10::DispatchKey::ZeroTensor,
                                   c10::DispatchKey::Conjugate, c10::DispatchKey::Negative});

// The address of a tensor of at least n elements of type st on GPU dev.  None is taken where n is 0.
bool address(PyObject *o, at::ScalarType st, int dev, int64_t n, const void **out) {
    *out = nullptr;
    if (o == Py_None) return n <= 0;
    if (!THPVariable_CheckExact(o)) return false;
    const at::Tensor &t = THPVariable_Unpack(o);
    if (!t.defined() || !t.has_storage() || t.key_set().has_any(wrapped)) return false;
    if (t.scalar_type() != st || !t.is_cuda() || t.get_device() != dev || !t.is_contiguous() || t.numel() < n) return false;
    *out = t.data_ptr();
    return true;
}
template <typename T>
bool address(PyObject *o, at::ScalarType st, int dev, int64_t n, T **out) {
    const void *p;
    if (!address(o, st, dev, n, &p)) return false;
    *out = static_cast<T *>(const_cast<void *>(p));
    return true;
}

bool whole(PyObject *o, int64_t *out) {
    if (!PyLong_CheckExact(o)) return false;
    int over;
    *out = PyLong_AsLongLongAndOverflow(o, &over);
    return !over;
}

// the arguments in front: handle, device, stream
struct Target {
    sd_ctx *ctx;
    int dev;
    void *stream;
};
bool target(PyObject *const *a, Target *t) {
    if (!PyLong_CheckExact(a[0]) || !PyLong_CheckExact(a[1]) || !PyLong_CheckExact(a[2])) return false;
    t->ctx = static_cast<sd_ctx *>(PyLong_AsVoidPtr(a[0]));
    t->dev = (int)PyLong_AsLong(a[1]);
    t->stream = PyLong_AsVoidPtr(a[2]);
    return t->ctx && !PyErr_Occurred();
}

// A Trees object's buffers for `batch` requests (batch < 0: as many as it holds), references kept until the
// call is made.
struct Trees {
    PyObject *held[N_NAMES] = {};
    int64_t holds = 0, mn = 0;
    sd_trees s{};
    ~Trees() {
        for (PyObject *o : held) Py_XDECREF(o);
    }
    bool open(PyObject *o) {
        if ((PyObject *)Py_TYPE(o) != trees_class) return false;
        for (int i = 0; i < N_NAMES; i++)
            if (!(held[i] = PyObject_GetAttr(o, interned[i]))) return false;
        return whole(held[BATCH], &holds) && whole(held[MAX_NODES], &mn) && mn >= 0 && mn <= INT32_MAX;
    }
    bool take(int dev, int64_t batch) {
        const auto i32 = at::kInt, f64 = at::kDouble;
        s.max_nodes = (int32_t)mn;
        return batch >= 0 && batch <= INT32_MAX && address(held[N_NODES], i32, dev, batch, &s.d_n_nodes) &&
               address(held[TOKENS], i32, dev, batch * mn, &s.d_tokens) &&
               address(held[PARENTS], i32, dev, batch * mn, &s.d_parents) &&
               address(held[MATCH_LEN], i32, dev, batch, &s.d_match_len) &&
               address(held[SOURCE], i32, dev, batch, &s.d_source) &&
               address(held[SCORES], f64, dev, batch * mn, &s.d_scores) &&
               address(held[TREE_SCORE], f64, dev, batch, &s.d_tree_score) &&
               address(held[USE_DRAFT], i32, dev, batch, &s.d_use_draft);
    }
};

// slot ids, and the batch they stand for: None is the identity over all the trees
bool slots(PyObject *o, int dev, const Trees &t, int64_t *batch, const int32_t **out) {
    *out = nullptr;
    *batch = t.holds;
    if (o == Py_None) return true;
    if (!THPVariable_CheckExact(o)) return false;
    *batch = THPVariable_Unpack(o).numel();
    return *batch <= t.holds && address(o, at::kInt, dev, *batch, out);
}

struct Said {  // the target's tokens, and where acceptance goes
    const int32_t *target;
    int32_t *len, *path, *bonus;
    bool take(PyObject *const *a, int dev, int64_t batch, int64_t mn) {
        return address(a[0], at::kInt, dev, batch * (mn + 1), &target) && address(a[1], at::kInt, dev, batch, &len) &&
               address(a[2], at::kInt, dev, batch * mn, &path) && address(a[3], at::kInt, dev, batch, &bonus);
    }
};

PyObject *left() {  // to binding.py
    PyErr_Clear();
    Py_RETURN_NONE;
}
template <typename F>
PyObject *call(F f) {
    sd_status rc;
    Py_BEGIN_ALLOW_THREADS
    rc = f();
    Py_END_ALLOW_THREADS
    return PyLong_FromLong((long)rc);
}

// (handle, device, stream, slot_ids, trees)
PyObject *speculate(PyObject *, PyObject *const *a, Py_ssize_t n) {
    Target g;
    Trees t;
    int64_t batch;
    const int32_t *ids;
    if (n != 5 || !target(a, &g) || !t.open(a[4]) || !slots(a[3], g.dev, t, &batch, &ids) || !t.take(g.dev, batch)) return left();
    return call([&] { return sd_speculate(g.ctx, ids, (int32_t)batch, t.s, g.stream); });
}

// (handle, device, stream, trees, batch, target_tokens, accept_len, accept_path, bonus)
PyObject *accept(PyObject *, PyObject *const *a, Py_ssize_t n) {
    Target g;
    Trees t;
    Said s;
    int64_t batch;
    if (n != 9 || !target(a, &g) || !t.open(a[3]) || !whole(a[4], &batch) || !t.take(g.dev, batch) || !s.take(a + 5, g.dev, batch, t.mn)) return left();
    return call([&] { return sd_accept(g.ctx, t.s, (int32_t)batch, s.target, s.len, s.path, s.bonus, g.stream); });
}

// (handle, device, stream, trees, slot_ids, target_tokens, accept_len, accept_path, bonus)
template <sd_status (*F)(sd_ctx *, sd_trees, const int32_t *, int32_t, const int32_t *, int32_t *, int32_t *, int32_t *, void *)>
PyObject *accept_append(PyObject *, PyObject *const *a, Py_ssize_t n) {
    Target g;
    Trees t;
    Said s;
    int64_t batch;
    const int32_t *ids;
    if (n != 9 || !target(a, &g) || !t.open(a[3]) || !slots(a[4], g.dev, t, &batch, &ids) || !t.take(g.dev, batch) || !s.take(a + 5, g.dev, batch, t.mn)) return left();
    return call([&] { return F(g.ctx, t.s, ids, (int32_t)batch, s.target, s.len, s.path, s.bonus, g.stream); });
}

// (handle, device, stream, slot_ids, new_tokens, new_offsets)
PyObject *append(PyObject *, PyObject *const *a, Py_ssize_t n) {
    Target g;
    const int32_t *ids = nullptr, *tokens, *offsets;
    if (n != 6 || !target(a, &g) || !THPVariable_CheckExact(a[5]) || (a[3] != Py_None && !THPVariable_CheckExact(a[3]))) return left();
    const int64_t count = a[3] == Py_None ? THPVariable_Unpack(a[5]).numel() - 1 : THPVariable_Unpack(a[3]).numel();
    if (count < 0 || count > INT32_MAX || !address(a[3], at::kInt, g.dev, 0, &ids) || !address(a[4], at::kInt, g.dev, count == 0 ? 0 : 1, &tokens) ||
        !address(a[5], at::kInt, g.dev, count + 1, &offsets))
        return left();
    return call([&] { return sd_index_append(g.ctx, ids, tokens, offsets, (int32_t)count, g.stream); });
}

PyObject *set_trees(PyObject *, PyObject *cls) {
    Py_INCREF(cls);
    Py_XDECREF(trees_class);
    trees_class = cls;
    Py_RETURN_NONE;
}

#define FAST(f) (PyCFunction)(void (*)(void))(f)
PyMethodDef methods[] = {
    {"set_trees", set_trees, METH_O, "the class whose objects stand for sd_trees"},
    {"speculate", FAST(speculate), METH_FASTCALL, "sd_speculate"},
    {"accept", FAST(accept), METH_FASTCALL, "sd_accept"},
    {"accept_append", FAST(accept_append<sd_accept_append>), METH_FASTCALL, "sd_accept_append"},
    {"accept_append_speculate", FAST(accept_append<sd_accept_append_speculate>), METH_FASTCALL, "sd_accept_append_speculate"},
    {"append", FAST(append), METH_FASTCALL, "sd_index_append"},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_sdcalls", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__sdcalls() {
    for (int i = 0; i < N_NAMES; i++)
        if (!(interned[i] = PyUnicode_InternFromString(names[i]))) return nullptr;
    return PyModule_Create(&module);
}
