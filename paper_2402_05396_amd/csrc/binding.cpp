// Native half of the Python binding: the calls of a training loop, whose Python cost (checks, allocation of
// the outputs, marshalling of pointers) was a multiple of their time on the GPU for small batches.
//
// Every function here takes the arguments of the Python function of the same name, serves the plain case
// (exact torch tensors of the expected types, ordinary integers) and returns None for anything else, which the
// Python function then handles, or refuses, itself; so also where the library's own allocations find no memory.
// Errors of the C library become TaserError. The library's entry points come in as addresses (bind), so this file
// links against torch only.
//
// One mini-batch of 1800 roots with edge rows: 24.6 us a call when marshalled in Python, 11.5 us so, of which the
// two kernel launches take about 6; its kernels take 9.
#include <Python.h>

#include <ATen/ATen.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "taser.h"

namespace {

struct Api {
    decltype(&taser_sample_temporal) sample_temporal;
    decltype(&taser_sample_temporal_rows) sample_temporal_rows;
    decltype(&taser_gather_features) gather_features;
    decltype(&taser_candidate_encodings) candidate_encodings;
    decltype(&taser_select_weighted) select_weighted;
    decltype(&taser_cache_lookup) cache_lookup;
    decltype(&taser_selector_draw) selector_draw;
    decltype(&taser_selector_update) selector_update;
    decltype(&taser_selector_scores) selector_scores;
    decltype(&taser_last_error) last_error;
} api;
PyObject* error_class = nullptr;                                  // TaserError
PyObject *s_nbr, *s_eid, *s_ts, *s_count, *s_cuda_stream;         // interned names

struct Ref {   // an owned reference
    PyObject* p;
    explicit Ref(PyObject* o = nullptr) : p(o) {}
    ~Ref() { Py_XDECREF(p); }
    Ref(const Ref&) = delete;
    Ref& operator=(const Ref&) = delete;
    PyObject* release() { PyObject* o = p; p = nullptr; return o; }
};

// ---- arguments: false means "not the plain case" ------------------------------------
bool get_int(PyObject* o, int64_t low, int64_t high, int64_t* v) {
    if (!PyLong_CheckExact(o)) return false;
    int overflow = 0;
    *v = PyLong_AsLongLongAndOverflow(o, &overflow);
    return !overflow && *v >= low && *v <= high;
}
bool get_u64(PyObject* o, uint64_t* v) {   // modulo 2^64, as a C integer argument takes it
    if (!PyLong_CheckExact(o)) return false;
    *v = PyLong_AsUnsignedLongLongMask(o);
    return true;
}
bool get_handle(PyObject* o, void** p) {
    if (!PyLong_CheckExact(o)) return false;
    *p = PyLong_AsVoidPtr(o);
    return *p != nullptr;
}
const at::Tensor* plain(PyObject* o) { return THPVariable_CheckExact(o) ? &THPVariable_Unpack(o) : nullptr; }
const at::Tensor* device_array(PyObject* o, at::ScalarType type) {
    const at::Tensor* t = plain(o);
    return t && t->scalar_type() == type && t->is_cuda() && t->layout() == at::kStrided && t->is_contiguous() ? t : nullptr;
}
const at::Tensor* device_table(PyObject* o) {
    const at::Tensor* t = plain(o);
    return t && t->is_cuda() && t->layout() == at::kStrided && t->dim() == 2 && t->stride(1) == 1 ? t : nullptr;
}
bool get_stream(PyObject* o, void** stream) {
    if (o == Py_None) {
        *stream = c10::hip::getCurrentHIPStream().stream();
        return true;
    }
    Ref value(PyObject_GetAttr(o, s_cuda_stream));
    if (!value.p || !PyLong_CheckExact(value.p)) {
        PyErr_Clear();
        return false;
    }
    *stream = PyLong_AsVoidPtr(value.p);
    return true;
}

PyObject* not_plain() { Py_RETURN_NONE; }

PyObject* raise(int rc) {
    Ref e(PyObject_CallFunction(error_class, "is", rc, api.last_error()));
    if (e.p) PyErr_SetObject(error_class, e.p);
    return nullptr;
}

at::Tensor make(at::IntArrayRef size, at::ScalarType type, at::Device device) {
    return at::empty(size, at::TensorOptions().dtype(type).device(device));
}

bool put(PyObject* dict, PyObject* name, const at::Tensor& t) {
    Ref o(THPVariable_Wrap(t));
    return o.p && PyDict_SetItem(dict, name, o.p) == 0;
}

// ---- sample_temporal, sample_temporal_rows ---------------------------------------------
// (handle, roots, times, k, hops, policy, seed, m, edge_weight, stream[, table, row_elems])
PyObject* sample(PyObject*, PyObject* const* a, Py_ssize_t n_args) {
    HANDLE_TH_ERRORS
    if (n_args != 10 && n_args != 12) return not_plain();
    void *handle, *stream;
    int64_t k, hops, policy, m;
    uint64_t seed;
    const at::Tensor *roots = device_array(a[1], at::kInt), *times = device_array(a[2], at::kLong), *weight = nullptr, *table = nullptr;
    if (!get_handle(a[0], &handle) || !roots || !times || !get_int(a[3], 1, TASER_MAX_K, &k) || !get_int(a[4], 1, TASER_MAX_HOPS, &hops) ||
        !get_int(a[5], 0, 3, &policy) || !get_u64(a[6], &seed) || !get_int(a[7], INT32_MIN, INT32_MAX, &m))
        return not_plain();
    if (a[8] != Py_None && !(weight = device_array(a[8], at::kInt))) return not_plain();
    if (!get_stream(a[9], &stream)) return not_plain();
    const int64_t n = roots->numel();
    if (times->numel() != n) return not_plain();
    int64_t slots = n;
    for (int64_t h = 0; h < hops; ++h)
        if ((slots *= k) >= (int64_t)1 << 31) return not_plain();
    int64_t elems = 0, size = 0;
    if (n_args == 12) {
        if (!(table = device_table(a[10]))) return not_plain();
        size = table->element_size();
        elems = table->size(1);
        if (a[11] != Py_None && !get_int(a[11], 1, INT32_MAX, &elems)) return not_plain();
        if (elems * size > INT32_MAX) return not_plain();
    }
    taser_hop_out out[TASER_MAX_HOPS];
    void* rows_out[TASER_MAX_HOPS];
    Ref list(PyList_New(hops)), rows(table ? PyList_New(hops) : nullptr);
    if (!list.p || (table && !rows.p)) return nullptr;
    int64_t r = n;
    for (int64_t h = 0; h < hops; ++h) {
        const at::Device device = roots->device();
        const at::Tensor nbr = make({r, k}, at::kInt, device), eid = make({r, k}, at::kInt, device), ts = make({r, k}, at::kLong, device),
                         count = make({r}, at::kInt, device);
        out[h] = taser_hop_out{static_cast<int32_t*>(nbr.data_ptr()), static_cast<int32_t*>(eid.data_ptr()),
                               static_cast<int64_t*>(ts.data_ptr()), static_cast<int32_t*>(count.data_ptr())};
        PyObject* d = PyDict_New();
        if (!d) return nullptr;
        PyList_SET_ITEM(list.p, h, d);
        if (!put(d, s_nbr, nbr) || !put(d, s_eid, eid) || !put(d, s_ts, ts) || !put(d, s_count, count)) return nullptr;
        r *= k;
        if (table) {
            const at::Tensor t = make({r, elems}, table->scalar_type(), table->device());
            rows_out[h] = t.data_ptr();
            PyObject* o = THPVariable_Wrap(t);
            if (!o) return nullptr;
            PyList_SET_ITEM(rows.p, h, o);
        }
    }
    const int32_t* p_roots = static_cast<const int32_t*>(roots->data_ptr());
    const int64_t* p_times = static_cast<const int64_t*>(times->data_ptr());
    const uint32_t* p_weight = weight ? static_cast<const uint32_t*>(weight->data_ptr()) : nullptr;
    const void* p_table = table ? table->data_ptr() : nullptr;
    int rc;
    Py_BEGIN_ALLOW_THREADS
    if (table)
        rc = api.sample_temporal_rows(static_cast<taser_tcsr*>(handle), p_roots, p_times, n, (int32_t)k, (int32_t)hops, (int32_t)policy, seed,
                                      (int32_t)m, p_weight, p_table, table->size(0), (int32_t)(elems * size), table->stride(0) * size, out,
                                      rows_out, stream);
    else
        rc = api.sample_temporal(static_cast<taser_tcsr*>(handle), p_roots, p_times, n, (int32_t)k, (int32_t)hops, (int32_t)policy, seed,
                                 (int32_t)m, p_weight, out, stream);
    Py_END_ALLOW_THREADS
    if (rc == TASER_E_OOM) return not_plain();
    if (rc != TASER_OK) return raise(rc);
    if (!table) return list.release();
    return PyTuple_Pack(2, list.p, rows.p);
    END_HANDLE_TH_ERRORS
}

// ---- gather_features(table, ids, out, row_elems, stream) --------------------------------
PyObject* gather(PyObject*, PyObject* const* a, Py_ssize_t n_args) {
    HANDLE_TH_ERRORS
    void* stream;
    const at::Tensor *table = n_args == 5 ? device_table(a[0]) : nullptr, *ids = table ? device_array(a[1], at::kInt) : nullptr;
    if (!ids) return not_plain();
    int64_t elems = table->size(1);
    const int64_t size = table->element_size(), n = ids->numel();
    if (a[3] != Py_None && !get_int(a[3], 1, INT32_MAX, &elems)) return not_plain();
    if (elems * size > INT32_MAX || !get_stream(a[4], &stream)) return not_plain();
    at::Tensor made;
    const at::Tensor* out = &made;
    if (a[2] == Py_None) made = make({n, elems}, table->scalar_type(), table->device());
    else if (!(out = device_array(a[2], table->scalar_type())) || out->numel() < n * elems) return not_plain();
    const void *p_table = table->data_ptr(), *p_ids = ids->data_ptr();
    void* p_out = out->data_ptr();
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = api.gather_features(p_table, table->size(0), (int32_t)(elems * size), table->stride(0) * size, static_cast<const int32_t*>(p_ids), n,
                             p_out, stream);
    Py_END_ALLOW_THREADS
    if (rc != TASER_OK) return raise(rc);
    if (a[2] == Py_None) return THPVariable_Wrap(made);
    Py_INCREF(a[2]);
    return a[2];
    END_HANDLE_TH_ERRORS
}

// ---- candidate_encodings(nbr, count, want_identity, stream) -----------------------------
PyObject* encodings(PyObject*, PyObject* const* a, Py_ssize_t n_args) {
    HANDLE_TH_ERRORS
    void* stream;
    const at::Tensor *nbr = n_args == 4 ? device_array(a[0], at::kInt) : nullptr, *count = nbr ? device_array(a[1], at::kInt) : nullptr;
    if (!count || nbr->dim() != 2 || count->numel() != nbr->size(0) || !PyBool_Check(a[2]) || !get_stream(a[3], &stream)) return not_plain();
    const int64_t n = nbr->size(0), m = nbr->size(1);
    if (m < 1 || m > TASER_MAX_M) return not_plain();
    const at::Tensor freq = make({n, m}, at::kInt, nbr->device());
    at::Tensor identity;
    if (a[2] == Py_True) identity = make({n, m, m}, at::kByte, nbr->device());
    const void *p_nbr = nbr->data_ptr(), *p_count = count->data_ptr();
    void *p_freq = freq.data_ptr(), *p_identity = a[2] == Py_True ? identity.data_ptr() : nullptr;
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = api.candidate_encodings(static_cast<const int32_t*>(p_nbr), static_cast<const int32_t*>(p_count), n, (int32_t)m,
                                 static_cast<int32_t*>(p_freq), static_cast<uint8_t*>(p_identity), stream);
    Py_END_ALLOW_THREADS
    if (rc != TASER_OK) return raise(rc);
    Ref f(THPVariable_Wrap(freq)), i(a[2] == Py_True ? THPVariable_Wrap(identity) : nullptr);
    if (!f.p || (a[2] == Py_True && !i.p)) return nullptr;
    return PyTuple_Pack(2, f.p, i.p ? i.p : Py_None);
    END_HANDLE_TH_ERRORS
}

// ---- select_weighted(weight, count, k, seed, hop, candidates, stream) --------------------
PyObject* select(PyObject*, PyObject* const* a, Py_ssize_t n_args) {
    HANDLE_TH_ERRORS
    void* stream;
    int64_t k, hop;
    uint64_t seed;
    const at::Tensor *weight = n_args == 7 ? device_array(a[0], at::kInt) : nullptr, *count = weight ? device_array(a[1], at::kInt) : nullptr;
    if (!count || weight->dim() != 2 || count->numel() != weight->size(0) || !get_int(a[2], 1, TASER_MAX_K, &k) || !get_u64(a[3], &seed) ||
        !get_int(a[4], 0, UINT32_MAX, &hop) || !get_stream(a[6], &stream))
        return not_plain();
    const int64_t n = weight->size(0), m = weight->size(1);
    if (m < 1 || m > TASER_MAX_M || n * (m > k ? m : k) >= (int64_t)1 << 31) return not_plain();
    taser_hop_out from = {}, to = {};
    const bool with = a[5] != Py_None;
    if (with) {
        if (!PyDict_CheckExact(a[5])) return not_plain();
        PyObject *o_nbr = PyDict_GetItem(a[5], s_nbr), *o_eid = PyDict_GetItem(a[5], s_eid), *o_ts = PyDict_GetItem(a[5], s_ts);
        if (!o_nbr || !o_eid || !o_ts) return not_plain();
        const at::Tensor *nbr = device_array(o_nbr, at::kInt), *eid = device_array(o_eid, at::kInt), *ts = device_array(o_ts, at::kLong);
        if (!nbr || !eid || !ts || nbr->numel() != n * m || eid->numel() != n * m || ts->numel() != n * m) return not_plain();
        from = taser_hop_out{static_cast<int32_t*>(nbr->data_ptr()), static_cast<int32_t*>(eid->data_ptr()),
                             static_cast<int64_t*>(ts->data_ptr()), nullptr};
    }
    const at::Device device = weight->device();
    const at::Tensor sel = make({n, k}, at::kInt, device), out_count = make({n}, at::kInt, device);
    Ref kept, o_sel(THPVariable_Wrap(sel)), o_count(THPVariable_Wrap(out_count));
    if (!o_sel.p || !o_count.p) return nullptr;
    if (with) {
        const at::Tensor nbr = make({n, k}, at::kInt, device), eid = make({n, k}, at::kInt, device), ts = make({n, k}, at::kLong, device);
        to = taser_hop_out{static_cast<int32_t*>(nbr.data_ptr()), static_cast<int32_t*>(eid.data_ptr()),
                           static_cast<int64_t*>(ts.data_ptr()), nullptr};
        kept.p = PyDict_New();
        if (!kept.p || !put(kept.p, s_nbr, nbr) || !put(kept.p, s_eid, eid) || !put(kept.p, s_ts, ts) ||
            PyDict_SetItem(kept.p, s_count, o_count.p) != 0)
            return nullptr;
    }
    const void *p_weight = weight->data_ptr(), *p_count = count->data_ptr();
    void *p_sel = sel.data_ptr(), *p_out_count = out_count.data_ptr();
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = api.select_weighted(static_cast<const uint32_t*>(p_weight), static_cast<const int32_t*>(p_count), n, (int32_t)m, (int32_t)k, seed,
                             (uint32_t)hop, static_cast<int32_t*>(p_sel), static_cast<int32_t*>(p_out_count), with ? &from : nullptr,
                             with ? &to : nullptr, stream);
    Py_END_ALLOW_THREADS
    if (rc != TASER_OK) return raise(rc);
    return PyTuple_Pack(3, o_sel.p, o_count.p, kept.p ? kept.p : Py_None);
    END_HANDLE_TH_ERRORS
}

// ---- cache_lookup(handle, host_table, row_elems, ids, out, hit_miss, stream) --------------
PyObject* lookup(PyObject*, PyObject* const* a, Py_ssize_t n_args) {
    HANDLE_TH_ERRORS
    void *handle, *stream;
    int64_t elems;
    const at::Tensor *host = n_args == 7 ? plain(a[1]) : nullptr, *ids = host ? device_array(a[3], at::kInt) : nullptr, *hit_miss = nullptr;
    if (!ids || !get_handle(a[0], &handle) || !get_int(a[2], 1, INT32_MAX, &elems) || !get_stream(a[6], &stream)) return not_plain();
    if (a[5] != Py_None && !(hit_miss = device_array(a[5], at::kLong))) return not_plain();
    const int64_t n = ids->numel();
    at::Tensor made;
    const at::Tensor* out = &made;
    if (a[4] == Py_None) made = make({n, elems}, host->scalar_type(), ids->device());
    else if (!(out = device_array(a[4], host->scalar_type())) || out->numel() < n * elems) return not_plain();
    const void* p_ids = ids->data_ptr();
    void *p_out = out->data_ptr(), *p_hit_miss = hit_miss ? hit_miss->data_ptr() : nullptr;
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = api.cache_lookup(static_cast<taser_cache*>(handle), static_cast<const int32_t*>(p_ids), n, p_out, static_cast<uint64_t*>(p_hit_miss),
                          stream);
    Py_END_ALLOW_THREADS
    if (rc == TASER_E_OOM) return not_plain();
    if (rc != TASER_OK) return raise(rc);
    if (a[4] == Py_None) return THPVariable_Wrap(made);
    Py_INCREF(a[4]);
    return a[4];
    END_HANDLE_TH_ERRORS
}

// ---- selector_draw(handle, b, seed, iteration, out, stream) --------------------------------
PyObject* draw(PyObject*, PyObject* const* a, Py_ssize_t n_args) {
    HANDLE_TH_ERRORS
    void *handle, *stream;
    int64_t b;
    uint64_t seed, iteration;
    if (n_args != 6 || !get_handle(a[0], &handle) || !get_int(a[1], 0, INT32_MAX, &b) || !get_u64(a[2], &seed) || !get_u64(a[3], &iteration) ||
        !get_stream(a[5], &stream))
        return not_plain();
    at::Tensor made;
    const at::Tensor* out = &made;
    if (a[4] == Py_None) made = make({b}, at::kInt, at::Device(at::kCUDA));
    else if (!(out = device_array(a[4], at::kInt)) || out->numel() < b) return not_plain();
    void* p_out = out->data_ptr();
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = api.selector_draw(static_cast<taser_selector*>(handle), b, seed, iteration, static_cast<int32_t*>(p_out), stream);
    Py_END_ALLOW_THREADS
    if (rc != TASER_OK) return raise(rc);
    if (a[4] == Py_None) return THPVariable_Wrap(made);
    Py_INCREF(a[4]);
    return a[4];
    END_HANDLE_TH_ERRORS
}

// ---- selector_update(handle, batch, new_scores, stream) -> True -----------------------------
PyObject* update(PyObject*, PyObject* const* a, Py_ssize_t n_args) {
    HANDLE_TH_ERRORS
    void *handle, *stream;
    const at::Tensor *batch = n_args == 4 ? device_array(a[1], at::kInt) : nullptr, *scores = batch ? device_array(a[2], at::kInt) : nullptr;
    if (!scores || !get_handle(a[0], &handle) || batch->numel() != scores->numel() || !get_stream(a[3], &stream)) return not_plain();
    const void *p_batch = batch->data_ptr(), *p_scores = scores->data_ptr();
    const int64_t b = batch->numel();
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = api.selector_update(static_cast<taser_selector*>(handle), static_cast<const int32_t*>(p_batch), static_cast<const uint32_t*>(p_scores),
                             b, stream);
    Py_END_ALLOW_THREADS
    if (rc != TASER_OK) return raise(rc);
    Py_RETURN_TRUE;
    END_HANDLE_TH_ERRORS
}

// ---- selector_scores(handle, n, stream) -> tensor (without the total) ------------------------
PyObject* scores(PyObject*, PyObject* const* a, Py_ssize_t n_args) {
    HANDLE_TH_ERRORS
    void *handle, *stream;
    int64_t n;
    if (n_args != 3 || !get_handle(a[0], &handle) || !get_int(a[1], 1, INT32_MAX, &n) || !get_stream(a[2], &stream)) return not_plain();
    const at::Tensor out = make({n}, at::kInt, at::Device(at::kCUDA));
    void* p_out = out.data_ptr();
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = api.selector_scores(static_cast<taser_selector*>(handle), static_cast<uint32_t*>(p_out), nullptr, stream);
    Py_END_ALLOW_THREADS
    if (rc != TASER_OK) return raise(rc);
    return THPVariable_Wrap(out);
    END_HANDLE_TH_ERRORS
}

// bind(TaserError, {entry point: address})
template <typename F> bool entry(PyObject* addresses, const char* name, F* to) {
    PyObject* o = PyDict_GetItemString(addresses, name);
    *to = o ? reinterpret_cast<F>(PyLong_AsVoidPtr(o)) : nullptr;
    if (*to) return true;
    if (!PyErr_Occurred()) PyErr_Format(PyExc_ValueError, "bind: no address for %s", name);
    return false;
}
PyObject* bind(PyObject*, PyObject* args) {
    PyObject *cls, *addresses;
    if (!PyArg_ParseTuple(args, "OO!", &cls, &PyDict_Type, &addresses)) return nullptr;
    Api to = {};
    if (!entry(addresses, "taser_sample_temporal", &to.sample_temporal) || !entry(addresses, "taser_sample_temporal_rows", &to.sample_temporal_rows) ||
        !entry(addresses, "taser_gather_features", &to.gather_features) || !entry(addresses, "taser_candidate_encodings", &to.candidate_encodings) ||
        !entry(addresses, "taser_select_weighted", &to.select_weighted) || !entry(addresses, "taser_cache_lookup", &to.cache_lookup) ||
        !entry(addresses, "taser_selector_draw", &to.selector_draw) || !entry(addresses, "taser_selector_update", &to.selector_update) ||
        !entry(addresses, "taser_selector_scores", &to.selector_scores) || !entry(addresses, "taser_last_error", &to.last_error))
        return nullptr;
    api = to;
    Py_INCREF(cls);
    Py_XSETREF(error_class, cls);
    Py_RETURN_NONE;
}

#define FAST(name, function) {name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(function)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {{"bind", bind, METH_VARARGS, nullptr}, FAST("sample", sample), FAST("gather", gather), FAST("encodings", encodings),
                         FAST("select", select), FAST("lookup", lookup), FAST("draw", draw), FAST("update", update), FAST("scores", scores),
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_binding", "Native half of the Python binding, built for " TASER_BINDING_TAG ".", -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__binding() {
    s_nbr = PyUnicode_InternFromString("nbr");
    s_eid = PyUnicode_InternFromString("eid");
    s_ts = PyUnicode_InternFromString("ts");
    s_count = PyUnicode_InternFromString("count");
    s_cuda_stream = PyUnicode_InternFromString("cuda_stream");
    if (!s_nbr || !s_eid || !s_ts || !s_count || !s_cuda_stream) return nullptr;
    return PyModule_Create(&module);
}
