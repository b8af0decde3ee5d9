// The binding's calls with their ordinary arguments, without the interpreter: checks, dims struct, output tensors, stream
// and the C-ABI call in one native function each.  A Python wrapper spends 6-12 us per call on attribute lookups, asserts
// and ctypes conversions (MI355X host; a kernel launch is 3 us), which is what a small call consists of.
//
// Every function here either makes the call and returns its result, or returns NotImplemented and has done nothing that
// counts: the wrapper in binding.py then goes on in Python, which raises the right error or handles the unusual form.
// NotImplemented is the answer to anything that is not plain: tensor subclasses, active torch modes, a forced path, timing
// events, a failed check, a status that the library's checks answer with (nothing has been enqueued then), any C++ exception.
// ADASPEC_ERR_HIP may come after a launch: it is raised here, and the call is not made a second time.
//
// The entry points of libadaspec.so arrive as addresses from binding.py, which owns the library's handle; the default
// workspaces are binding.py's as well (one owner for both ways into the library), held here by reference.
#include <ATen/ATen.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <torch/csrc/Dtype.h>
#include <torch/csrc/autograd/python_variable.h>

#include <array>
#include <optional>
#include <vector>

#include "../../include/adaspec.h"

namespace {

struct Bail {};                                        // not a plain call: leave it to Python
struct Raised {};                                      // a Python exception is set: the caller's
// After a Python call that failed: an ordinary error is left to the Python path, which runs into it as well; a
// KeyboardInterrupt or the like is not an answer of what was called, and goes up from here.
[[noreturn]] void failed_in_python()
{
    if (PyErr_Occurred() && !PyErr_ExceptionMatches(PyExc_Exception)) throw Raised{};
    PyErr_Clear();
    throw Bail{};
}

// (a build for the tests of this file: tensors without memory stand in for device memory, stubs for the library)
#ifdef ADASPEC_FASTCALL_ON_META
constexpr at::DeviceType kDevice = at::kMeta;
int meta_index = 0;                                    // they have no device index of their own
int device_index(const at::Tensor &) { return meta_index; }
#else
constexpr at::DeviceType kDevice = at::kCUDA;
int device_index(const at::Tensor &t) { return t.get_device(); }
#endif

struct Api {
    decltype(&adaspec_verify_attn_workspace_bytes) attn_ws;
    decltype(&adaspec_verify_attn) attn;
    decltype(&adaspec_verify_attn_tree) attn_tree;
    decltype(&adaspec_accept_workspace_bytes) accept_ws;
    decltype(&adaspec_accept) accept;
    decltype(&adaspec_accept_tree) accept_tree;
    decltype(&adaspec_kv_append) kv_append;
    decltype(&adaspec_kv_compact_path) kv_compact;
    decltype(&adaspec_commit) commit;
    decltype(&adaspec_draft_sample_workspace_bytes) draft_ws;
    decltype(&adaspec_draft_sample) draft;
} api;
PyObject *get_workspace, *raw_stream, *current_device;   // binding._workspace, torch._C._cuda_getCurrentRawStream / _getDevice
PyObject *error_class;                                   // binding.AdaspecError
bool ready = false;

// the default workspaces in use: [family][device], the tensors of binding._ws_cache
enum Family { kAttn, kAccept, kDraft, kFamilies };
const char *const kFamilyName[kFamilies] = {"attn", "accept", "draft"};
// (never destroyed: at process exit the allocator may be gone before a static's destructor runs)
auto &workspaces = *new std::array<std::vector<at::Tensor>, kFamilies>;

void no_modes()
{
    if (!ready || at::impl::torch_function_mode_enabled() || c10::impl::TorchDispatchModeTLS::stack_len() > 0 ||
        c10::impl::TorchDispatchModeTLS::any_modes_set())
        throw Bail{};
}

const at::Tensor &tensor(PyObject *o)
{
    if (!THPVariable_CheckExact(o)) throw Bail{};
    const at::Tensor &t = THPVariable_Unpack(o);
    if (!t.defined() || t.device().type() != kDevice || t.layout() != at::kStrided) throw Bail{};
    return t;
}
const at::Tensor &dense(PyObject *o, at::ScalarType dt)
{
    const at::Tensor &t = tensor(o);
    if (!t.is_contiguous() || t.scalar_type() != dt) throw Bail{};
    return t;
}
void need(bool ok)
{
    if (!ok) throw Bail{};
}
template <class P = void>
P *ptr(const at::Tensor &t)
{
    return static_cast<P *>(t.data_ptr());
}
template <class P = void>
P *ptr_or_null(PyObject *o)
{
    return o == Py_None ? nullptr : ptr<P>(tensor(o));
}
int32_t dtype_code(at::ScalarType t)
{
    if (t == at::kFloat) return ADASPEC_F32;
    if (t == at::kHalf) return ADASPEC_F16;
    if (t == at::kBFloat16) return ADASPEC_BF16;
    throw Bail{};
}
at::ScalarType scalar_type(int64_t code)
{
    switch (code) {
    case ADASPEC_F32: return at::kFloat;
    case ADASPEC_F16: return at::kHalf;
    case ADASPEC_BF16: return at::kBFloat16;
    default: throw Bail{};
    }
}
int32_t small_int(PyObject *o)
{
    if (!PyLong_CheckExact(o)) throw Bail{};
    int overflow = 0;
    const long long v = PyLong_AsLongLongAndOverflow(o, &overflow);
    if (overflow || v < INT32_MIN || v > INT32_MAX) throw Bail{};
    return (int32_t)v;
}
int32_t size32(int64_t n)
{
    if (n > INT32_MAX) throw Bail{};
    return (int32_t)n;
}
bool is_word(PyObject *o, const char *w) { return PyUnicode_CheckExact(o) && PyUnicode_CompareWithASCIIString(o, w) == 0; }

void *stream_of(PyObject *stream)
{
    PyObject *v;
    if (stream == Py_None) {
        PyObject *dev = PyObject_CallNoArgs(current_device);
        if (!dev) failed_in_python();
        v = PyObject_CallOneArg(raw_stream, dev);
        Py_DECREF(dev);
    } else {
        v = PyObject_GetAttrString(stream, "cuda_stream");
    }
    if (!v) failed_in_python();
    if (!PyLong_Check(v)) { Py_DECREF(v); throw Bail{}; }
    void *p = PyLong_AsVoidPtr(v);
    Py_DECREF(v);
    if (PyErr_Occurred()) failed_in_python();
    return p;
}

// the caller's workspace, or the default one of this device and call family
at::Tensor workspace(PyObject *given, size_t nbytes, Family family, const at::Tensor &like)
{
    if (given != Py_None) return tensor(given);
    auto &all = workspaces[family];
    const size_t dev = (size_t)device_index(like);
    if (dev < all.size() && all[dev].defined() && (size_t)all[dev].numel() >= nbytes) return all[dev];
    // (the interpreter lock may change hands in this call, and another thread's device lengthen the table: nothing in it
    // is referred to across the call)
    PyObject *device = PyObject_GetAttrString(py::cast(like).ptr(), "device");
    PyObject *t = device ? PyObject_CallFunction(get_workspace, "nOOs", (Py_ssize_t)nbytes, device, Py_None, kFamilyName[family]) : nullptr;
    Py_XDECREF(device);
    if (!t) failed_in_python();
    if (!THPVariable_CheckExact(t)) { Py_DECREF(t); throw Bail{}; }
    const at::Tensor ws = THPVariable_Unpack(t);
    Py_DECREF(t);
    if (all.size() <= dev) all.resize(dev + 1);
    all[dev] = ws;
    return ws;
}

at::Tensor empty(at::IntArrayRef shape, at::ScalarType dt, const at::Tensor &like)
{
    return at::empty(shape, at::TensorOptions().dtype(dt).device(like.device()));
}
// an output argument: the caller's object (checked by nobody but the library, as in Python) or a new tensor, whose Python
// object exists before the call is made: after it nothing may fail that could send the call to Python again
struct Output {
    at::Tensor t;
    PyObject *object;
    Output(PyObject *given, at::IntArrayRef shape, at::ScalarType dt, const at::Tensor &like)
    {
        t = given != Py_None ? tensor(given) : empty(shape, dt, like);
        object = given != Py_None ? Py_NewRef(given) : THPVariable_Wrap(t);
        if (!object) failed_in_python();
    }
    ~Output() { Py_DECREF(object); }
    Output(const Output &) = delete;
    PyObject *result() const { return Py_NewRef(object); }
};

struct Unlocked {                                      // the interpreter lock is given up for the life of this object
    PyThreadState *state = PyEval_SaveThread();
    ~Unlocked() { PyEval_RestoreThread(state); }
};
// The C call runs without the interpreter lock, as it does through ctypes.  Its arguments are values: whatever looks at
// Python objects has been done, and may have thrown, before the lock is given up.
template <class F, class... A>
void call(const char *name, F entry, A... args)
{
    const int rc = [&] {
        const Unlocked unlocked;
        return entry(args...);
    }();
    if (rc == ADASPEC_ERR_HIP) {
        if (PyObject *e = PyObject_CallFunction(error_class, "is", rc, name)) {
            PyErr_SetObject(error_class, e);
            Py_DECREF(e);
        }
        throw Raised{};
    }
    if (rc != ADASPEC_OK) throw Bail{};
}

template <class F>
PyObject *guarded(Py_ssize_t nargs, Py_ssize_t want, F &&f)
{
    if (nargs == want) {
        try {
            no_modes();
            return f();                                // (null: the result's tuple could not be made)
        } catch (const Raised &) {
            return nullptr;
        } catch (...) {
            if (PyErr_Occurred()) PyErr_Clear();
        }
    }
    Py_RETURN_NOTIMPLEMENTED;
}

// (q, k_pages, v_pages, block_table, ctx_lens, spec_lens, out, max_spec_len, scale, out_dtype, plan, workspace, stream, parents)
PyObject *verify_attn(PyObject *, PyObject *const *a, Py_ssize_t nargs)
{
    return guarded(nargs, 14, [&]() -> PyObject * {
        const at::Tensor &q = tensor(a[0]), &k = tensor(a[1]), &v = tensor(a[2]);
        const at::Tensor &bt = dense(a[3], at::kInt), &ctx = dense(a[4], at::kInt), &spec = dense(a[5], at::kInt);
        need(q.dim() == 3 && k.dim() == 4 && bt.dim() == 2 && q.is_contiguous() && k.is_contiguous() && v.is_contiguous());
        need(v.sizes() == k.sizes() && q.scalar_type() == k.scalar_type() && v.scalar_type() == k.scalar_type());
        adaspec_attn_dims d = {};
        d.batch = size32(bt.size(0));
        d.total_q = size32(q.size(0));
        d.max_spec_len = small_int(a[7]);
        d.n_q_heads = size32(q.size(1));
        d.n_kv_heads = size32(k.size(1));
        d.head_dim = size32(q.size(2));
        d.page_size = size32(k.size(2));
        d.num_pages = size32(k.size(0));
        d.max_pages_per_req = size32(bt.size(1));
        d.dtype = dtype_code(q.scalar_type());
        d.out_dtype = a[9] == Py_None ? d.dtype : small_int(a[9]);
        need(PyFloat_CheckExact(a[8]));
        d.scale = (float)PyFloat_AS_DOUBLE(a[8]);
        const bool build = is_word(a[10], "build"), reuse = is_word(a[10], "reuse");
        need(build || reuse || is_word(a[10], "run"));
        need(!(build || reuse) || a[11] != Py_None);
        d.plan_mode = build ? ADASPEC_PLAN_BUILD_ONLY : reuse ? ADASPEC_PLAN_REUSE : ADASPEC_PLAN_BUILD_AND_RUN;
        const size_t nbytes = api.attn_ws(&d);
        need(nbytes > 0);
        const at::Tensor ws = workspace(a[11], nbytes, kAttn, q);
        void *s = stream_of(a[12]);
        const int32_t *parents = nullptr;
        if (a[13] != Py_None) {
            const at::Tensor &p = dense(a[13], at::kInt);
            need(p.dim() == 1 && p.size(0) == q.size(0));
            parents = ptr<int32_t>(p);
        }
        const auto run = [&](void *out) {
            if (a[13] != Py_None)
                call("adaspec_verify_attn_tree", api.attn_tree, ptr(q), ptr(k), ptr(v), ptr<int32_t>(bt), ptr<int32_t>(ctx), ptr<int32_t>(spec), parents, out, &d,
                     ptr(ws), (size_t)ws.numel(), s);
            else
                call("adaspec_verify_attn", api.attn, ptr(q), ptr(k), ptr(v), ptr<int32_t>(bt), ptr<int32_t>(ctx), ptr<int32_t>(spec), out, &d, ptr(ws),
                     (size_t)ws.numel(), s);
        };
        if (build && a[6] == Py_None) {
            run(nullptr);
            Py_RETURN_NONE;
        }
        const Output out(a[6], q.sizes(), scalar_type(d.out_dtype), q);
        run(ptr(out.t));
        return out.result();
    });
}

struct Rows {                                          // what accept and accept_tree share
    adaspec_accept_dims d = {};
    const void *probs = nullptr;
    const int32_t *tokens = nullptr;
    Rows(const at::Tensor &logits, PyObject *draft_probs, PyObject *draft_tokens, const at::Tensor &spec, PyObject *max_spec_len,
         PyObject *out_stride)
    {
        need(logits.dim() == 2 && logits.stride(1) == 1 && spec.scalar_type() == at::kInt && spec.dim() == 1);
        const int64_t V = logits.size(1);
        d.batch = size32(spec.size(0));
        d.total_q = size32(logits.size(0));
        d.total_draft = d.total_q - d.batch;
        d.max_spec_len = small_int(max_spec_len);
        d.vocab = size32(V);
        d.logits_dtype = d.probs_dtype = dtype_code(logits.scalar_type());
        need(d.max_spec_len < INT32_MAX);
        d.out_stride = out_stride == Py_None ? d.max_spec_len + 1 : small_int(out_stride);
        need(d.out_stride >= 0);
        d.logits_row_stride = logits.stride(0);
        d.probs_row_stride = V;
        if (d.total_draft > 0) {
            const at::Tensor &p = tensor(draft_probs), &x = tensor(draft_tokens);
            need(p.dim() == 2 && p.size(0) == d.total_draft && p.size(1) == V && p.stride(1) == 1);
            need(x.scalar_type() == at::kInt && x.dim() == 1 && x.size(0) == d.total_draft);
            d.probs_dtype = dtype_code(p.scalar_type());
            d.probs_row_stride = p.stride(0);
            probs = ptr(p);
            tokens = ptr<int32_t>(x);
        }
    }
};

// (target_logits, draft_probs, draft_tokens, uniforms, spec_lens, temperature, max_spec_len, out_tokens, out_accept_len,
//  out_stride, workspace, stream)
PyObject *accept(PyObject *, PyObject *const *a, Py_ssize_t nargs)
{
    return guarded(nargs, 12, [&]() -> PyObject * {
        const at::Tensor &logits = tensor(a[0]), &uni = dense(a[3], at::kFloat), &spec = tensor(a[4]), &temp = tensor(a[5]);
        need(temp.scalar_type() == at::kFloat);
        const Rows r(logits, a[1], a[2], spec, a[6], a[9]);
        const Output toks(a[7], {r.d.batch, r.d.out_stride}, at::kInt, logits), lens(a[8], {r.d.batch}, at::kInt, logits);
        const at::Tensor ws = workspace(a[10], std::max<size_t>(api.accept_ws(&r.d), 256), kAccept, logits);
        void *s = stream_of(a[11]);
        call("adaspec_accept", api.accept, ptr(logits), r.probs, r.tokens, ptr<float>(uni), ptr<int32_t>(spec), ptr<float>(temp), ptr<int32_t>(toks.t),
             ptr<int32_t>(lens.t), &r.d, ptr(ws), (size_t)ws.numel(), s);
        return Py_BuildValue("(NN)", toks.result(), lens.result());
    });
}

// (target_logits, draft_probs, draft_tokens, parents, uniforms, spec_lens, temperature, max_spec_len, out_tokens,
//  out_accept_len, out_path, out_stride, workspace, stream)
PyObject *accept_tree(PyObject *, PyObject *const *a, Py_ssize_t nargs)
{
    return guarded(nargs, 14, [&]() -> PyObject * {
        const at::Tensor &logits = tensor(a[0]), &parents = dense(a[3], at::kInt), &uni = dense(a[4], at::kFloat);
        const at::Tensor &spec = tensor(a[5]), &temp = dense(a[6], at::kFloat);
        need(parents.dim() == 1 && parents.size(0) == logits.size(0));
        const Rows r(logits, a[1], a[2], spec, a[7], a[11]);
        const Output toks(a[8], {r.d.batch, r.d.out_stride}, at::kInt, logits), lens(a[9], {r.d.batch}, at::kInt, logits);
        const Output path(a[10], {r.d.batch, r.d.out_stride}, at::kInt, logits);
        const at::Tensor ws = workspace(a[12], std::max<size_t>(api.accept_ws(&r.d), 256), kAccept, logits);
        void *s = stream_of(a[13]);
        call("adaspec_accept_tree", api.accept_tree, ptr(logits), r.probs, r.tokens, ptr<int32_t>(parents), ptr<float>(uni), ptr<int32_t>(spec),
             ptr<float>(temp), ptr<int32_t>(toks.t), ptr<int32_t>(lens.t), ptr<int32_t>(path.t), &r.d, ptr(ws), (size_t)ws.numel(), s);
        return Py_BuildValue("(NNN)", toks.result(), lens.result(), path.result());
    });
}

// dims of kv_append and kv_compact_path
adaspec_attn_dims cache_dims(const at::Tensor &k, const at::Tensor &bt, int32_t total_q, PyObject *max_spec_len)
{
    adaspec_attn_dims d = {};
    d.batch = size32(bt.size(0));
    d.total_q = total_q;
    d.max_spec_len = small_int(max_spec_len);
    d.n_q_heads = d.n_kv_heads = size32(k.size(1));
    d.head_dim = size32(k.size(3));
    d.page_size = size32(k.size(2));
    d.num_pages = size32(k.size(0));
    d.max_pages_per_req = size32(bt.size(1));
    d.dtype = d.out_dtype = dtype_code(k.scalar_type());
    return d;
}

// (k_new, v_new, k_pages, v_pages, block_table, ctx_lens, spec_lens, max_spec_len, stream)
PyObject *kv_append(PyObject *, PyObject *const *a, Py_ssize_t nargs)
{
    return guarded(nargs, 9, [&]() -> PyObject * {
        const at::Tensor &kn = tensor(a[0]), &vn = tensor(a[1]), &k = tensor(a[2]), &v = tensor(a[3]);
        const at::Tensor &bt = dense(a[4], at::kInt), &ctx = dense(a[5], at::kInt), &spec = dense(a[6], at::kInt);
        need(kn.dim() == 3 && k.dim() == 4 && bt.dim() == 2 && vn.sizes() == kn.sizes() && v.sizes() == k.sizes());
        need(k.size(1) == kn.size(1) && k.size(3) == kn.size(2));
        for (const at::Tensor *t : {&kn, &vn, &k, &v}) need(t->is_contiguous() && t->scalar_type() == kn.scalar_type());
        const adaspec_attn_dims d = cache_dims(k, bt, size32(kn.size(0)), a[7]);
        void *s = stream_of(a[8]);
        call("adaspec_kv_append", api.kv_append, ptr(kn), ptr(vn), ptr(k), ptr(v), ptr<int32_t>(bt), ptr<int32_t>(ctx), ptr<int32_t>(spec), &d, s);
        Py_RETURN_NONE;
    });
}

// (k_pages, v_pages, block_table, ctx_lens, spec_lens, out_path, out_accept_len, max_spec_len, stream)
PyObject *kv_compact_path(PyObject *, PyObject *const *a, Py_ssize_t nargs)
{
    return guarded(nargs, 9, [&]() -> PyObject * {
        const at::Tensor &k = tensor(a[0]), &v = tensor(a[1]);
        const at::Tensor &bt = dense(a[2], at::kInt), &ctx = dense(a[3], at::kInt), &spec = dense(a[4], at::kInt);
        const at::Tensor &path = dense(a[5], at::kInt), &lens = dense(a[6], at::kInt);
        need(k.dim() == 4 && bt.dim() == 2 && path.dim() == 2 && v.sizes() == k.sizes());
        need(k.is_contiguous() && v.is_contiguous() && v.scalar_type() == k.scalar_type());
        const adaspec_attn_dims d = cache_dims(k, bt, size32(bt.size(0)), a[7]);
        void *s = stream_of(a[8]);
        call("adaspec_kv_compact_path", api.kv_compact, ptr(k), ptr(v), ptr<int32_t>(bt), ptr<int32_t>(ctx), ptr<int32_t>(spec), ptr<int32_t>(path),
             ptr<int32_t>(lens), &d, size32(path.size(1)), s);
        Py_RETURN_NONE;
    });
}

// (out_tokens, out_accept_len, spec_lens, ctx_lens, max_spec_len, next_spec_lens, committed_lens, next_ctx_lens, last_token,
//  seq_tokens, seq_lens, stream)
PyObject *commit(PyObject *, PyObject *const *a, Py_ssize_t nargs)
{
    return guarded(nargs, 12, [&]() -> PyObject * {
        const at::Tensor &toks = dense(a[0], at::kInt), &lens = dense(a[1], at::kInt);
        const at::Tensor &spec = dense(a[2], at::kInt), &ctx = dense(a[3], at::kInt);
        need(toks.dim() == 2);
        adaspec_commit_dims d = {};
        d.batch = size32(toks.size(0));
        d.max_spec_len = small_int(a[4]);
        d.out_stride = size32(toks.size(1));
        const Output kept(a[6], {d.batch}, at::kInt, toks), last(a[8], {d.batch}, at::kInt, toks);
        std::optional<Output> next;
        if (a[5] != Py_None || a[7] != Py_None) next.emplace(a[7], at::IntArrayRef{d.batch}, at::kInt, toks);
        if (a[9] != Py_None) {
            const at::Tensor &seq = dense(a[9], at::kInt);
            need(seq.dim() == 2 && a[10] != Py_None && tensor(a[10]).scalar_type() == at::kInt);
            d.seq_stride = size32(seq.size(1));
        }
        void *s = stream_of(a[11]);
        call("adaspec_commit", api.commit, ptr<int32_t>(toks), ptr<int32_t>(lens), ptr<int32_t>(spec), ptr<int32_t>(ctx), ptr_or_null<int32_t>(a[5]),
             ptr<int32_t>(kept.t), next ? ptr<int32_t>(next->t) : nullptr, ptr<int32_t>(last.t), ptr_or_null<int32_t>(a[9]),
             ptr_or_null<int32_t>(a[10]), &d, s);
        return Py_BuildValue("(NNN)", kept.result(), next ? next->result() : Py_NewRef(Py_None), last.result());
    });
}

// (draft_logits, temperature, uniforms, probs_dtype, draft_probs, out_rows, draft_tokens, confidence, workspace, stream)
PyObject *draft_sample(PyObject *, PyObject *const *a, Py_ssize_t nargs)
{
    return guarded(nargs, 10, [&]() -> PyObject * {
        const at::Tensor &logits = tensor(a[0]), &temp = tensor(a[1]), &uni = tensor(a[2]);
        need(logits.dim() == 2 && logits.stride(1) == 1 && temp.scalar_type() == at::kFloat && uni.scalar_type() == at::kFloat);
        const int64_t R = logits.size(0), V = logits.size(1);
        at::ScalarType pt = logits.scalar_type();
        if (a[3] != Py_None) {
            need(THPDtype_Check(a[3]));
            pt = reinterpret_cast<THPDtype *>(a[3])->scalar_type;
        }
        need(a[4] != Py_None || a[5] == Py_None);
        const Output probs(a[4], {R, V}, pt, logits);
        need(probs.t.dim() == 2 && probs.t.stride(1) == 1 && probs.t.size(1) == V);
        const Output toks(a[6], {R}, at::kInt, logits), conf(a[7], {R}, at::kFloat, logits);
        adaspec_draft_dims d = {};
        d.rows = size32(R);
        d.vocab = size32(V);
        d.logits_dtype = dtype_code(logits.scalar_type());
        d.probs_dtype = dtype_code(probs.t.scalar_type());
        d.logits_row_stride = logits.stride(0);
        d.probs_row_stride = probs.t.stride(0);
        const size_t nbytes = api.draft_ws(&d);
        at::Tensor ws;
        if (nbytes) ws = workspace(a[8], nbytes, kDraft, logits);
        void *s = stream_of(a[9]);
        call("adaspec_draft_sample", api.draft, ptr(logits), ptr<float>(temp), ptr<float>(uni), ptr_or_null<int32_t>(a[5]), ptr(probs.t), ptr<int32_t>(toks.t),
             ptr<float>(conf.t), &d, nbytes ? ptr(ws) : nullptr, nbytes ? (size_t)ws.numel() : (size_t)0, s);
        return Py_BuildValue("(NNN)", probs.result(), toks.result(), conf.result());
    });
}

// (tuple of the entry points' addresses in Api's order, binding._workspace, raw stream getter, current device getter,
//  binding.AdaspecError)
PyObject *setup(PyObject *, PyObject *args)
{
    PyObject *table, *ws, *stream, *device, *error;
    if (!PyArg_ParseTuple(args, "O!OOOO", &PyTuple_Type, &table, &ws, &stream, &device, &error)) return nullptr;
    void **slot = reinterpret_cast<void **>(&api);
    constexpr Py_ssize_t n = sizeof(Api) / sizeof(void *);
    if (PyTuple_GET_SIZE(table) != n) {
        PyErr_Format(PyExc_ValueError, "expected %zd entry points", n);
        return nullptr;
    }
    for (Py_ssize_t i = 0; i < n; ++i) {
        slot[i] = PyLong_AsVoidPtr(PyTuple_GET_ITEM(table, i));
        if (PyErr_Occurred()) return nullptr;
    }
    get_workspace = Py_NewRef(ws);
    raw_stream = Py_NewRef(stream);
    current_device = Py_NewRef(device);
    error_class = Py_NewRef(error);
    ready = true;
    Py_RETURN_NONE;
}

#ifdef ADASPEC_FASTCALL_ON_META
PyObject *set_meta_index(PyObject *, PyObject *i)
{
    meta_index = (int)PyLong_AsLong(i);
    Py_RETURN_NONE;
}
#endif

#define FASTCALL(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(name)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {FASTCALL(verify_attn), FASTCALL(accept), FASTCALL(accept_tree), FASTCALL(kv_append),
                         FASTCALL(kv_compact_path), FASTCALL(commit), FASTCALL(draft_sample),
#ifdef ADASPEC_FASTCALL_ON_META
                         {"set_meta_index", set_meta_index, METH_O, nullptr},
#endif
                         {"setup", setup, METH_VARARGS, nullptr}, {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_fastcall", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__fastcall()
{
    PyObject *m = PyModule_Create(&module);
    if (m && PyModule_AddStringConstant(m, "torch_version", ADASPEC_TORCH_VERSION) < 0) Py_CLEAR(m);
    return m;
}
