// The binding's plain calls without Python in between: checks, output and workspace tensors and the library call of one operator in one C function.
//
// An operator on small matrices takes 2 to 10 us on the GPU; the same steps in
// Python take 8 to 10 us of host time a call, here 4.3 to 5, 3 of them the launch (16 matrices of 32 x 32).  A function
// here answers None, having done nothing, for everything but a plain call -- torch.Tensor arguments on the current device, dense, contiguous, of one
// precision, of shapes that fit, no mode or transform of torch active, flags and numbers of the usual types, sizes the library accepts -- and
// the Python code then runs as it would without it, errors included.
#include <Python.h>
#include <dlfcn.h>

#include <ATen/ATen.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <ATen/hip/impl/HIPStreamMasqueradingAsCUDA.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/hip/HIPFunctions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <initializer_list>
#include <mutex>
#include <stdexcept>
#include <tuple>
#include <unordered_map>

#include "la.h"

namespace {

struct Lib {
    decltype(&la_workspace_bytes) workspace_bytes;
    decltype(&la_gp_workspace_bytes) gp_workspace_bytes;
    decltype(&la_potrf_batched_ws) potrf;
    decltype(&la_potrf_backward_ws) potrf_backward;
    decltype(&la_trsm_batched_ws) trsm, trmm;
    decltype(&la_trsm_backward_ws) trsm_backward, trmm_backward;
    decltype(&la_syrk_batched_ws) syrk;
    decltype(&la_syrk_backward_ws) syrk_backward;
    decltype(&la_gemm2_batched_ws) gemm2;
    decltype(&la_gemm2_backward_ws) gemm2_backward;
    decltype(&la_potri_ws) potri;
    decltype(&la_potri_backward_ws) potri_backward;
    decltype(&la_sumlogdiag) sumlogdiag;
    decltype(&la_gp_criterion) gp_criterion;
} lib;
bool bound = false;

// Dense tensors of ordinary autograd; anything that wraps or records them (vmap, functionalisation, fake tensors, subclasses) goes by the Python code.
const c10::DispatchKeySet plain_keys({c10::DispatchKey::CUDA, c10::DispatchKey::AutogradCUDA, c10::DispatchKey::ADInplaceOrView,
                                      c10::DispatchKey::AutocastCUDA});

bool plain(const at::Tensor &t) { return (t.key_set() | plain_keys) == plain_keys; }

// A result or scratch tensor: plain as well, or the call is none of this file's.
at::Tensor fresh(at::IntArrayRef sizes, const at::TensorOptions &options)
{
    at::Tensor t = at::empty(sizes, options.requires_grad(false));
    if (!plain(t))
        throw std::runtime_error("not a plain tensor");
    return t;
}

// One call's tensors.
struct Call {
    const at::Tensor *first = nullptr;
    la_dtype dt = LA_F32;
    int device = -1;
    int64_t batch = 0;
    at::Tensor workspace;  // kept until the call is enqueued
    void *wp = nullptr;
    size_t wb = 0;

    // the tensor behind `o`, or null where the call is not a plain one
    const at::Tensor *tensor(PyObject *o)
    {
        if (!THPVariable_CheckExact(o))
            return nullptr;
        const at::Tensor &t = THPVariable_Unpack(o);
        if (!t.defined() || !t.is_cuda() || t.layout() != c10::kStrided || !plain(t) || !t.is_contiguous() ||
            t.dim() > 8)
            return nullptr;
        if (!first) {
            if (t.scalar_type() == at::kFloat)
                dt = LA_F32;
            else if (t.scalar_type() == at::kDouble)
                dt = LA_F64;
            else
                return nullptr;
            device = t.get_device();
            first = &t;
        } else if (t.scalar_type() != first->scalar_type() || t.get_device() != device) {
            return nullptr;
        }
        return &t;
    }
    // plain circumstances: asked once the tensors are there.  (A mode or a transform -- grad, jvp, vmap, functionalisation, tracing -- wraps what is
    // allocated inside it, whatever the arguments are: its key is among the included ones.)
    bool here() const
    {
        return bound && device == c10::hip::current_device() && !c10::impl::TorchDispatchModeTLS::any_modes_set() &&
               !at::impl::torch_function_mode_enabled() &&
               (c10::impl::tls_local_dispatch_key_set().included_ | c10::default_included_set) == c10::default_included_set;
    }
    void scratch(size_t need)
    {
        if (!need)
            return;
        workspace = fresh({(int64_t)need}, first->options().dtype(at::kByte));
        wp = workspace.data_ptr();
        wb = need;
    }
    // bytes of an operator's workspace; the answers are remembered, they depend on the sizes only
    void scratch(la_op op, int n, int m, int k)
    {
        using Key = std::tuple<int, int, int64_t, int, int, int>;
        struct Hash {
            size_t operator()(const Key &x) const
            {
                size_t h = (size_t)std::get<2>(x);
                for (size_t v : {(size_t)std::get<0>(x), (size_t)std::get<1>(x), (size_t)std::get<3>(x), (size_t)std::get<4>(x), (size_t)std::get<5>(x)})
                    h = h * 1000003u + v;
                return h;
            }
        };
        static std::mutex mutex;
        static std::unordered_map<Key, size_t, Hash> sizes;
        const Key key{(int)op, (int)dt, batch, n, m, k};
        size_t need;
        {
            std::lock_guard<std::mutex> lock(mutex);
            const auto it = sizes.find(key);
            if (it != sizes.end()) {
                need = it->second;
            } else {
                need = lib.workspace_bytes(op, dt, batch, n, m, k);
                if (sizes.size() >= 4096)  // (a program with that many sizes asks again)
                    sizes.clear();
                sizes.emplace(key, need);
            }
        }
        scratch(need);
    }
    void *stream() const { return (void *)c10::hip::getCurrentHIPStreamMasqueradingAsCUDA(device).stream(); }
};

int64_t leading(const at::Tensor &t, int trailing)
{
    int64_t b = 1;
    for (int64_t i = 0; i < t.dim() - trailing; ++i)
        b *= t.size(i);
    return b;
}

bool small(int64_t x) { return x >= 0 && x <= (1 << 20); }
bool flag(PyObject *o, int &v)
{
    if (!PyBool_Check(o))
        return false;
    v = o == Py_True;
    return true;
}
bool number(PyObject *o, double &v)
{
    if (!PyFloat_CheckExact(o))
        return false;
    v = PyFloat_AS_DOUBLE(o);
    return true;
}

// Allocations and the library's call, without the GIL, as torch makes its own: an allocation may wait for the GPU, and the GPU for a callback in
// Python.  An exception does not leave with the GIL released.  (Only std::exception is caught, here and below: a thread that meets the end of the
// interpreter where it takes the GIL back is unwound, which must not be held up.)
template <class F>
la_status unlocked(F &&f)
{
    la_status s = LA_ERR_RUNTIME;
    PyThreadState *state = PyEval_SaveThread();
    try {
        s = f();
    } catch (const std::exception &) {
    }
    PyEval_RestoreThread(state);
    return s;
}

PyObject *wrap(const at::Tensor &t) { return THPVariable_Wrap(t); }
PyObject *pair(const at::Tensor &a, const at::Tensor &b)
{
    PyObject *x = wrap(a), *y = x ? wrap(b) : nullptr, *r = y ? PyTuple_Pack(2, x, y) : nullptr;
    Py_XDECREF(x);
    Py_XDECREF(y);
    return r;
}
at::Tensor like(const at::Tensor &t) { return fresh(t.sizes(), t.options()); }
at::Tensor shaped(const at::Tensor &t, int drop, std::initializer_list<int64_t> last)
{
    std::vector<int64_t> s(t.sizes().begin(), t.sizes().end() - drop);
    s.insert(s.end(), last);
    return fresh(s, t.options());
}

// A C++ exception (no memory, say) leaves the call to the Python code, which meets it again and reports it as ever.
#define LA_FUNCTION(name, count)                                                       \
    PyObject *name##_call(PyObject *const *a);                                         \
    PyObject *name(PyObject *, PyObject *const *a, Py_ssize_t n)                       \
    {                                                                                  \
        if (n == (count)) {                                                            \
            try {                                                                      \
                if (PyObject *r = name##_call(a))                                      \
                    return r;                                                          \
            } catch (const std::exception &) {                                         \
            }                                                                          \
            if (PyErr_Occurred())                                                      \
                PyErr_Clear();                                                         \
        }                                                                              \
        Py_RETURN_NONE;                                                                \
    }                                                                                  \
    PyObject *name##_call(PyObject *const *a)

// a batch of square matrices
bool square(const at::Tensor *t, int64_t &n)
{
    if (!t || t->dim() < 2)
        return false;
    n = t->size(-1);
    return t->size(-2) == n && small(n);
}

LA_FUNCTION(potrf, 2)
{
    Call c;
    int64_t n;
    int lower;
    const at::Tensor *A = c.tensor(a[0]);
    if (!square(A, n) || !flag(a[1], lower) || !c.here())
        return nullptr;
    c.batch = leading(*A, 2);
    at::Tensor L;
    void *st = c.stream();
    const la_status s = unlocked([&] {
        L = like(*A);
        c.scratch(LA_OP_POTRF, (int)n, 0, 0);
        return lib.potrf(c.dt, lower, c.batch, (int)n, A->data_ptr(), L.data_ptr(), nullptr, c.wp, c.wb, st);
    });
    return s == LA_OK ? wrap(L) : nullptr;
}

LA_FUNCTION(potrf_backward, 3)
{
    Call c;
    int64_t n;
    int lower;
    const at::Tensor *L = c.tensor(a[0]), *G = L ? c.tensor(a[1]) : nullptr;
    if (!square(L, n) || !G || G->sizes() != L->sizes() || !flag(a[2], lower) || !c.here())
        return nullptr;
    c.batch = leading(*L, 2);
    at::Tensor W;
    void *st = c.stream();
    const la_status s = unlocked([&] {
        W = like(*G);
        c.scratch(LA_OP_POTRF_BACKWARD, (int)n, 0, 0);
        return lib.potrf_backward(c.dt, lower, c.batch, (int)n, L->data_ptr(), G->data_ptr(), W.data_ptr(), c.wp, c.wb, st);
    });
    return s == LA_OK ? wrap(W) : nullptr;
}

// the vectors of trsm / trmm: m of them, or -1
int64_t vectors(const at::Tensor &L, const at::Tensor *X, int64_t n, int right)
{
    if (!X || X->dim() < 2 || X->size(right ? -1 : -2) != n || leading(*X, 2) != leading(L, 2))
        return -1;
    return X->size(right ? -2 : -1);
}

// (solve, L, A, lower, trans, rightside, alpha)
LA_FUNCTION(tri, 7)
{
    Call c;
    int64_t n;
    int solve, lower, trans, right;
    double alpha;
    const at::Tensor *L = c.tensor(a[1]), *A = L ? c.tensor(a[2]) : nullptr;
    if (!square(L, n) || !flag(a[0], solve) || !flag(a[3], lower) || !flag(a[4], trans) || !flag(a[5], right) || !number(a[6], alpha))
        return nullptr;
    const int64_t m = vectors(*L, A, n, right);
    if (m < 0 || m > INT32_MAX || !c.here())
        return nullptr;
    c.batch = leading(*L, 2);
    at::Tensor B;
    void *st = c.stream();
    const la_status s = unlocked([&] {
        B = like(*A);
        c.scratch(solve ? LA_OP_TRSM : LA_OP_TRMM, (int)n, (int)m, 0);
        return (solve ? lib.trsm : lib.trmm)(c.dt, lower, trans, right, alpha, c.batch, (int)n, (int)m, L->data_ptr(), A->data_ptr(), B.data_ptr(),
                                             c.wp, c.wb, st);
    });
    return s == LA_OK ? wrap(B) : nullptr;
}

// (solve, L, X, Bbar, lower, trans, rightside, alpha)
LA_FUNCTION(tri_backward, 8)
{
    Call c;
    int64_t n;
    int solve, lower, trans, right;
    double alpha;
    const at::Tensor *L = c.tensor(a[1]), *X = L ? c.tensor(a[2]) : nullptr, *G = X ? c.tensor(a[3]) : nullptr;
    if (!square(L, n) || !G || !flag(a[0], solve) || !flag(a[4], lower) || !flag(a[5], trans) || !flag(a[6], right) || !number(a[7], alpha) ||
        X->sizes() != G->sizes())
        return nullptr;
    const int64_t m = vectors(*L, X, n, right);
    if (m < 0 || m > INT32_MAX || !c.here())
        return nullptr;
    c.batch = leading(*L, 2);
    at::Tensor Ab, Lb;
    void *st = c.stream();
    const la_status s = unlocked([&] {
        Ab = like(*G);
        Lb = like(*L);
        c.scratch(solve ? LA_OP_TRSM_BACKWARD : LA_OP_TRMM_BACKWARD, (int)n, (int)m, 0);
        return (solve ? lib.trsm_backward : lib.trmm_backward)(c.dt, lower, trans, right, alpha, c.batch, (int)n, (int)m, L->data_ptr(),
                                                               X->data_ptr(), G->data_ptr(), Ab.data_ptr(), Lb.data_ptr(), c.wp, c.wb, st);
    });
    return s == LA_OK ? pair(Ab, Lb) : nullptr;
}

LA_FUNCTION(syrk, 3)
{
    Call c;
    int trans;
    double alpha;
    const at::Tensor *A = c.tensor(a[0]);
    if (!A || A->dim() < 2 || !flag(a[1], trans) || !number(a[2], alpha))
        return nullptr;
    const int64_t n = A->size(trans ? -1 : -2), k = A->size(trans ? -2 : -1);
    if (!small(n) || k > INT32_MAX || !c.here())
        return nullptr;
    c.batch = leading(*A, 2);
    at::Tensor B;
    void *st = c.stream();
    const la_status s = unlocked([&] {
        B = shaped(*A, 2, {n, n});
        c.scratch(LA_OP_SYRK, (int)n, 0, (int)k);
        return lib.syrk(c.dt, trans, alpha, c.batch, (int)n, (int)k, A->data_ptr(), B.data_ptr(), c.wp, c.wb, st);
    });
    return s == LA_OK ? wrap(B) : nullptr;
}

LA_FUNCTION(syrk_backward, 4)
{
    Call c;
    int trans;
    double alpha;
    const at::Tensor *A = c.tensor(a[0]), *G = A ? c.tensor(a[1]) : nullptr;
    if (!G || A->dim() < 2 || G->dim() < 2 || !flag(a[2], trans) || !number(a[3], alpha))
        return nullptr;
    const int64_t n = A->size(trans ? -1 : -2), k = A->size(trans ? -2 : -1);
    if (G->size(-1) != n || G->size(-2) != n || leading(*A, 2) != leading(*G, 2) || !small(n) || k > INT32_MAX || !c.here())
        return nullptr;
    c.batch = leading(*A, 2);
    at::Tensor B;
    void *st = c.stream();
    const la_status s = unlocked([&] {
        B = like(*A);
        c.scratch(LA_OP_SYRK_BACKWARD, (int)n, 0, (int)k);
        return lib.syrk_backward(c.dt, trans, alpha, c.batch, (int)n, (int)k, A->data_ptr(), G->data_ptr(), B.data_ptr(), c.wp, c.wb, st);
    });
    return s == LA_OK ? wrap(B) : nullptr;
}

// sizes of C = t_a(A) t_b(B)
bool product(const at::Tensor *A, const at::Tensor *B, int ta, int tb, int64_t &m, int64_t &n, int64_t &k)
{
    if (!A || !B || A->dim() < 2 || B->dim() < 2)
        return false;
    m = A->size(ta ? -1 : -2);
    k = A->size(ta ? -2 : -1);
    n = B->size(tb ? -2 : -1);
    return B->size(tb ? -1 : -2) == k && leading(*A, 2) == leading(*B, 2) && m <= INT32_MAX && n <= INT32_MAX && k <= INT32_MAX;
}

LA_FUNCTION(gemm2, 5)
{
    Call c;
    int ta, tb;
    double alpha;
    int64_t m, n, k;
    const at::Tensor *A = c.tensor(a[0]), *B = A ? c.tensor(a[1]) : nullptr;
    if (!flag(a[2], ta) || !flag(a[3], tb) || !number(a[4], alpha) || !product(A, B, ta, tb, m, n, k) || !c.here())
        return nullptr;
    c.batch = leading(*A, 2);
    at::Tensor C;
    void *st = c.stream();
    const la_status s = unlocked([&] {
        C = shaped(*A, 2, {m, n});
        c.scratch(LA_OP_GEMM2, (int)n, (int)m, (int)k);
        return lib.gemm2(c.dt, ta, tb, alpha, c.batch, (int)m, (int)n, (int)k, A->data_ptr(), B->data_ptr(), C.data_ptr(), c.wp, c.wb, st);
    });
    return s == LA_OK ? wrap(C) : nullptr;
}

LA_FUNCTION(gemm2_backward, 6)
{
    Call c;
    int ta, tb;
    double alpha;
    int64_t m, n, k;
    const at::Tensor *A = c.tensor(a[0]), *B = A ? c.tensor(a[1]) : nullptr, *G = B ? c.tensor(a[2]) : nullptr;
    if (!G || !flag(a[3], ta) || !flag(a[4], tb) || !number(a[5], alpha) || !product(A, B, ta, tb, m, n, k) || G->dim() < 2 || G->size(-2) != m ||
        G->size(-1) != n || leading(*G, 2) != leading(*A, 2) || !c.here())
        return nullptr;
    c.batch = leading(*A, 2);
    at::Tensor Ab, Bb;
    void *st = c.stream();
    const la_status s = unlocked([&] {
        Ab = like(*A);
        Bb = like(*B);
        c.scratch(LA_OP_GEMM2_BACKWARD, (int)n, (int)m, (int)k);
        return lib.gemm2_backward(c.dt, ta, tb, alpha, c.batch, (int)m, (int)n, (int)k, A->data_ptr(), B->data_ptr(), G->data_ptr(), Ab.data_ptr(),
                                  Bb.data_ptr(), c.wp, c.wb, st);
    });
    return s == LA_OK ? pair(Ab, Bb) : nullptr;
}

LA_FUNCTION(potri, 2)
{
    Call c;
    int64_t n;
    int lower;
    const at::Tensor *L = c.tensor(a[0]);
    if (!square(L, n) || !flag(a[1], lower) || !c.here())
        return nullptr;
    c.batch = leading(*L, 2);
    at::Tensor B;
    void *st = c.stream();
    const la_status s = unlocked([&] {
        B = like(*L);
        c.scratch(LA_OP_POTRI, (int)n, 0, 0);
        return lib.potri(c.dt, lower, c.batch, (int)n, L->data_ptr(), B.data_ptr(), c.wp, c.wb, st);
    });
    return s == LA_OK ? wrap(B) : nullptr;
}

LA_FUNCTION(potri_backward, 4)
{
    Call c;
    int64_t n;
    int lower;
    const at::Tensor *L = c.tensor(a[0]), *B = L ? c.tensor(a[1]) : nullptr, *G = B ? c.tensor(a[2]) : nullptr;
    if (!square(L, n) || !G || B->sizes() != L->sizes() || G->sizes() != L->sizes() || !flag(a[3], lower) || !c.here())
        return nullptr;
    c.batch = leading(*L, 2);
    at::Tensor X;
    void *st = c.stream();
    const la_status s = unlocked([&] {
        X = like(*L);
        c.scratch(LA_OP_POTRI_BACKWARD, (int)n, 0, 0);
        return lib.potri_backward(c.dt, lower, c.batch, (int)n, L->data_ptr(), B->data_ptr(), G->data_ptr(), X.data_ptr(), c.wp, c.wb, st);
    });
    return s == LA_OK ? wrap(X) : nullptr;
}

LA_FUNCTION(sumlogdiag, 1)
{
    Call c;
    const at::Tensor *L = c.tensor(a[0]);
    int64_t n;
    if (!square(L, n) || !c.here())
        return nullptr;
    at::Tensor o;
    void *st = c.stream();
    const int64_t batch = leading(*L, 2);
    const la_status s = unlocked([&] {
        o = shaped(*L, 2, {});
        return lib.sumlogdiag(c.dt, batch, (int)n, L->data_ptr(), o.data_ptr(), st);
    });
    return s == LA_OK ? wrap(o) : nullptr;
}

LA_FUNCTION(gp_criterion, 2)
{
    Call c;
    int64_t n;
    const at::Tensor *A = c.tensor(a[0]), *y = A ? c.tensor(a[1]) : nullptr;
    if (!square(A, n) || !y || y->dim() < 1 || y->size(-1) != n || leading(*y, 1) != leading(*A, 2) || !c.here())
        return nullptr;
    c.batch = leading(*A, 2);
    at::Tensor Ab, loss;
    void *st = c.stream();
    const la_status s = unlocked([&] {
        Ab = like(*A);
        loss = shaped(*A, 2, {});
        c.scratch(lib.gp_workspace_bytes(c.dt, c.batch, (int)n));
        return lib.gp_criterion(c.dt, c.batch, (int)n, A->data_ptr(), y->data_ptr(), loss.data_ptr(), Ab.data_ptr(), nullptr, c.wp, c.wb, st);
    });
    return s == LA_OK ? pair(loss, Ab) : nullptr;
}

// bind(path): the library whose functions are called
PyObject *bind(PyObject *, PyObject *path)
{
    const char *p = PyUnicode_AsUTF8(path);
    if (!p)
        return nullptr;
    void *h = dlopen(p, RTLD_NOW | RTLD_LOCAL);
    if (!h)
        return PyErr_Format(PyExc_OSError, "%s", dlerror());
#define LA_BIND(member, symbol)                                                         \
    if (!(lib.member = reinterpret_cast<decltype(lib.member)>(dlsym(h, #symbol))))      \
    return PyErr_Format(PyExc_OSError, "%s has no %s", p, #symbol)
    LA_BIND(workspace_bytes, la_workspace_bytes);
    LA_BIND(gp_workspace_bytes, la_gp_workspace_bytes);
    LA_BIND(potrf, la_potrf_batched_ws);
    LA_BIND(potrf_backward, la_potrf_backward_ws);
    LA_BIND(trsm, la_trsm_batched_ws);
    LA_BIND(trmm, la_trmm_batched_ws);
    LA_BIND(trsm_backward, la_trsm_backward_ws);
    LA_BIND(trmm_backward, la_trmm_backward_ws);
    LA_BIND(syrk, la_syrk_batched_ws);
    LA_BIND(syrk_backward, la_syrk_backward_ws);
    LA_BIND(gemm2, la_gemm2_batched_ws);
    LA_BIND(gemm2_backward, la_gemm2_backward_ws);
    LA_BIND(potri, la_potri_ws);
    LA_BIND(potri_backward, la_potri_backward_ws);
    LA_BIND(sumlogdiag, la_sumlogdiag);
    LA_BIND(gp_criterion, la_gp_criterion);
#undef LA_BIND
    bound = true;
    Py_RETURN_NONE;
}

#define LA_METHOD(name) {#name, (PyCFunction)(void (*)(void))name, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {LA_METHOD(potrf), LA_METHOD(potrf_backward), LA_METHOD(tri), LA_METHOD(tri_backward), LA_METHOD(syrk), LA_METHOD(syrk_backward),
                         LA_METHOD(gemm2), LA_METHOD(gemm2_backward), LA_METHOD(potri), LA_METHOD(potri_backward), LA_METHOD(sumlogdiag),
                         LA_METHOD(gp_criterion), {"bind", bind, METH_O, nullptr}, {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_la_host", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__la_host() { return PyModule_Create(&module); }
