// The short way of `api.matmul`: a call on two plain CUDA tensors whose plan is known and needs no workspace, without Python
// objects per argument.  What it does not recognise (subclasses, modes, transforms, other devices, mistakes in the
// arguments) it leaves to the general way by returning None before anything has been done.
//
// Host time of a call whose kernel is shorter (16x64x64 bf16; processes come in two kinds, whose launches differ by 0.7 us):
// the general way 7.0 and 7.7 us, this one 3.6 and 4.3.  (Allocated through the dispatcher and launched by <<<>>> 4.05 and 4.75.)
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/Context.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <ATen/hip/EmptyTensor.h>
#include <ATen/ops/empty.h>
#include <c10/core/impl/LocalDispatchKeySet.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/hip/HIPFunctions.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstring>
#include <unordered_map>

#include "../../include/gemm.h"

namespace {
typedef int (*RunFn)(const gemm_cfg *, const void *, const void *, void *, void *);
RunFn run_fn = nullptr;
PyObject *make_plan = nullptr;    // api._fast_plan
PyObject *check_status = nullptr; // binding._check
PyObject *api_dict = nullptr;     // the module's namespace: holds the memo of picks

struct Key {
    int64_t v[8];      // M, N, K, dtype, B's layout, lda, ldb, ldc
    bool operator==(const Key &o) const { return !std::memcmp(v, o.v, sizeof(v)); }
};
struct KeyHash {
    size_t operator()(const Key &k) const
    {
        uint64_t h = 0x9e3779b97f4a7c15ull;
        for (int64_t x : k.v)
            h = (h ^ (uint64_t)x) * 0xff51afd7ed558ccdull, h ^= h >> 32;
        return (size_t)h;
    }
};
struct Plan {
    PyObject *pick_key, *base;   // the plan holds while the memo of picks holds `base` under `pick_key`
    gemm_cfg cfg;
    bool short_way;              // no workspace
};
constexpr size_t kMaxPlans = 4096;     // a program with more shapes than this starts over
typedef std::unordered_map<Key, Plan, KeyHash> Plans;
Plans plans;                           // (guarded by the interpreter lock)

// Gives up the plans of a map that is no longer `plans` (releasing an object may run code that comes back here).
void release(const Plans &gone)
{
    for (const auto &p : gone) {
        Py_DECREF(p.second.pick_key);
        Py_DECREF(p.second.base);
    }
}
void drop(Plans::iterator it)
{
    Plans gone;
    gone.insert(*it);
    plans.erase(it);
    release(gone);
}

// The plan of a call: its cfg and whether it goes the short way; false: a Python error if one is set, else the general way.
bool plan_of(const Key &key, gemm_cfg *cfg, bool *short_way)
{
    static PyObject *const memo_name = PyUnicode_InternFromString("_cfg_cache");
    PyObject *const memo = PyDict_GetItemWithError(api_dict, memo_name);
    if (!memo || !PyDict_CheckExact(memo))
        return false;
    auto it = plans.find(key);
    if (it != plans.end()) {
        if (PyDict_GetItemWithError(memo, it->second.pick_key) == it->second.base) {
            *cfg = it->second.cfg;
            *short_way = it->second.short_way;
            return true;
        }
        drop(it);
    }
    PyObject *const r = PyObject_CallFunction(make_plan, "LLLLLLLL", (long long)key.v[0], (long long)key.v[1], (long long)key.v[2],
                                              (long long)key.v[3], (long long)key.v[4], (long long)key.v[5], (long long)key.v[6],
                                              (long long)key.v[7]);
    if (!r)
        return false;
    Plan p;
    unsigned long long address, need;
    PyObject *cfg_object;     // (held by the result: the address stays good until it is released)
    if (!PyArg_ParseTuple(r, "OOOKK", &p.base, &p.pick_key, &cfg_object, &address, &need)) {
        Py_DECREF(r);
        return false;
    }
    Py_INCREF(p.pick_key);
    Py_INCREF(p.base);
    std::memcpy(&p.cfg, (const void *)(uintptr_t)address, sizeof(p.cfg));
    p.short_way = need == 0;
    *cfg = p.cfg;
    *short_way = p.short_way;
    Py_DECREF(r);
    it = plans.find(key);     // (another thread, or a call from inside this one, may have made it meanwhile)
    if (it != plans.end())
        drop(it);
    Plans gone;
    if (plans.size() >= kMaxPlans)
        gone.swap(plans);
    if (!plans.emplace(key, p).second) {
        Py_DECREF(p.pick_key);
        Py_DECREF(p.base);
    }
    release(gone);
    return true;
}

// Without the interpreter lock: the launch, and the result's allocation, which may wait for the device.
struct Unlocked {
    PyThreadState *const state = PyEval_SaveThread();
    ~Unlocked() { PyEval_RestoreThread(state); }
};

// A tensor that is nothing but memory on a GPU: no wrapper of a transform, no lazy bit.
inline bool plain(const at::Tensor &t)
{
    constexpr c10::DispatchKeySet known = c10::DispatchKeySet({c10::DispatchKey::CUDA, c10::DispatchKey::ADInplaceOrView}) |
                                          c10::autograd_dispatch_keyset_with_ADInplaceOrView | c10::autocast_dispatch_keyset;
    // (the difference of two key sets keeps the backend's bit: what counts is that no functionality is left)
    return t.is_cuda() && t.layout() == at::kStrided && t.has_storage() &&
           (t.key_set() - known).highestFunctionalityKey() == c10::DispatchKey::Undefined;
}

// at::empty of whole rows on the current device.  Without the dispatcher (0.25 us), except where something beside the operator
// would see the call (a transform, a trace, functionalisation, a Python dispatcher: what a thread adds to the keys that are
// always there), or the operator fills new memory.
at::Tensor empty_rows(int64_t rows, int64_t columns, at::ScalarType type, at::Device device)
{
    const auto &context = at::globalContext();
    if (!(c10::impl::tls_local_dispatch_key_set().included_ - c10::default_included_set).empty() ||
        (context.deterministicAlgorithms() && context.deterministicFillUninitializedMemory()))
        return at::empty({rows, columns}, at::TensorOptions().dtype(type).device(device));
    return at::Tensor(at::detail::empty_cuda({rows, columns}, type, device, std::nullopt));
}

PyObject *matmul(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    // A, B, out, alpha, beta, b_k_contiguous, stream
    if (n != 7 || !THPVariable_CheckExact(args[0]) || !THPVariable_CheckExact(args[1]) || !PyFloat_CheckExact(args[3]) ||
        !PyFloat_CheckExact(args[4]) || !PyBool_Check(args[5]) || args[6] != Py_None ||
        (args[2] != Py_None && !THPVariable_CheckExact(args[2])) || at::impl::torch_function_mode_enabled() ||
        c10::impl::dispatch_mode_enabled())
        Py_RETURN_NONE;
    const at::Tensor &A = THPVariable_Unpack(args[0]), &B = THPVariable_Unpack(args[1]);
    if (!plain(A) || !plain(B) || A.dim() != 2 || B.dim() != 2 || A.scalar_type() != B.scalar_type() || A.device() != B.device())
        Py_RETURN_NONE;
    int64_t dtype;
    switch (A.scalar_type()) {
    case at::kBFloat16: dtype = GEMM_BF16; break;
    case at::kHalf: dtype = GEMM_FP16; break;
    case at::kFloat8_e4m3fn: dtype = GEMM_FP8_E4M3; break;
    default: Py_RETURN_NONE;
    }
    const bool kc = args[5] == Py_True;
    const int64_t M = A.size(0), K = A.size(1), N = B.size(kc ? 0 : 1);
    const double alpha = PyFloat_AS_DOUBLE(args[3]), beta = PyFloat_AS_DOUBLE(args[4]);
    if (A.stride(1) != 1 || B.stride(1) != 1 || B.size(kc ? 1 : 0) != K || c10::hip::current_device() != A.device().index())
        Py_RETURN_NONE;
    const auto out_type = dtype == GEMM_FP16 ? at::kHalf : at::kBFloat16;
    int64_t ldc = (N + 7) / 8 * 8;
    if (args[2] != Py_None) {
        const at::Tensor &out = THPVariable_Unpack(args[2]);
        if (!plain(out) || out.dim() != 2 || out.size(0) != M || out.size(1) != N || out.scalar_type() != out_type ||
            out.stride(1) != 1 || out.device() != A.device())
            Py_RETURN_NONE;
        ldc = out.stride(0);
    } else if (beta != 0.0) {
        Py_RETURN_NONE;
    }
    gemm_cfg cfg;
    bool short_way = false;
    // (what making the plan raises, the general way would have raised: its own checks of the arguments have passed above)
    if (!plan_of({{M, N, K, dtype, kc, A.stride(0), B.stride(0), ldc}}, &cfg, &short_way) && PyErr_Occurred())
        return nullptr;
    if (!short_way)
        Py_RETURN_NONE;
    cfg.alpha = (float)alpha;
    cfg.beta = (float)beta;
    const bool own = args[2] == Py_None;
    at::Tensor made;
    int status;
    {
        Unlocked unlocked;
        void *c;
        if (own) {
            // rows of C start on 16-byte boundaries: a ragged N gets a padded row stride (the result is a view)
            made = empty_rows(M, ldc, out_type, A.device());
            if (ldc != N)
                made = made.narrow(1, 0, N);
            c = made.data_ptr();
        } else {
            c = THPVariable_Unpack(args[2]).data_ptr();
        }
        status = run_fn(&cfg, A.data_ptr(), B.data_ptr(), c, (void *)c10::hip::getCurrentHIPStream(A.device().index()).stream());
    }
    if (status != GEMM_OK) {
        PyObject *const r = PyObject_CallFunction(check_status, "is", status, "gemm_run");
        Py_XDECREF(r);
        if (!r)
            return nullptr;
        Py_RETURN_NONE;
    }
    if (own)
        return THPVariable_Wrap(std::move(made));
    Py_INCREF(args[2]);
    return args[2];
    END_HANDLE_TH_ERRORS
}

// (address of gemm_run, sizeof(gemm_cfg) as the caller knows it, api._fast_plan, binding._check, the api module's namespace)
PyObject *init(PyObject *, PyObject *args)
{
    unsigned long long address, cfg_bytes;
    PyObject *plan, *check, *names;
    if (!PyArg_ParseTuple(args, "KKOOO!", &address, &cfg_bytes, &plan, &check, &PyDict_Type, &names))
        return nullptr;
    if (cfg_bytes != sizeof(gemm_cfg)) {
        PyErr_SetString(PyExc_ImportError, "_fastcall and the binding disagree about gemm_cfg: build again");
        return nullptr;
    }
    Py_INCREF(plan);
    Py_INCREF(check);
    Py_INCREF(names);
    run_fn = (RunFn)(uintptr_t)address;
    make_plan = plan;
    check_status = check;
    api_dict = names;
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {{"matmul", (PyCFunction)(void (*)(void))matmul, METH_FASTCALL, nullptr},
                         {"init", init, METH_VARARGS, nullptr},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_fastcall", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};
}  // namespace

PyMODINIT_FUNC PyInit__fastcall()
{
    PyObject *const m = PyModule_Create(&module);
    if (m && PyModule_AddStringConstant(m, "torch_version", FASTCALL_TORCH) != 0) {
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
