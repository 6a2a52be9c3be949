// C ABI (include/wht_affine.h) and host-side dispatch of the Walsh-Hadamard output layer
//     y = alpha (.) (H x) + beta                                   (paper Sec. 4.1, Eq. 1)
// for gfx950.  The kernels live in wht_device.h, the stage schedules in wht_plan.h.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stdlib.h>
#include <string.h>

#include <mutex>

#include "../../include/wht_affine.h"
#include "wht_device.h"
#include "wht_validate.h"

namespace wht {

// ------------------------------------------------------------------------------------------------
// host side: launch shapes and dispatch

constexpr int kNumCU = 256;             // MI355X

enum class Op { Forward, Backward, Workspace };

struct Args {
    const void* x; const void* dy; const void* resid; const float* alpha; const float* beta;
    void* y; void* dx; float* dalpha; float* dbeta; float* sumsq;
    int64_t N; void* workspace; hipStream_t stream;
    size_t workspace_out;
};

// Workgroups launched per CU: the grid is persistent, each workgroup strides over token groups.  The
// per-configuration figures (C::kFwdGroupsPerCU, C::kBwdGroupsPerCU) are measured optima; the launch
// shape, and with it the backward workspace size, depends on (N, d, dtype) alone.
template <class C>
static int grid_for(int64_t N, bool backward) {
    const int64_t groups = (N + C::G - 1) / C::G;
    int per_cu = backward ? C::kBwdGroupsPerCU : C::kFwdGroupsPerCU;
    // float32 d = 4096: up to three token groups per CU a second workgroup there costs more in partial rows
    // than it saves (one / two per CU, us per call: N = 512 15.8 / 18.9, 768 18.9 / 19.2, 1024 22.2 / 21.9)
    if constexpr (C::kWave)
        if (backward && C::w == 1 && groups <= 3 * kNumCU) per_cu = 1;
    const int64_t cap = (int64_t)kNumCU * per_cu;
    return (int)(groups < cap ? groups : cap);
}

// Workgroups per cluster of the forward kernel: the configuration's figure when the grid divides
// into such clusters and every workgroup has many token groups to walk, else the whole grid.  Clusters spread
// the loss at unlucky address distances (see MfmaCfg), but each ends with its own ragged last round and their
// windows make short tensors slower.  us per call over 32 distances between x and y, clustered mean (worst) / plain mean
// (worst): 16 rounds of 4096 45.7 (48.4) / 45.1 (48.7), of 8192 46.5 (48.2) / 45.8 (49.2); 20 rounds 55.8 (57.0) / 56.9
// (64.1) and 56.5 (57.8) / 56.8 (64.3); 28 rounds 77.7 (79.0) / 80.6 (93.2) and 78.2 (79.8) / 79.2 (90.4), of float32
// 1024 76.6 (78.1) / 78.5 (89.4); 40 rounds 111.5 (113.1) / 116.2 (134.4) and 111.8 (113.5) / 117.4 (134.8); 8 rounds 25.1 / 24.2
// and 24.9 / 24.3.  Rows of 12 * 2^m: 28 rounds of 3072 61.1 (61.9) / 60.3 (62.2), 48 102.7 (104.4) / 103.0 (111.7), of 6144 28
// 61.0 / 60.9, 48 103.1 (104.5) / 103.5 (112.4).
template <class C>
static int forward_cluster(int64_t N, int grid, bool resid) {
    const int64_t groups = (N + C::G - 1) / C::G;
    const int want = resid ? C::kFwdClusterResid : C::kFwdCluster;
    constexpr int rounds = C::kTwelve ? 48 : 20;
    if (want > 0 && grid % want == 0 && grid > want && groups >= rounds * (int64_t)grid) return want;
    return grid;
}

template <class C>
static int64_t bytes_of(int64_t N) { return N * C::kRow * (int64_t)sizeof(typename C::io::elem_t); }

// f(false type or true type): a choice made at run time as a template argument.
template <class F>
static void with_bool(bool b, F&& f) {
    if (b) f(std::true_type{});
    else f(std::false_type{});
}

template <class C, Out OUT, bool THROUGH, int R>
static void launch_forward_once(const Args& a) {
    using T = typename C::io::elem_t;
    const int grid = (int)((a.N + C::G * R - 1) / (C::G * R));
    hipLaunchKernelGGL((forward_once_kernel<C, OUT != Out::Y, OUT == Out::Stats, THROUGH, R>), dim3(grid), dim3(C::BT), 0, a.stream,
                       static_cast<const T*>(a.x), a.alpha, a.beta, static_cast<const T*>(a.resid), static_cast<T*>(a.y), a.sumsq, a.N);
}

template <class C, Out OUT, bool THROUGH>
static void launch_forward(const Args& a) {
    using T = typename C::io::elem_t;
    const int grid = grid_for<C>(a.N, false);
    const int cluster = forward_cluster<C>(a.N, grid, OUT != Out::Y);
    hipLaunchKernelGGL((forward_kernel<C, OUT != Out::Y, OUT == Out::Stats, THROUGH>), dim3(grid), dim3(C::BT), 0, a.stream,
                       static_cast<const T*>(a.x), a.alpha, a.beta, static_cast<const T*>(a.resid), static_cast<T*>(a.y), a.sumsq, a.N,
                       cluster);
}

// CF: configuration of the persistent kernel, CO: of the one-pass kernel.
template <class CF, class CO, Out OUT>
static int forward_out(const Args& a) {
    const Way way = forward_way(rows_of<CO>(), OUT, bytes_of<CO>(a.N));
    constexpr auto reaches = [](Way w) { return forward_reaches(rows_of<CO>(), OUT, w); };
    static_assert(reaches(Way::Plain) && reaches(Way::Stream) && (CO::kMfma || !reaches(Way::Pair)));
    if (way == Way::Plain) launch_forward_once<CO, OUT, false, 1>(a);
    if constexpr (reaches(Way::Through))
        if (way == Way::Through) launch_forward_once<CO, OUT, true, 1>(a);
    if constexpr (reaches(Way::Pair))
        if (way == Way::Pair) launch_forward_once<CO, OUT, true, 2>(a);
    if (way == Way::Stream) launch_forward<CF, OUT, false>(a);
    if constexpr (reaches(Way::Flow) && !CF::kKeep)                 // x that is kept lies below the sizes of Flow
        if (way == Way::Flow) launch_forward<CF, OUT, true>(a);
    return hipGetLastError() == hipSuccess ? WHT_OK : WHT_ERR_LAUNCH;
}

template <class CF, class CO>
static int forward(const Args& a) {
    if (!a.resid) return forward_out<CF, CO, Out::Y>(a);
    return a.sumsq ? forward_out<CF, CO, Out::Stats>(a) : forward_out<CF, CO, Out::Resid>(a);
}

// Configurations whose calls of few elements run on backward_few_kernel; of rows of 768, the one of small calls.
template <class C>
constexpr bool has_few() { return has_few_backward(rows_of<C>()) && (!C::kTwelve || (C::kKeep && (C::kRow > 768 || C::BT == 128))); }

template <class C>
static int launch_backward(const void* dy, const void* x, const float* alpha, void* dx, float* dalpha,
                           float* dbeta, int64_t N, void* workspace, hipStream_t stream) {
    using T = typename C::io::elem_t;
    const bool grads = dalpha != nullptr;
    if constexpr (has_few<C>()) {
        const bool in_place = dx && (dx == dy || dx == x);
        if (grads && takes_few_backward(rows_of<C>(), N, dalpha == alpha || dbeta == alpha)) {
            const int64_t groups = dx && !in_place ? (N + C::G - 1) / C::G : 0;
            hipLaunchKernelGGL(backward_few_kernel<C>, dim3((unsigned)(FewSlices<C>::A + groups)), dim3(kFewThreads), 0, stream,
                               static_cast<const T*>(dy), static_cast<const T*>(x), alpha, static_cast<T*>(dx), dalpha, dbeta, N);
            if (hipGetLastError() != hipSuccess) return WHT_ERR_LAUNCH;
            return in_place ? launch_backward<C>(dy, nullptr, alpha, dx, nullptr, nullptr, N, nullptr, stream) : WHT_OK;
        }
    }
    const bool direct = grads && N <= one_workgroup_groups(rows_of<C>()) * C::G;
    const int grid = direct ? 1 : grid_for<C>(N, grads);      // dx alone streams like a forward pass
    float* ws = static_cast<float*>(workspace);
    const SumRows sums = direct ? SumRows{dalpha, dbeta, 0} : SumRows{ws, ws + C::kRow, 2 * C::kRow};

    auto launch = [&](auto kernel, int threads) {
        hipLaunchKernelGGL(kernel, dim3(grid), dim3(threads), 0, stream, static_cast<const T*>(dy), static_cast<const T*>(x),
                           alpha, static_cast<T*>(dx), sums, N);
    };
    const bool through = dx_through(rows_of<C>(), grads, bytes_of<C>(N));
    if (grads && !dx) {
        if constexpr (C::kWave) launch(backward_wave_kernel<C, true, false, false>, C::BT);
        else launch(backward_kernel<C, true, false, false>, C::BT);
    } else if (grads) {
        with_bool(through, [&](auto b) {
            constexpr bool THROUGH = (C::kTwelve && C::kKeep) || decltype(b)::value;      // always where x and dy are kept
            if constexpr (C::kWave) launch(backward_wave_kernel<C, true, true, THROUGH>, C::BT);
            else if constexpr (C::kBwdTeams) launch(backward_teams_kernel<C, THROUGH>, 3 * C::BT);
            else launch(backward_kernel<C, true, true, THROUGH>, C::BT);
        });
    } else {
        with_bool(through, [&](auto b) {
            if constexpr (C::kWave) launch(backward_wave_kernel<C, false, true, decltype(b)::value>, C::BT);
            else launch(backward_kernel<C, false, true, decltype(b)::value>, C::BT);
        });
    }
    if (hipGetLastError() != hipSuccess) return WHT_ERR_LAUNCH;
    if (!grads || direct) return WHT_OK;
    constexpr int CG = reduce_columns(C::kRow);
    hipLaunchKernelGGL(reduce_partials_kernel<CG>, dim3((C::kRow / 4 + CG - 1) / CG, 2), dim3(kReduceThreads), 0, stream,
                       ws, grid, C::kRow, dalpha, dbeta);
    return hipGetLastError() == hipSuccess ? WHT_OK : WHT_ERR_LAUNCH;
}

template <class C>
static size_t workspace_for(int64_t N) { return (size_t)grid_for<C>(N, true) * 2 * C::kRow * sizeof(float); }

// CF: configuration of the forward kernels, CB: of the backward kernels (and its workspace), CO: of
// the forward kernel for few tokens.
template <class CF, class CB = CF, class CO = CF>
static int run(Op op, Args& a) {
    switch (op) {
    case Op::Forward:
        return forward<CF, CO>(a);
    case Op::Backward: return launch_backward<CB>(a.dy, a.x, a.alpha, a.dx, a.dalpha, a.dbeta, a.N,
                                                  a.workspace, a.stream);
    default:           a.workspace_out = workspace_for<CB>(a.N); return WHT_OK;
    }
}

// Schedule choice: bfloat16 tokens of 1024 elements or more take the matrix-core schedule, the
// rest the wave schedule, in which every stage is additions.  WHT_AFFINE_SCHEDULE=butterfly in the
// environment (read once per process; the library's only environment variable) forces the wave
// schedule for those too: it exists so that both schedules of one build can be tested and profiled against each other.
static bool use_mfma() {
    static const bool on = [] {
        const char* v = getenv("WHT_AFFINE_SCHEDULE");
        return !(v && strcmp(v, "butterfly") == 0);
    }();
    return on;
}

template <class Io, int LOGD>
static int run_d(Op op, Args& a) {
    if constexpr (std::is_same<Io, IoBF16>::value && LOGD >= 10) {
        if (use_mfma())
            return run<MfmaCfg<LOGD, mfma_log_tiles(LOGD, false)>, MfmaCfg<LOGD, mfma_log_tiles(LOGD, true)>,
                       MfmaCfg<LOGD, mfma_log_tiles_few(LOGD)>>(op, a);
    }
    return run<WaveCfg<LOGD, wave_log_e(LOGD, Io::kLogVec), Io>>(op, a);
}

// The debug build that poisons LDS after every read (WHT_POISON_LDS, libwht_affine_poison.so, loaded
// by one GPU test only) carries a few widths that between them use every kernel and every kind of
// LDS hand-over; the others are left out of it to keep its compile time short.
#ifdef WHT_POISON_LDS
#define WHT_ALL_WIDTHS 0
#else
#define WHT_ALL_WIDTHS 1
#endif

template <class Io>
static int dispatch_d(int logd, Op op, Args& a) {
    switch (logd) {
#if WHT_ALL_WIDTHS
    case 5:  return run_d<Io, 5>(op, a);
    case 6:  return run_d<Io, 6>(op, a);
    case 7:  return run_d<Io, 7>(op, a);
    case 8:  return run_d<Io, 8>(op, a);
    case 10: return run_d<Io, 10>(op, a);
    case 11: return run_d<Io, 11>(op, a);
#endif
    case 9:  return run_d<Io, 9>(op, a);
    case 12: return run_d<Io, 12>(op, a);
    case 13: return run_d<Io, 13>(op, a);
    case 14:
        if constexpr (std::is_same<Io, IoBF16>::value) return run_d<Io, 14>(op, a);
        return WHT_ERR_BAD_DIM;
    default: return WHT_ERR_BAD_DIM;
    }
}

// Rows of 12 * 2^m elements (bfloat16); logd = m + 4.
using SmallBackwardCfg = TwelveCfg<6, true, 128>;

template <int M>
static int run_twelve(Op op, Args& a) {
    const int64_t bytes = bytes_of<TwelveCfg<M>>(a.N);
    if (op == Op::Forward) {
        if (forward_keeps(M, a.resid != nullptr, bytes)) return forward<TwelveCfg<M, true>, TwelveCfg<M, false, 64>>(a);
        return forward<TwelveCfg<M>, TwelveCfg<M, false, 64>>(a);
    }
    if (op == Op::Workspace) {
        a.workspace_out = workspace_for<TwelveCfg<M>>(a.N);
        if constexpr (M == 6)
            if (a.N > 2 * TwelveCfg<M>::G) {                // what suffices for N tokens suffices for fewer
                const size_t small = workspace_for<SmallBackwardCfg>(a.N < kSmallBackwardTokens ? a.N : kSmallBackwardTokens);
                if (a.workspace_out < small) a.workspace_out = small;
            }
        return WHT_OK;
    }
    if constexpr (M == 6) {
        // What is neither few elements nor up to four tokens, and fits one workgroup of 256 threads, runs there: it saves the second
        // launch, and the workspace of so few tokens has no rows for groups of four.
        constexpr Rows rows = rows_of<SmallBackwardCfg>();
        const bool few = takes_few_backward(rows, a.N, a.dalpha == a.alpha || a.dbeta == a.alpha);
        if (a.N <= kSmallBackwardTokens &&
            (!a.dalpha || few || a.N <= SmallBackwardCfg::G || a.N > one_workgroup_groups(rows) * TwelveCfg<M>::G))
            return launch_backward<SmallBackwardCfg>(a.dy, a.x, a.alpha, a.dx, a.dalpha, a.dbeta, a.N, a.workspace, a.stream);
    }
    if (backward_keeps(a.dalpha != nullptr, bytes))
        return launch_backward<TwelveCfg<M, true>>(a.dy, a.x, a.alpha, a.dx, a.dalpha, a.dbeta, a.N, a.workspace, a.stream);
    return launch_backward<TwelveCfg<M>>(a.dy, a.x, a.alpha, a.dx, a.dalpha, a.dbeta, a.N, a.workspace, a.stream);
}

static int dispatch_twelve(int logd, Op op, Args& a) {
    switch (logd) {
#if WHT_ALL_WIDTHS
    case 11: return run_twelve<7>(op, a);
#endif
    case 10: return run_twelve<6>(op, a);
    case 12: return run_twelve<8>(op, a);
    case 14: return run_twelve<10>(op, a);
    case 13: return run_twelve<9>(op, a);
    default: return WHT_ERR_BAD_DIM;
    }
}

static int dispatch(Width w, int dtype, Op op, Args& a) {
    if (w.twelve) return dispatch_twelve(w.logd, op, a);
    return dtype == WHT_DTYPE_F32 ? dispatch_d<IoF32>(w.logd, op, a) : dispatch_d<IoBF16>(w.logd, op, a);
}

// ------------------------------------------------------------------------------------------------
// Partial-sum scratch that lives in the library's own code object, for wht_affine_backward_static:
// callers that cannot allocate pass no workspace.  Every GPU the library runs on holds its own copy
// of the array, at its own address, until the process ends.  In host code the array's name is only a
// handle for hipGetSymbolAddress: what kernels and copies take is the device address it returns.
static __device__ __align__(256) unsigned char scratch[WHT_STATIC_WORKSPACE_BYTES];

constexpr int kMaxDevices = 64;
static std::mutex scratch_mutex;
static void* scratch_address[kMaxDevices];       // per device, filled on the first call there

// Device address of the current device's copy of `scratch`, or nullptr if it cannot be had.
static void* static_scratch() {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return nullptr;
    std::lock_guard<std::mutex> lock(scratch_mutex);
    if (!scratch_address[dev]) {
        void* ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess) {
            (void)hipGetLastError();
            return nullptr;
        }
        scratch_address[dev] = ptr;
    }
    return scratch_address[dev];
}

}  // namespace wht

// ------------------------------------------------------------------------------------------------
// C ABI

extern "C" {

static int forward_common(const void* x, const float* alpha, const float* beta, const void* resid,
                          bool with_resid, void* y, float* sumsq, bool with_stats, int64_t N, int32_t d,
                          int32_t dtype, void* stream) {
    using namespace wht;
    Width w{};
    if (int rc = validate_forward(x, alpha, beta, resid, with_resid, y, sumsq, with_stats, N, d, dtype, &w)) return rc;
    if (N == 0) return WHT_OK;
    Args a{};
    a.x = x; a.alpha = alpha; a.beta = beta; a.resid = with_resid ? resid : nullptr; a.y = y; a.N = N;
    a.sumsq = with_stats ? sumsq : nullptr;
    a.stream = static_cast<hipStream_t>(stream);
    return dispatch(w, dtype, Op::Forward, a);
}

int wht_affine_forward(const void* x, const float* alpha, const float* beta, void* y, int64_t N,
                       int32_t d, int32_t dtype, void* stream) {
    return forward_common(x, alpha, beta, nullptr, false, y, nullptr, false, N, d, dtype, stream);
}

int wht_affine_forward_residual(const void* x, const float* alpha, const float* beta, const void* resid,
                                void* y, int64_t N, int32_t d, int32_t dtype, void* stream) {
    return forward_common(x, alpha, beta, resid, true, y, nullptr, false, N, d, dtype, stream);
}

int wht_affine_forward_residual_stats(const void* x, const float* alpha, const float* beta,
                                      const void* resid, void* y, float* sumsq, int64_t N, int32_t d,
                                      int32_t dtype, void* stream) {
    return forward_common(x, alpha, beta, resid, true, y, sumsq, true, N, d, dtype, stream);
}

size_t wht_affine_backward_workspace_bytes(int64_t N, int32_t d, int32_t dtype) {
    using namespace wht;
    Width w{};
    if (check_dims(N, d, dtype, &w) != WHT_OK || N == 0) return 0;
    Args a{};
    a.N = N;
    dispatch(w, dtype, Op::Workspace, a);
    return a.workspace_out;
}

// Both backward entry points: `own_scratch` takes the partial-sum workspace from the library's
// static buffer instead of the caller.
static int backward_common(const void* dy, const void* x, const float* alpha, void* dx, float* dalpha,
                           float* dbeta, int64_t N, int32_t d, int32_t dtype, void* workspace,
                           size_t workspace_bytes, bool own_scratch, void* stream) {
    using namespace wht;
    const bool grads = dalpha != nullptr || dbeta != nullptr;
    Width w{};
    if (int rc = validate_backward(dy, x, alpha, dx, dalpha, dbeta, N, d, dtype, &w)) return rc;
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (N == 0) {
        if (!grads) return WHT_OK;
        hipLaunchKernelGGL(zero_kernel, dim3((d + 255) / 256), dim3(256), 0, s, dalpha, dbeta, d);
        return hipGetLastError() == hipSuccess ? WHT_OK : WHT_ERR_LAUNCH;
    }
    if (grads) {
        const size_t need = wht_affine_backward_workspace_bytes(N, d, dtype);
        if (own_scratch) {
            if (need > (size_t)WHT_STATIC_WORKSPACE_BYTES) return WHT_ERR_WORKSPACE;
            workspace = static_scratch();
            if (!workspace) return WHT_ERR_LAUNCH;
        } else {
            if (int rc = validate_workspace(workspace, workspace_bytes, need)) return rc;
        }
    }
    Args a{};
    a.dy = dy; a.x = x; a.alpha = alpha; a.dx = dx; a.dalpha = dalpha; a.dbeta = dbeta; a.N = N;
    a.workspace = workspace; a.stream = s;
    return dispatch(w, dtype, Op::Backward, a);
}

int wht_affine_backward(const void* dy, const void* x, const float* alpha, void* dx, float* dalpha,
                        float* dbeta, int64_t N, int32_t d, int32_t dtype, void* workspace,
                        size_t workspace_bytes, void* stream) {
    return backward_common(dy, x, alpha, dx, dalpha, dbeta, N, d, dtype, workspace, workspace_bytes, false, stream);
}

int wht_affine_backward_static(const void* dy, const void* x, const float* alpha, void* dx, float* dalpha,
                               float* dbeta, int64_t N, int32_t d, int32_t dtype, void* stream) {
    return backward_common(dy, x, alpha, dx, dalpha, dbeta, N, d, dtype, nullptr, 0, true, stream);
}

const char* wht_affine_status_string(int status) {
    switch (status) {
    case WHT_OK:             return "ok";
    case WHT_ERR_NULL_PTR:   return "a required pointer is NULL";
    case WHT_ERR_BAD_DIM:    return "d must be a power of two in [WHT_MIN_D, WHT_MAX_D] (WHT_MAX_D_F32 for float32) or, for bfloat16, 12*2^m in [WHT_MIN_D_TWELVE, WHT_MAX_D_TWELVE]; N >= 0";
    case WHT_ERR_BAD_DTYPE:  return "dtype must be WHT_DTYPE_F32 or WHT_DTYPE_BF16";
    case WHT_ERR_MISALIGNED: return "tensor pointers must be 16-byte aligned";
    case WHT_ERR_WORKSPACE:  return "workspace is NULL or smaller than wht_affine_backward_workspace_bytes (wht_affine_backward_static: the call needs more than WHT_STATIC_WORKSPACE_BYTES)";
    case WHT_ERR_LAUNCH:     return "the HIP runtime refused a kernel launch";
    default:                 return "unknown status";
    }
}

int wht_affine_version(void) { return 100; }

}  // extern "C"
