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

// Forward calls by the size of x in bytes.  Few tokens (decoding, short prefills): one token group per workgroup and no
// token loop (forward_once_kernel), with plain stores up to `through`, through L2 from there on, and from `pair` on with
// two token groups per workgroup, both requested at once: alpha and beta, two to four times as many bytes as a thread's
// part of x, are then read half as often.  From `limit` on the persistent kernel.
// What each is worth, us per call under graph replay, three sets of inputs and two of outputs in turn / everything from memory:
//   plain against through: 4097 x 1024 4.53 / 5.41 and 4.02 / 5.04, 1024 x 4096 4.68 / 5.66 and 3.74 / 4.75, 16385 x 256 4.36 / 5.46
//     and 3.62 / 5.53; one token of 4096 with the statistic 2.65 and 2.77 (the kernel ends when memory, not L2, has the results);
//   one group against two, 2048 wide: 1025 tokens 3.05 / 3.86 and 3.03 / 3.76, 4097 6.9 / 9.8 and 6.3 / 8.0; 8 MiB of 1536 wide
//     7.0 / 7.7 and 5.6 / 6.3, of 12288 wide 10.6 / 11.4 and 7.9 / 8.8 (there the persistent kernel took over from 2^22 elements on);
//     below, half the workgroups leave CUs idle: 1 MiB of 2048 wide 2.8 and 3.2;
//   persistent against one pass: 32 MiB of 256 wide (bfloat16) 13.4 / 14.4 and 11.1 / 14.4, of 2048 13.1 / 15.3 and 11.4 / 18.0 (so 24 there), 8 MiB
//     of 16384 9.9 / 10.8 and 6.0 / 8.6, 32 MiB of 1536 11.5 / 13.5 and 14.2 / 15.3; with the residual 25 MiB of 1024 14.6 / 14.7 and 12.5 /
//     14.6, 29 of 2048 17.5 / 17.5 and 14.8 / 19.1, of float32 2048 17.0 / 17.4 and 14.2 / 17.5 (so 33 there);
//   two groups with the statistic, 2048 wide: 18 MiB 10.9 / 14.0, one 10.3 / 13.8, so one.
// Rows of 12 * 2^m elements have workgroups of one token (two of 768): workgroups of 256 threads, with up to eight tokens,
// leave CUs without any, and from 257 of them on put two on one CU beside others with one (341 x 768 3.33 / 2.34, 1365 x
// 1536 5.60 / 4.80, 683 x 3072 6.01 / 4.83).
// The kernels do the same arithmetic on a token in the same order, so the switches are invisible in y
// (the norm statistic is summed in the order of the launch shape: its last bits may differ).
struct OnceSizes { int64_t through, pair, limit; };
template <class C>
constexpr OnceSizes once_sizes(bool resid, bool stats) {
    constexpr int64_t MiB = 1 << 20, none = INT64_MAX;
    const int64_t through = stats ? 5 * MiB / 2 : MiB;
    if constexpr (C::kTwelve) {
        switch (C::m) {
        case 6:  return {through, resid ? 5 * MiB : 7 * MiB, 22 * MiB};
        case 7:  return {resid ? 7 * MiB / 2 : 5 * MiB / 2, resid ? 7 * MiB / 2 : 5 * MiB / 2, resid ? 22 * MiB : 17 * MiB};
        case 8:  return {through, stats ? 3 * MiB : 2 * MiB, resid ? 14 * MiB : 17 * MiB};
        case 9:  return {resid ? 7 * MiB / 2 : MiB, 7 * MiB / 2, stats ? 7 * MiB : resid ? 12 * MiB : 17 * MiB};
        default: return {4 * MiB, 7 * MiB, 34 * MiB};
        }
    } else if constexpr (C::kWave) {
        const int64_t from = resid && C::v == 2 && C::n <= 10 ? 6 * MiB : through;
        if (C::v == 3 || C::n <= 10) return {from, none, (resid ? 33 : 48) * MiB};
        return {from, none, (C::n == 11 ? (resid ? 33 : 20) : C::n == 12 || resid ? 17 : 9) * MiB};
    } else {
        switch (C::n) {
        case 10: return {through, resid ? none : 5 * MiB / 2, (resid ? 33 : 24) * MiB};
        case 11: return {through, stats ? none : resid ? 7 * MiB : 7 * MiB / 2, (resid ? 33 : 24) * MiB};
        case 12: return {through, resid ? 7 * MiB : 10 * MiB, (stats ? 9 : 17) * MiB};
        case 13: return {through, none, (resid ? 7 : 13) * MiB};
        default: return {4 * MiB, none, 24 * MiB};
        }
    }
}

// Whether the persistent forward kernels and the backward kernels write y and dx through L2 rather than streaming them
// past the caches ("nt").  Written through, results stay in the Infinity Cache: the next kernel finds them there, and a
// program that gets the same output buffers back overwrites them there.  us per call, streamed / through, everything from
// memory: 32768 x 1024 forward 24.5 / 24.1, backward 39.4 / 38.6; forward, forward on its result with the residual and backward, 32 MiB
// each, 47.5 / 43.1, 128 MiB each 182 / 172; with two sets of outputs in turn forward 32768 x 2048 44.1 / 40.6, a step of
// 32768 x 1024 64.4 / 59.3.  Above 136 MiB the three kinds of stream no longer fit together and streaming is ahead
// (backward of 32768 x 8192 276 / 281, a step of 16384 x 4096 float32 231 / 236).  Where a workgroup of the persistent forward
// has few rounds, each waits for the stores of the one before it, and those come back from memory, not L2: forward of 16 MiB of
// 8192 wide 8.6 / 9.3, of 32 MiB of 16384 wide 17.0 / 18.0, dx alone of 16 MiB of 2048 wide 7.6 / 8.5.
// Rows of 12 * 2^m: where x or dy is read with the default policy (kKeep) dx always and y never, elsewhere by the limits at
// run_twelve.
template <class C>
static bool write_through(int64_t N, bool backward, bool grads) {
    constexpr int64_t MiB = 1 << 20;
    const int64_t bytes = N * C::kRow * (int64_t)sizeof(typename C::io::elem_t);
    if constexpr (C::kTwelve)
        return C::kKeep ? backward : bytes <= 136 * MiB && (!backward || (C::m < 10 && (bytes < 56 * MiB || bytes >= 80 * MiB)));
    if (!backward && bytes < (C::n >= 13 ? 56 : 24) * MiB) return false;
    if (backward && !grads && (C::n == 14 ? bytes < 56 * MiB : bytes >= 12 * MiB && bytes < 24 * MiB)) return false;
    return bytes <= 136 * MiB;
}
// f(false type or true type): a choice made at run time as a template argument.
template <class F>
static void with_bool(bool b, F&& f) {
    if (b) f(std::true_type{});
    else f(std::false_type{});
}

template <class C, bool THROUGH, int R>
static int launch_forward_once(const void* x, const float* alpha, const float* beta, const void* resid,
                               void* y, float* sumsq, int64_t N, hipStream_t stream) {
    using T = typename C::io::elem_t;
    const int grid = (int)((N + C::G * R - 1) / (C::G * R));
    auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(grid), dim3(C::BT), 0, stream, static_cast<const T*>(x), alpha, beta,
                           static_cast<const T*>(resid), static_cast<T*>(y), sumsq, N);
    };
    if (resid && sumsq) launch(forward_once_kernel<C, true, true, THROUGH, R>);
    else if (resid) launch(forward_once_kernel<C, true, false, THROUGH, R>);
    else launch(forward_once_kernel<C, false, false, THROUGH, R>);
    return hipGetLastError() == hipSuccess ? WHT_OK : WHT_ERR_LAUNCH;
}

template <class C>
static int launch_forward(const void* x, const float* alpha, const float* beta, const void* resid, void* y,
                          float* sumsq, int64_t N, hipStream_t stream) {
    using T = typename C::io::elem_t;
    const int grid = grid_for<C>(N, false);
    const int cluster = forward_cluster<C>(N, grid, resid != nullptr);
    auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(grid), dim3(C::BT), 0, stream, static_cast<const T*>(x), alpha, beta,
                           static_cast<const T*>(resid), static_cast<T*>(y), sumsq, N, cluster);
    };
    with_bool(write_through<C>(N, false, false), [&](auto b) {
        constexpr bool THROUGH = !(C::kTwelve && C::kKeep) && decltype(b)::value;
        if (resid && sumsq) launch(forward_kernel<C, true, true, THROUGH>);
        else if (resid) launch(forward_kernel<C, true, false, THROUGH>);
        else launch(forward_kernel<C, false, false, THROUGH>);
    });
    return hipGetLastError() == hipSuccess ? WHT_OK : WHT_ERR_LAUNCH;
}

template <class CF, class CO>
static int forward(const Args& a) {
    const int64_t bytes = a.N * CO::kRow * (int64_t)sizeof(typename CO::io::elem_t);
    const OnceSizes at = once_sizes<CO>(a.resid != nullptr, a.sumsq != nullptr);
    if (bytes >= at.limit) return launch_forward<CF>(a.x, a.alpha, a.beta, a.resid, a.y, a.sumsq, a.N, a.stream);
    if constexpr (CO::kMfma && once_sizes<CO>(false, false).pair < INT64_MAX)
        if (bytes >= at.pair)
            return launch_forward_once<CO, true, 2>(a.x, a.alpha, a.beta, a.resid, a.y, a.sumsq, a.N, a.stream);
    if (bytes >= at.through)
        return launch_forward_once<CO, true, 1>(a.x, a.alpha, a.beta, a.resid, a.y, a.sumsq, a.N, a.stream);
    return launch_forward_once<CO, false, 1>(a.x, a.alpha, a.beta, a.resid, a.y, a.sumsq, a.N, a.stream);
}

// Rows that backward_few_kernel does not take (shorter than 8 slices, float32 4): a call of up to three token groups runs on one
// workgroup, which writes dalpha and dbeta itself: no partial rows and no second launch, which costs the stream
// 2.5 us and the host 3.3.  The groups then run one after the other; up to here that is no slower (us per call under graph
// replay, two launches / one: 3 groups at d = 256 6.0 / 5.7).
template <class C>
static bool one_workgroup(int64_t N) { return N <= 3 * (int64_t)C::G; }

// A call of few elements runs on backward_few_kernel: no partial rows and no second launch, which cost the stream 2.5 us and
// the host 3.3, and a workgroup for every 64 columns where one_workgroup has a single one.  Rows must have 8 slices of 64
// columns (float32: 4).  Its workgroups read x and dy while others write dx: where dx lies over one of them, dx is a launch of its own, and a call that
// writes dalpha or dbeta over alpha stays on the other kernels.
// us per call under graph replay, before / this kernel, backward: 1 x 512 3.8 / 2.2, 64 x 512 6.1 / 3.4, 64 x 1024 5.7 / 3.9 (91: 5.8 /
// 5.9), 60 x 1536 7.5 / 4.6 (85: 7.6 / 7.1), 16 x 4096 6.3 / 3.1, 32 6.3 / 4.3 (45: 6.4 / 5.5, from memory 6.9 / 7.2), 16 x 8192 6.7 / 4.4 (23: 6.8 / 5.3,
// from memory 7.2 / 6.8), 12 x 16384 12.0 / 9.4 (16: 12.1 / 10.5), 64 x 768 6.5 / 3.9 (121: 6.5 / 6.0), 16 x 12288 12.2 / 5.8; float32
// 64 x 512 6.3 / 3.7 (128: 6.4 / 5.6), 64 x 1024 6.1 / 4.5, 32 x 2048 8.0 / 4.0 (64: 8.0 / 6.1), 12 x 8192 8.9 / 5.1 (16: 9.0 / 6.0).
template <class C>
constexpr bool has_few_backward() {
    if (C::kTwelve) return C::kKeep && (C::kRow > 768 || C::BT == 128);         // what calls of so few elements run on
    return C::kRow % 64 == 0 && C::kRow / 64 >= 16 / (int)sizeof(typename C::io::elem_t);
}
template <class C>
constexpr int64_t few_backward_elements() {
    if (sizeof(typename C::io::elem_t) == 4) return C::kRow <= 512 ? 3 << 14 : C::kRow == 1024 ? 1 << 16 : 3 << 15;
    return C::kRow <= 1024 ? 1 << 16 : C::kRow < 2048 ? 3 << 15 : C::kRow < 12288 ? 1 << 17 : 3 << 16;
}

template <class C>
static int launch_backward(const void* dy, const void* x, const float* alpha, void* dx, float* dalpha,
                           float* dbeta, int64_t N, void* workspace, hipStream_t stream) {
    using T = typename C::io::elem_t;
    const bool grads = dalpha != nullptr;
    if constexpr (has_few_backward<C>())
        if (grads && N * C::kRow <= few_backward_elements<C>() && dalpha != alpha && dbeta != alpha) {
            const bool apart = dx && (dx == dy || dx == x);
            const int64_t groups = dx && !apart ? (N + C::G - 1) / C::G : 0;
            hipLaunchKernelGGL(backward_few_kernel<C>, dim3((unsigned)(FewSlices<C>::A + groups)), dim3(kFewThreads), 0, stream,
                               static_cast<const T*>(dy), static_cast<const T*>(x), alpha, static_cast<T*>(dx), dalpha, dbeta, N);
            if (hipGetLastError() != hipSuccess) return WHT_ERR_LAUNCH;
            return apart ? launch_backward<C>(dy, nullptr, alpha, dx, nullptr, nullptr, N, nullptr, stream) : WHT_OK;
        }
    const bool direct = !has_few_backward<C>() && grads && one_workgroup<C>(N);
    const int grid = direct ? 1 : grid_for<C>(N, grads);      // dx alone streams like a forward pass
    float* ws = static_cast<float*>(workspace);
    const SumRows sums = direct ? SumRows{dalpha, dbeta, 0} : SumRows{ws, ws + C::kRow, 2 * C::kRow};

    auto launch = [&](auto kernel, int threads) {
        hipLaunchKernelGGL(kernel, dim3(grid), dim3(threads), 0, stream, static_cast<const T*>(dy), static_cast<const T*>(x),
                           alpha, static_cast<T*>(dx), sums, N);
    };
    with_bool(write_through<C>(N, true, grads), [&](auto b) {
        constexpr bool THROUGH = (C::kTwelve && C::kKeep) || decltype(b)::value;
        if constexpr (C::kWave) {
            if (grads && dx) launch(backward_wave_kernel<C, true, true, THROUGH>, C::BT);
            else if (!grads) launch(backward_wave_kernel<C, false, true, THROUGH>, C::BT);
            else launch(backward_wave_kernel<C, true, false, false>, C::BT);
        } else if (grads && dx) {
            if constexpr (C::kBwdTeams) launch(backward_teams_kernel<C, THROUGH>, 3 * C::BT);
            else launch(backward_kernel<C, true, true, THROUGH>, C::BT);
        } else if (!grads) launch(backward_kernel<C, false, true, THROUGH>, C::BT);
        else launch(backward_kernel<C, true, false, false>, C::BT);
    });
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
// Small tensors are read with the default cache policy, as these rows always have been, larger ones streamed: x of a forward
// call below 80 MiB (with the residual, 48 MiB up to m = 8 and 56 above), x and dy of a backward call up to 32 MiB, dy where dx
// is made alone up to 128.  What has been read with the default policy stays in the Infinity Cache: a backward call that
// follows its forward call finds x there, and a caller that comes back to the same small tensors finds them.
// y is streamed where x is kept (through L2, y and dx would push x out before the backward call reads it) and goes through
// L2 where x is streamed, both up to 136 MiB.  us per call, kept and streamed y / streamed x and y through, three sets of
// inputs in turn and inputs from memory:
//     forward     64 MiB of 768 22.0 / 23.5 and 26.2 / 23.6, 96 36.7 / 32.3 and 36.7 / 32.4, 128 47.6 / 41.5; 96 of 3072 38.4 / 34.1, of 12288 43.0 / 40.5;
//     residual    40 MiB of 768 21.6 / 22.5 and 25.8 / 22.6, 48 26.9 / 25.6 and 29.9 / 25.6, 128 72.3 / 60.2; 48 of 6144 27.8 / 28.8 and 30.6 / 29.4,
//                 64 39.4 / 35.1; 64 of 12288 41.8 / 39.7.
// dx of a backward call above 32 MiB goes through L2 up to 136 MiB but for 56 to 80 MiB, where x, y, dy and dx of a step just
// fill the Infinity Cache, and for m = 10.  us per call, streamed / through, backward and a step: 48 MiB of 768 32.6 / 31.4 and
// 48.6 / 48.7 (from memory 50.2 / 49.4), 64 41.6 / 39.4 and 62.9 / 63.5, 128 73.8 / 67.9 and 112.2 / 110.6; 48 of 6144 36.2 / 34.8 and 54.7 / 53.9,
// 128 of 1536 75.0 / 68.5 and 121.6 / 111.3; 48 of 12288 47.1 / 44.1 and 67.5 / 69.6.
// The 32 MiB: backward, default policy / streamed, three sets of buffers in turn and inputs from memory (rows padded to
// 16 * 2^m, before: always default):
//     10923 x 768    16.0 / 17.9   18.1 / 18.4   (16.9, 18.0)        1365 x 6144    18.5 / 22.0   20.3 / 22.3   (19.4, 21.3)
//     16384 x 768    19.2 / 21.3   21.8 / 21.7   (21.0, 22.5)        2048 x 6144    21.9 / 25.4   23.5 / 25.7   (23.9, 25.3)
//     8192 x 1536    19.8 / 22.7   22.5 / 22.9   (22.8, 23.9)        683 x 12288    25.3 / 31.1   26.4 / 31.4   (39.5, 41.6)
//     2731 x 3072    16.9 / 18.3   19.7 / 18.7   (18.9, 20.3)        1365 x 12288   35.7 / 39.7   37.3 / 40.8   (56.1, 56.6)
//     5461 x 3072    24.6 / 26.0   27.0 / 26.0   (28.3, 28.6)
// So the default policy costs up to 5 % from memory at 768 and 3072 and gains more elsewhere; streamed, calls of 6144 and
// 768 would be slower than before.  The power-of-two rows have always been streamed and lose by a change.
// Backward, rows of 768, up to 512 tokens: workgroups of 128 threads (four tokens), so that twice as many share a call
// that has few.  us per call under graph replay, 256 / 128 threads, inputs that come back: 341 7.00 / 6.63, 512 7.09 / 6.99, 683 7.26 /
// 7.31, 1365 8.22 / 9.87; dx alone 64 3.26 / 2.84, 512 3.33 / 2.95, 1365 3.51 / 3.77.
constexpr int64_t kSmallBackwardTokens = 512;
using SmallBackwardCfg = TwelveCfg<6, true, 128>;

template <int M>
static int run_twelve(Op op, Args& a) {
    const int64_t elems = a.N * TwelveCfg<M>::kRow, bytes = 2 * elems;
    if (op == Op::Forward) {
        if (bytes < (int64_t(!a.resid ? 80 : M <= 8 ? 48 : 56) << 20)) return forward<TwelveCfg<M, true>, TwelveCfg<M, false, 64>>(a);
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
        // Up to two token groups of 256 threads the workspace has a row for each of those and none for groups of four tokens:
        // a call that backward_few_kernel declines there runs on one workgroup of 256 threads, without partial rows.
        const bool over_alpha = a.dalpha && (a.dalpha == a.alpha || a.dbeta == a.alpha);
        if (a.N <= kSmallBackwardTokens && !(over_alpha && a.N <= 2 * TwelveCfg<M>::G))
            return launch_backward<SmallBackwardCfg>(a.dy, a.x, a.alpha, a.dx, a.dalpha, a.dbeta, a.N, a.workspace, a.stream);
    }
    if (bytes <= (int64_t(a.dalpha ? 32 : 128) << 20))             // dx alone reads dy only
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
