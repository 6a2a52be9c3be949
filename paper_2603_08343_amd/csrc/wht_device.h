// Device code of the Walsh-Hadamard output layer  y = alpha (.) (H x) + beta  (paper Sec. 4.1,
// Eq. 1) for gfx950: the per-token transform H_raw x (Fig. 2's butterfly stages, scheduled by
// wht_plan.h), the fused affine epilogue, the backward pass with z recomputed, and the fixed-order
// reduction of dalpha / dbeta.  1/sqrt(d) is folded into alpha.  Two schedules share the kernels:
//   - wave schedule (float32 I/O, and bfloat16 below d = 1024): every stage is additions, in registers
//     or between the lanes of one wave; float32 tokens above 2048 elements take two or four waves and
//     one LDS exchange;
//   - matrix-core schedule (bfloat16 I/O, d >= 1024): ten of the log2(d) stages run as two rounds
//     of 32x32 +-1 products on the MFMA unit (exact products, float32 accumulation), the rest as
//     register butterflies plus one LDS exchange across the waves of a token.
// Widths d = 12 * 2^m (bfloat16, d >= 768; the paper's Table 2 trains d = 768 and 1536 and leaves the
// matrix undefined there) use H_raw = P12 (x) S_{2^m}, P12 a symmetric order-12 Hadamard matrix: a
// matrix-core schedule of their own, with P12 inside the second round's +-1 matrix (see TwelveCfg).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <type_traits>

#include "wht_plan.h"
#include "wht_route.h"

namespace wht {

// ------------------------------------------------------------------------------------------------
// small helpers

template <int I, int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        static_for<I + 1, N>(f);
    }
}

// Cache-policy operands of loads and stores:
//   kStreamPolicy   "nt": read or written once, retained nowhere;
//   kThroughPolicy  "sc1" (device scope): a store passes through L2 at once instead of lying there dirty until the end of
//                   the kernel writes it back, and stays in the Infinity Cache for the kernel that reads it.
constexpr int kStreamPolicy = 2, kThroughPolicy = 16;

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// Stores through L2 go through a buffer resource: the compiler has no other 16-byte store with a device scope.  Its base is
// the same for a wave, a lane's part of the address is 32 bits, and what lies past its end is dropped.
typedef __amdgpu_buffer_rsrc_t rsrc_t;
__device__ __forceinline__ rsrc_t make_rsrc(const void* base, unsigned bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, bytes, 0x00027000);
}
__device__ __forceinline__ void store16_through(rsrc_t to, unsigned offset, const uint4& q) {
    const u32x4 v = {q.x, q.y, q.z, q.w};
    __builtin_amdgcn_raw_buffer_store_b128(v, to, offset, 0, kThroughPolicy);
}
__device__ __forceinline__ void stream_store16(void* p, const uint4& q) {
    const u32x4 v = {q.x, q.y, q.z, q.w};
    __builtin_nontemporal_store(v, static_cast<u32x4*>(p));
}
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

// I/O element traits: how one 16-byte global vector maps to float32 registers.
struct IoF32 {
    using elem_t = float;
    static constexpr int kLogVec = 2;   // 4 elements per 16 bytes
    static __device__ __forceinline__ void unpack(const uint4& raw, float* out) {
        out[0] = __uint_as_float(raw.x); out[1] = __uint_as_float(raw.y);
        out[2] = __uint_as_float(raw.z); out[3] = __uint_as_float(raw.w);
    }
    static __device__ __forceinline__ uint4 pack(const float* in) {
        return make_uint4(__float_as_uint(in[0]), __float_as_uint(in[1]),
                          __float_as_uint(in[2]), __float_as_uint(in[3]));
    }
};

struct IoBF16 {
    using elem_t = uint16_t;
    static constexpr int kLogVec = 3;   // 8 elements per 16 bytes
    // bfloat16 is the upper half of binary32: widening is a shift / a mask
    static __device__ __forceinline__ void unpack(const uint4& raw, float* out) {
        const uint32_t w[4] = {raw.x, raw.y, raw.z, raw.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            out[2 * i]     = __uint_as_float(w[i] << 16);
            out[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
        }
    }
    // round to nearest even (the hardware's packed float32 -> bfloat16 convert)
    static __device__ __forceinline__ uint32_t pack2(float lo, float hi) {
        f32x2 f = {lo, hi};
        bf16x2 b = __builtin_convertvector(f, bf16x2);
        return __builtin_bit_cast(uint32_t, b);
    }
    static __device__ __forceinline__ uint4 pack(const float* in) {
        return make_uint4(pack2(in[0], in[1]), pack2(in[2], in[3]),
                          pack2(in[4], in[5]), pack2(in[6], in[7]));
    }
};

// ------------------------------------------------------------------------------------------------
// per-(d, dtype) configuration

// Matrix-core schedule (bfloat16 I/O, d >= 1024): 2^LOGT MFMA tiles of 1024 elements per wave.
template <int LOGD, int LOGT>
struct MfmaCfg {
    using io = IoBF16;
    static constexpr bool kMfma = true, kWave = false, kTwelve = false;
    static constexpr int kPair = 1;             // tokens per slot
    static constexpr int kSums = 1 << (4 + LOGT);                   // column sums per thread
    static constexpr bool kKeep = false;        // see TwelveCfg
    static constexpr int n = LOGD, t = LOGT, e = 4 + LOGT, v = 3;
    static constexpr int w = n - 10 - t;        // log2(waves per token)
    static_assert(n >= 10 && w >= 0 && w <= 2 * (1 + t) && e <= kMaxRegBits, "bad tile");
    static constexpr PlanDesc plan = make_mfma_plan(n, t);
    static_assert(plan_is_complete(plan), "every stage must run exactly once");
    static_assert(plan_keeps_vectors(plan), "16 bytes per LDS access");
    static constexpr int P = plan.nphase;
    static constexpr int D = 1 << n;
    static constexpr int E = 1 << e;
    static constexpr int V = 8;
    static constexpr int NV = E / V;
    static constexpr int T = 1 << t;            // MFMA tiles per wave
    static constexpr int TPT = 1 << (n - e);
    static_assert(TPT >= 64, "a token occupies whole waves");
    static constexpr int BT = TPT > 256 ? TPT : 256;
    static constexpr int G = BT / TPT;
    // persistent-grid size in workgroups per CU (measured optima at N = 32768 tokens: more
    // workgroups than this only add concurrent streams to the memory system)
    static constexpr int kFwdGroupsPerCU = 2;
    // the full backward of a schedule with one LDS exchange runs on three teams of waves
    // (backward_teams_kernel), one workgroup per CU
    static constexpr bool kBwdTeams = plan.nphase == 2 && 3 * BT <= 1024;
    static constexpr int kBwdGroupsPerCU = kBwdTeams || n == 11 || n >= 13 ? 1 : 2;
    static constexpr int kBwdWavesPerSimd = 1;
    // Forward: workgroups per cluster (0 = one interleave over the whole grid).  With every
    // workgroup in one moving window of rows, the read stream and the write stream keep a fixed
    // address distance, and for about 40 % of the distances y - x (period 128 MiB, and again 512 KiB)
    // the kernel runs 8..29 % slower at d >= 4096 -- DRAM bank conflicts between the two streams.
    // Four windows spread over the tensor take the worst case from +29 % to +11 % and improve the
    // mean over all distances, for +1.5 % in the best case.  Rows of 4 KiB and less show no such
    // dependence and keep the plain interleave.
    static constexpr int kFwdCluster = n >= 12 ? 128 : 0;
    // with the residual as a third stream two windows measured best (mean 263 us against 274 us
    // with four and 268 us with one, d = 8192)
    static constexpr int kFwdClusterResid = n >= 12 ? 256 : 0;
    static constexpr int kRow = D;
    static constexpr unsigned phys(unsigned i) { return lds_phys_rot(i); }
    // LDS word of registers I .. I+3 relative to the thread's own offset, in the layout of phase PH
    template <int PH> static constexpr unsigned lds_reg(int I) { return phys(reg_elem_offset(plan.ph[PH], e, I)); }
    static constexpr unsigned kTokenWords = D;
    static constexpr unsigned kExchangeBytes = (P > 1 || G > 1) ? G * kTokenWords * 4u : 16u;
    static constexpr unsigned kStageBytes = BT * NV * 16u;          // one tensor's token group, as stored
    static constexpr unsigned kLdsBytes = kExchangeBytes + kStageBytes;              // forward
    static constexpr unsigned kLdsBytesBackward = kExchangeBytes + 2u * kStageBytes; // x and dy
    static_assert(kLdsBytesBackward <= 160u * 1024u, "token group does not fit LDS");
};

// Rows of 12 * 2^LOGM elements (bfloat16): the matrix-core rounds of wht_plan.h, 24 values per lane and no lane,
// vector or 128-byte line in part.  It took the place of the power-of-two schedule on rows padded to 16 * 2^m, in
// which a quarter of the lanes sat out every load and store and every instruction worked on a quarter of zeros: the
// large calls were bound by instruction issue there (75 % of the vector slots at 6144) and are bound by memory
// (forward) or nearly so here.  us per call, before / after: forward 32768 x 6144 153 / 137 (5.9 TB/s; a copy in
// this layout 130), backward 262 / 229 (5.3 TB/s), a step of 32768 x 768 56.4 / 48.6, of 32768 x 1536 100 / 88,
// backward of 16384 x 12288 358 / 256 (one exchange per transform instead of two).  What is slower than
// on padded rows: the backward pass of up to 341 tokens of 6144 (64 tokens 8.4 / 8.9; 24 values per lane in dependent
// rounds with nothing else on the CU), forward calls of some sizes by up to 5 %.
// LEAST: threads of a workgroup, where a token (two of 768) takes fewer.
// KEEP: x and dy are read with the default cache policy and so stay in the Infinity Cache (see run_twelve).
template <int LOGM, bool KEEP = false, int LEAST = 256>
struct TwelveCfg {
    using io = IoBF16;
    static constexpr bool kMfma = true, kWave = false, kTwelve = true, kKeep = KEEP;
    static constexpr int m = LOGM, n = m + 4, v = 3, w = twelve_wave_bits(m);
    static_assert(m >= 6 && w <= 3, "three lane positions take wave bits");
    static constexpr int P = w > 0 ? 2 : 1;     // layouts: the second one only after an exchange
    static constexpr int V = 8, NV = 3, E = NV * V;
    static constexpr int TPT = 64 << w;         // threads per token (per two tokens of 768)
    static constexpr int kPair = m == 6 ? 2 : 1;                    // tokens per wave
    static constexpr int kSums = E - (kPair - 1) * V;               // column sums per thread: vectors 0 and 1 in one
    static constexpr int BT = TPT > LEAST ? TPT : LEAST;
    static constexpr int G = BT / TPT * kPair;
    static constexpr int kRow = 12 << m, D = kRow;
    static constexpr int kFwdGroupsPerCU = 2;
    static constexpr bool kBwdTeams = P == 2 && 3 * BT <= 1024;
    // two workgroups per CU; three and four: forward 32768 x 768 20.7 / 21.9 / 22.3 us, 6144 146 / 152 / 159
    static constexpr int kBwdGroupsPerCU = kBwdTeams || m == 10 ? 1 : 2;
    static constexpr int kBwdWavesPerSimd = m <= 7 ? 2 : 1;
    static constexpr int kFwdCluster = m >= 8 ? 128 : 0, kFwdClusterResid = m >= 8 ? 256 : 0;
    template <int PH> static constexpr unsigned lds_reg(int I) { return twelve_exchange_reg(I, w); }
    static constexpr unsigned phys(unsigned e) { return twelve_column(e, m); }      // column sums
    static constexpr unsigned kExchangeWords = P > 1 ? twelve_exchange_words(w) : 0u;
    static constexpr unsigned kColumnWords = 12u * ((1u << m) + 16u);
    static constexpr unsigned kTokenWords = kExchangeWords < kColumnWords ? kColumnWords : kExchangeWords;
    static constexpr unsigned kExchangeBytes = G / kPair * kTokenWords * 4u;
    static constexpr unsigned kStageBytes = BT * NV * 16u;
    static_assert(kExchangeBytes + 2u * kStageBytes <= 160u * 1024u, "token group does not fit LDS");
};

// Wave schedule: a token inside one wave, every stage in registers or between lanes (or on two or
// four whole waves, with one LDS exchange between them).
template <int LOGD, int LOGE, class Io>
struct WaveCfg {
    using io = Io;
    static constexpr bool kMfma = false, kWave = true, kTwelve = false, kKeep = false;
    static constexpr int kPair = 1, kSums = 1 << LOGE;
    static constexpr int n = LOGD, e = LOGE, v = Io::kLogVec;
    static constexpr int L = n - e < 6 ? n - e : 6, w = n - e - L;    // log2 lanes of a wave, waves per token
    static_assert(wave_fits(n, e, v), "bad tile");
    static constexpr PlanDesc plan = make_wave_plan(n, e, v);
    static_assert(plan_is_complete(plan), "every butterfly stage must run exactly once");
    static_assert(plan_keeps_vectors(plan), "16 bytes per LDS access");
    static constexpr int P = plan.nphase;
    static constexpr int D = 1 << n;
    static constexpr int E = 1 << e;
    static constexpr int V = 1 << v;
    static constexpr int NV = E / V;
    static constexpr int TPT = 1 << (n - e);    // threads per token
    static constexpr int BT = w > 0 ? TPT : 256;        // w = 0: four waves that share nothing but the parameters
    static constexpr int G = BT / TPT;
    // persistent-grid size in workgroups per CU (measured optima at 2^24 ... 2^26 elements): rows so
    // short that a workgroup pass is a few KiB want more of them in flight
    static constexpr int kFwdGroupsPerCU = v == 3 || n <= 6 ? 4 : 2;
    static constexpr int kBwdGroupsPerCU = n <= 6 ? 4 : (w == 2 || (v == 2 && n == 11) ? 1 : 2);
    static constexpr int kBwdWavesPerSimd = w > 0 ? 1 : (e >= 5 ? 2 : 3);   // register budget of the backward
    // windows of the forward walk (see MfmaCfg); mean / worst over twelve distances y - x, 256 MiB each
    // way: d = 4096 92.3 / 107.0 us with one window, 90.6 / 91.4 with four; d = 1024 89.4 / 104.6 and
    // 88.7 / 89.6; d = 8192 92.8 / 94.0 and 92.0 / 92.7 with two; d = 2048 92.2 / 93.6 and 91.8 / 92.6
    static constexpr int kFwdCluster = v == 2 && n >= 10 ? (n == 10 || n == 12 ? 128 : 256) : 0;
    static constexpr int kFwdClusterResid = v == 2 && n >= 10 ? 256 : 0;
    static constexpr int kRow = D;
    static constexpr unsigned phys(unsigned i) { return lds_phys_plain(i); }
    // LDS word of registers I .. I+3 relative to the thread's own offset, in the layout of phase PH
    template <int PH> static constexpr unsigned lds_reg(int I) { return phys(reg_elem_offset(plan.ph[PH], e, I)); }
    static constexpr unsigned kTokenWords = D;
    static constexpr unsigned kExchangeBytes = w > 0 ? G * D * 4u : 16u;
    static constexpr unsigned kStageBytes = BT * NV * 16u;          // one tensor's token group, as stored
    static_assert(G == 1 || 2u * kStageBytes >= G * kTokenWords * 4u, "the token sums reuse the stage buffers");
};

// What the rules of dispatch call a configuration's rows.
template <class C>
constexpr Rows rows_of() {
    if constexpr (C::kTwelve) return {Sched::Twelve, C::m, 2};
    else return {C::kWave ? Sched::Wave : Sched::Matrix, C::n, (int)sizeof(typename C::io::elem_t)};
}

// Workgroup barrier for the LDS exchange.  __syncthreads() carries a release/acquire fence that
// makes the wave wait for *all* its outstanding memory operations -- including the prefetches in
// flight and the stores of the previous token, which have nothing to do with the exchange.  The
// exchange only needs this wave's LDS writes to have completed (lgkmcnt) before the barrier.
__device__ __forceinline__ void exchange_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// Element offset of thread t (within its token) in phase PH.
template <class C, int PH>
__device__ __forceinline__ unsigned thread_elem_offset(unsigned t) {
    if constexpr (C::kWave) t = wave_lane_to_bits(t, C::L);
    unsigned off = 0;
    static_for<0, C::n - C::e>([&](auto k) {
        constexpr int K = decltype(k)::value;
        off |= ((t >> K) & 1u) << C::plan.ph[PH].tb[K];
    });
    return off;
}

// First stage of the reverse order -- element bit and the register-index bit that carries it.
template <class C>
constexpr int wave_first_back_bit() {
    return C::w > 0 ? C::v + 6 : C::L == 6 ? C::v + 5 : C::L == 5 ? C::v + 4 : 0;
}
template <class C>
constexpr int wave_first_back_reg() {
    int q = 0;
    while (C::plan.ph[C::P - 1].rb[q] != wave_first_back_bit<C>()) ++q;
    return q;
}

// Butterfly stages of phase PH, all in registers: (a, b) -> (a + b, a - b) on register pairs.
template <class C, int PH>
__device__ __forceinline__ void run_stages(float (&r)[C::E]) {
    static_for<0, C::e>([&](auto q) {
        constexpr int Q = decltype(q)::value;
        constexpr int bit = C::plan.ph[PH].rb[Q];
        if constexpr ((C::plan.ph[PH].stages >> bit) & 1u) {
            static_for<0, C::E>([&](auto i) {
                constexpr int I = decltype(i)::value;
                if constexpr (!((I >> Q) & 1)) {
                    const float a = r[I], b = r[I | (1 << Q)];
                    r[I] = a + b;
                    r[I | (1 << Q)] = a - b;
                }
            });
        }
    });
}

// Debug build (WHT_POISON_LDS, loaded by one GPU test only): a thread that has read its
// values from an exchange region or from its own stage slot overwrites them with NaN.  A read that
// comes too early -- before the data it is meant to see has been written or has landed, i.e. a
// missing barrier or a missing wait -- then returns NaN instead of last iteration's plausible
// values, and the comparison against the oracle fails loudly.
#ifdef WHT_POISON_LDS
constexpr bool kPoisonLds = true;
#else
constexpr bool kPoisonLds = false;
#endif

// Registers <-> LDS in the layout of phase PH.  `tok` points at this token's LDS region plus the
// thread's own (runtime) offset; register offsets are compile-time immediates.
template <class C, int PH>
__device__ __forceinline__ void lds_put(const float (&r)[C::E], float* tok) {
    static_for<0, C::E / 4>([&](auto i) {
        constexpr int I = decltype(i)::value * 4;
        constexpr unsigned off = C::template lds_reg<PH>(I);
        *reinterpret_cast<float4*>(tok + off) = make_float4(r[I], r[I + 1], r[I + 2], r[I + 3]);
    });
}

template <class C, int PH>
__device__ __forceinline__ void lds_get(float (&r)[C::E], const float* tok) {
    static_for<0, C::E / 4>([&](auto i) {
        constexpr int I = decltype(i)::value * 4;
        constexpr unsigned off = C::template lds_reg<PH>(I);
        const float4 q = *reinterpret_cast<const float4*>(tok + off);
        r[I] = q.x; r[I + 1] = q.y; r[I + 2] = q.z; r[I + 3] = q.w;
    });
    if constexpr (kPoisonLds) {
        const float nan = __uint_as_float(0x7fc00000u);
        static_for<0, C::E>([&](auto i) {
            constexpr int I = decltype(i)::value;
            constexpr unsigned off = C::template lds_reg<PH>(I & ~3) + (I & 3);
            const_cast<float*>(tok)[off] = nan;
        });
    }
}

__device__ __forceinline__ unsigned lds_byte_address(const void* p) {
    return (unsigned)(size_t)(const __attribute__((address_space(3))) unsigned char*)p;
}

// The same in assembly, for kernels in which the compiler would wait for every LDS-direct load in
// flight -- the prefetches of the next token group -- before an access to the exchange region that
// has nothing to do with them (the wave schedule's, and the backward pass of 2^14: 16384 tokens 353 -> 338 us,
// dx alone 222 -> 198, dalpha and dbeta alone 206 -> 194).  lds_get_raw waits for its own reads in the block that issues them.
template <unsigned OFF>
__device__ __forceinline__ void lds_write16(unsigned addr, const u32x4& q) {
    static_assert(OFF < 65536u, "offset field of the instruction");
    asm volatile("ds_write_b128 %0, %1 offset:%2" : : "v"(addr), "v"(q), "n"(OFF) : "memory");
}

template <class C, int PH>
__device__ __forceinline__ void lds_put_raw(const float (&r)[C::E], const float* tok) {
    const unsigned addr = lds_byte_address(tok);
    static_for<0, C::E / 4>([&](auto i) {
        constexpr int I = decltype(i)::value * 4;
        constexpr unsigned off = C::template lds_reg<PH>(I) * 4u;
        const u32x4 q = {__float_as_uint(r[I]), __float_as_uint(r[I + 1]), __float_as_uint(r[I + 2]), __float_as_uint(r[I + 3])};
        lds_write16<off>(addr, q);
    });
}

template <class C, int PH>
__device__ __forceinline__ void lds_get_raw(float (&r)[C::E], const float* tok) {
    static_assert(C::E % 16 == 0, "four accesses per block");
    const unsigned addr = lds_byte_address(tok);
    static_for<0, C::E / (C::E >= 32 ? 32 : 16)>([&](auto b) {
        constexpr int N4 = C::E >= 32 ? 8 : 4, B = decltype(b)::value * N4 * 4;
        const unsigned at = addr;
        u32x4 q[N4];
#define WHT_OFF(K) "n"(C::template lds_reg<PH>(B + 4 * (K)) * 4u)
        if constexpr (N4 == 8)
            asm volatile("ds_read_b128 %0, %8 offset:%9\n\tds_read_b128 %1, %8 offset:%10\n\t"
                         "ds_read_b128 %2, %8 offset:%11\n\tds_read_b128 %3, %8 offset:%12\n\t"
                         "ds_read_b128 %4, %8 offset:%13\n\tds_read_b128 %5, %8 offset:%14\n\t"
                         "ds_read_b128 %6, %8 offset:%15\n\tds_read_b128 %7, %8 offset:%16\n\ts_waitcnt lgkmcnt(0)"
                         : "=&v"(q[0]), "=&v"(q[1]), "=&v"(q[2]), "=&v"(q[3]), "=&v"(q[4]), "=&v"(q[5]), "=&v"(q[6]), "=&v"(q[7])
                         : "v"(at), WHT_OFF(0), WHT_OFF(1), WHT_OFF(2), WHT_OFF(3), WHT_OFF(4), WHT_OFF(5), WHT_OFF(6), WHT_OFF(7)
                         : "memory");
        else
            asm volatile("ds_read_b128 %0, %4 offset:%5\n\tds_read_b128 %1, %4 offset:%6\n\t"
                         "ds_read_b128 %2, %4 offset:%7\n\tds_read_b128 %3, %4 offset:%8\n\ts_waitcnt lgkmcnt(0)"
                         : "=&v"(q[0]), "=&v"(q[1]), "=&v"(q[2]), "=&v"(q[3])
                         : "v"(at), WHT_OFF(0), WHT_OFF(1), WHT_OFF(2), WHT_OFF(3) : "memory");
#undef WHT_OFF
#pragma unroll
        for (int k = 0; k < N4; ++k)
#pragma unroll
            for (int j = 0; j < 4; ++j) r[B + 4 * k + j] = __uint_as_float(q[k][j]);
    });
    if constexpr (kPoisonLds) {
        const u32x4 nan = {0x7fc00000u, 0x7fc00000u, 0x7fc00000u, 0x7fc00000u};
        static_for<0, C::E / 4>([&](auto i) {
            constexpr unsigned off = C::template lds_reg<PH>(decltype(i)::value * 4) * 4u;
            lds_write16<off>(addr, nan);
        });
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    }
}

// Per-thread constants: LDS word offset of the thread in every phase, element offset in the first
// and last phase (the global-memory layouts).
template <class C>
struct ThreadMap {
    unsigned lds_off[kMaxPhases];
    unsigned first_elem, last_elem;     // offset within the row in memory
    float lane_sign[4];                 // stages between lanes: -1 in the lanes of the lower butterfly output
    float sign;                         // their product (see lane_stage)
    __device__ __forceinline__ void init(unsigned t, unsigned slot) {
        static_for<0, C::P>([&](auto p) {
            constexpr int PH = decltype(p)::value;
            lds_off[PH] = slot * C::kTokenWords + C::phys(thread_elem_offset<C, PH>(t));
        });
        first_elem = thread_elem_offset<C, 0>(t);
        last_elem = thread_elem_offset<C, C::P - 1>(t);
        sign = 1.0f;
        if constexpr (C::kWave) {
            const unsigned c = wave_lane_to_bits(t, C::L);
            static_for<0, 4>([&](auto k) {
                constexpr int K = decltype(k)::value;
                lane_sign[K] = (K < C::L && ((c >> K) & 1u)) ? -1.0f : 1.0f;
                sign *= lane_sign[K];
            });
        }
    }
};

// Rows of 12 * 2^m elements: vector 0 (vector 1 lies a fixed distance behind it) and vector 2.
template <int LOGM, bool KEEP, int LEAST>
struct ThreadMap<TwelveCfg<LOGM, KEEP, LEAST>> {
    using C = TwelveCfg<LOGM, KEEP, LEAST>;
    unsigned lds_off[2];
    unsigned first_elem, last_elem, first_elem2, last_elem2;
    unsigned columns, columns2;         // LDS words of the column sums, in the last layout
    bool second;                        // vector 2 belongs to the second of the pair, in the first layout
    float lane_sign[3];                 // stages on the wave bits: -1 in the lanes of the lower butterfly output
    float sign;                         // their product
    __device__ __forceinline__ void init(unsigned t, unsigned slot) {
        const unsigned lane = t & 63u, wave = t >> 6;
        const LaneWave to = twelve_swap(lane, wave, C::w);
        lds_off[0] = slot * C::kTokenWords + twelve_place(to.lane, to.wave);
        lds_off[1] = slot * C::kTokenWords + twelve_place(lane, wave);
        first_elem = twelve_elem(lane, wave, 0, C::m);
        first_elem2 = twelve_elem(lane, wave, 2, C::m);
        last_elem = twelve_elem(to.lane, to.wave, 0, C::m);
        last_elem2 = twelve_elem(to.lane, to.wave, 2, C::m);
        second = twelve_pair(lane, 2) != 0u;
        sign = 1.0f;
        static_for<0, C::w>([&](auto k) {
            constexpr int K = decltype(k)::value;
            lane_sign[K] = ((lane >> twelve_lane_pos(K)) & 1u) ? -1.0f : 1.0f;
            sign *= lane_sign[K];
        });
        columns = slot * C::kTokenWords + C::phys(last_elem);
        columns2 = slot * C::kTokenWords + C::phys(last_elem2);
    }
};

// Offset in its row of vector VEC of the thread in the layout of phase PH.  next_row: rows of 768, two tokens
// to a wave, distance from the first token's row to the second's (0 where there is no second).
template <class C, int PH, int VEC>
__device__ __forceinline__ unsigned vector_offset(const ThreadMap<C>& tm, unsigned next_row) {
    if constexpr (C::kTwelve) {
        const unsigned step = C::kPair == 2 ? next_row : 64u;
        if constexpr (VEC == 2) return (PH > 0 ? tm.last_elem2 : tm.first_elem2) + (C::kPair == 2 && tm.second ? next_row : 0u);
        else return (PH > 0 ? tm.last_elem : tm.first_elem) + VEC * step;
    } else {
        constexpr unsigned off = reg_elem_offset(C::plan.ph[PH], C::e, VEC * C::V);
        return (PH == 0 ? tm.first_elem : tm.last_elem) + off;
    }
}

// One butterfly stage between lanes: position K of the lane index, the partner's value read through a
// DPP operand, one fused multiply-add per value:
//     v <- v + s * partner,   s = +1 in the upper lane of the pair, -1 in the lower.
// The lower lane so gets -(upper - lower), the negative of the butterfly's output.  Such signs pass
// unchanged through every other stage (both lanes of any other pair carry the same one), so after all
// lane stages a lane holds ThreadMap::sign times the transform, and the sign is folded into alpha.
// INPUT_SIGN is the transposed form, v <- v - s * partner: it takes input that carries the sign and
// gives the transform itself.  Products with +-1 are exact: the rounding is that of a plain addition.
// Written in assembly: the compiler keeps the DPP read as a move of its own in front of the multiply-
// add (twice the instructions).  It does not see the wait states around it either: two before a DPP
// operand that the preceding instruction wrote, hence the s_nop in front, and the one behind for a
// lane swap that may follow.
#define WHT_FMAC_DPP(R, CTRL) "v_fmac_f32_dpp %" #R ", %" #R ", %4 " CTRL " row_mask:0xf bank_mask:0xf\n\t"
#define WHT_FMAC_DPP4(CTRL)                                                                             \
    asm("s_nop 1\n\t" WHT_FMAC_DPP(0, CTRL) WHT_FMAC_DPP(1, CTRL) WHT_FMAC_DPP(2, CTRL)                 \
        WHT_FMAC_DPP(3, CTRL) "s_nop 1"                                                                \
        : "+v"(r[i]), "+v"(r[i + 1]), "+v"(r[i + 2]), "+v"(r[i + 3]) : "v"(s))
template <class C, int K, bool INPUT_SIGN>
__device__ __forceinline__ void lane_stage(float (&r)[C::E], const ThreadMap<C>& tm) {
    const float s = INPUT_SIGN ? -tm.lane_sign[K] : tm.lane_sign[K];
#pragma unroll
    for (int i = 0; i < C::E; i += 4) {
        if constexpr (K == 0)      WHT_FMAC_DPP4("quad_perm:[1,0,3,2]");     // l ^ 1
        else if constexpr (K == 1) WHT_FMAC_DPP4("quad_perm:[2,3,0,1]");     // l ^ 2
        else if constexpr (K == 2) WHT_FMAC_DPP4("row_half_mirror");         // l ^ 7
        else                       WHT_FMAC_DPP4("row_ror:8");               // l ^ 8
    }
}
#undef WHT_FMAC_DPP4
#undef WHT_FMAC_DPP

// Exchange register bit Q with lane position 4 (ROW16) or 5.
template <class C, int Q, bool ROW16>
__device__ __forceinline__ void lane_swap(float (&r)[C::E]) {
    static_for<0, C::E>([&](auto i) {
        constexpr int I = decltype(i)::value;
        if constexpr (!((I >> Q) & 1)) {
            constexpr int J = I | (1 << Q);
            const auto sw = [&] {
                if constexpr (ROW16)
                    return __builtin_amdgcn_permlane16_swap(__float_as_uint(r[I]), __float_as_uint(r[J]), false, false);
                else
                    return __builtin_amdgcn_permlane32_swap(__float_as_uint(r[I]), __float_as_uint(r[J]), false, false);
            }();
            r[I] = __uint_as_float(sw[0]);
            r[J] = __uint_as_float(sw[1]);
        }
    });
}

// The stage on element bit BIT while the token is in the layout of phase PH.
template <class C, int PH, int BIT, bool INPUT_SIGN>
__device__ __forceinline__ void wave_stage(float (&r)[C::E], const ThreadMap<C>& tm) {
    if constexpr ((C::plan.lane_bits >> BIT) & 1u) {
        lane_stage<C, BIT - C::v, INPUT_SIGN>(r, tm);
    } else {
        static_for<0, C::e>([&](auto q) {
            constexpr int Q = decltype(q)::value;
            if constexpr (C::plan.ph[PH].rb[Q] == BIT)
                static_for<0, C::E>([&](auto i) {
                    constexpr int I = decltype(i)::value;
                    if constexpr (!((I >> Q) & 1)) {
                        const float a = r[I], b = r[I | (1 << Q)];
                        r[I] = a + b;
                        r[I | (1 << Q)] = a - b;
                    }
                });
        });
    }
}

// H_raw on the values of a token.  Forward order enters in the first layout and leaves in the last,
// with the lanes' signs on the output; reverse order enters in the last layout with the signs on the
// input and leaves in the first.  `lds` is the region of the exchange between waves (unused without
// one); it is read after the barrier inside, so a put by another thread has to wait for a further one.
//   SKIP: element bit whose stage the caller has run already (-1: none).
template <class C, bool FORWARD_ORDER, int SKIP = -1>
__device__ __forceinline__ void wave_transform(float (&r)[C::E], float* lds, const ThreadMap<C>& tm) {
    constexpr int n = C::n, v = C::v, L = C::L, w = C::w;
    auto stage = [&](auto phase, auto bit) {
        if constexpr (decltype(bit)::value != SKIP)
            wave_stage<C, decltype(phase)::value, decltype(bit)::value, !FORWARD_ORDER>(r, tm);
    };
    std::integral_constant<int, 0> first;
    std::integral_constant<int, 1> second;
    std::integral_constant<int, 2> third;
    auto swaps = [&] {
        if constexpr (L >= 5) lane_swap<C, C::e - 1, true>(r);
        if constexpr (L == 6) lane_swap<C, C::e - 2, false>(r);
    };
    auto first_layout = [&] {
        static_for<0, n>([&](auto b) {
            constexpr int B = decltype(b)::value;
            if constexpr (B < v + 4 || B > v + 5 + w) stage(first, b);
        });
        if constexpr (n > v + 5 && L <= 5) stage(first, std::integral_constant<int, v + 5>{});
        if constexpr (n > v + 4 && L <= 4) stage(first, std::integral_constant<int, v + 4>{});
    };
    auto second_layout = [&] {
        if constexpr (L == 6) stage(second, std::integral_constant<int, v + 5>{});
        if constexpr (L >= 5) stage(second, std::integral_constant<int, v + 4>{});
    };
    auto exchange = [&](auto from, auto to) {
        lds_put_raw<C, decltype(from)::value>(r, lds + tm.lds_off[decltype(from)::value]);
        exchange_barrier();
        lds_get_raw<C, decltype(to)::value>(r, lds + tm.lds_off[decltype(to)::value]);
    };
    auto wave_bits = [&] {
        static_for<0, w>([&](auto k) { stage(third, std::integral_constant<int, v + 6 + decltype(k)::value>{}); });
    };
    if constexpr (FORWARD_ORDER) {
        first_layout(); swaps(); second_layout();
        if constexpr (w > 0) { exchange(second, third); wave_bits(); }
    } else {
        if constexpr (w > 0) { wave_bits(); exchange(third, second); }
        second_layout(); swaps(); first_layout();
    }
}

// Rows of 12 * 2^m elements: the stages on the wave bits, between the lanes of the last layout.  INPUT_SIGN as above.
#define WHT_FMAC_DPP12(CTRL)                                                                              \
    asm("s_nop 1\n\t" WHT_FMAC_DPP(0, CTRL) WHT_FMAC_DPP(1, CTRL) WHT_FMAC_DPP(2, CTRL) WHT_FMAC_DPP(3, CTRL)   \
        WHT_FMAC_DPP(4, CTRL) WHT_FMAC_DPP(5, CTRL) WHT_FMAC_DPP(6, CTRL) WHT_FMAC_DPP(7, CTRL)             \
        WHT_FMAC_DPP(8, CTRL) WHT_FMAC_DPP(9, CTRL) WHT_FMAC_DPP(10, CTRL) WHT_FMAC_DPP(11, CTRL)           \
        : "+v"(r[i]), "+v"(r[i + 1]), "+v"(r[i + 2]), "+v"(r[i + 3]), "+v"(r[i + 4]), "+v"(r[i + 5]),     \
          "+v"(r[i + 6]), "+v"(r[i + 7]), "+v"(r[i + 8]), "+v"(r[i + 9]), "+v"(r[i + 10]), "+v"(r[i + 11]) : "v"(s))
#define WHT_FMAC_DPP(R, CTRL) "v_fmac_f32_dpp %" #R ", %" #R ", %12 " CTRL " row_mask:0xf bank_mask:0xf\n\t"
template <class C, bool INPUT_SIGN>
__device__ __forceinline__ void wave_bit_stages(float (&r)[C::E], const ThreadMap<C>& tm) {
    static_for<0, C::w>([&](auto k) {
        constexpr int K = twelve_lane_pos(decltype(k)::value);
        const float s = INPUT_SIGN ? -tm.lane_sign[decltype(k)::value] : tm.lane_sign[decltype(k)::value];
#pragma unroll
        for (int i = 0; i < C::E; i += 12) {
            if constexpr (K == 0)      WHT_FMAC_DPP12("quad_perm:[1,0,3,2]");
            else if constexpr (K == 1) WHT_FMAC_DPP12("quad_perm:[2,3,0,1]");
            else                       WHT_FMAC_DPP12("row_ror:8");
        }
    });
}
#undef WHT_FMAC_DPP12
#undef WHT_FMAC_DPP

// The stages of the matrix-core schedule that are not in its rounds, on the 2^n values spread over the
// token's threads.
//   FORWARD_ORDER: registers enter in the first phase's layout and leave in the last phase's;
//   otherwise the phases run in reverse (enter in the last layout, leave in the first) -- the
//   backward pass uses this so that dy can be consumed in the layout z was produced in.
// With TRAILING_BARRIER it ends with a workgroup barrier when LDS was used, so the caller may reuse LDS at once.
template <class C, bool FORWARD_ORDER, bool TRAILING_BARRIER>
__device__ __forceinline__ void transform(float (&r)[C::E], float* lds, const ThreadMap<C>& tm) {
    if constexpr (C::kTwelve) {
        if constexpr (FORWARD_ORDER) {
            if constexpr (C::P > 1) {
                lds_put<C, 0>(r, lds + tm.lds_off[0]);
                exchange_barrier();
                lds_get<C, 1>(r, lds + tm.lds_off[1]);
                wave_bit_stages<C, false>(r, tm);
            }
        } else {
            if constexpr (C::P > 1) {
                wave_bit_stages<C, true>(r, tm);
                lds_put<C, 1>(r, lds + tm.lds_off[1]);
                exchange_barrier();
                lds_get<C, 0>(r, lds + tm.lds_off[0]);
            }
        }
    } else {
        // Two exchanges (d = 2^14 backward): the compiler would wait for the prefetches before the first get.  Not with
        // one tile per wave, where no stage lies between the products and the put: it does not see the wait states
        // between a product and an access in assembly either.
        constexpr bool RAW = C::P > 2 && C::t > 0;
        static_for<0, C::P>([&](auto s) {
            constexpr int S = decltype(s)::value;
            constexpr int PH = FORWARD_ORDER ? S : C::P - 1 - S;
            if constexpr (S > 0 && RAW) lds_get_raw<C, PH>(r, lds + tm.lds_off[PH]);
            else if constexpr (S > 0) lds_get<C, PH>(r, lds + tm.lds_off[PH]);
            run_stages<C, PH>(r);
            if constexpr (S + 1 < C::P) {
                // a middle phase rewrites exactly the words it read, so only the hand-over to the
                // next layout needs the barrier
                if constexpr (RAW) lds_put_raw<C, PH>(r, lds + tm.lds_off[PH]);
                else lds_put<C, PH>(r, lds + tm.lds_off[PH]);
                exchange_barrier();
            }
        });
    }
    // The next write into the exchange region must not overtake other waves' reads of this one.
    // When the next transform runs in the opposite order (the backward kernel alternates), its
    // first write goes, thread by thread, to exactly the words this thread has just read, and no
    // barrier is needed; a kernel that only runs forward-order transforms needs it.
    if constexpr (C::P > 1 && TRAILING_BARRIER) exchange_barrier();
}

// The tokens of a workgroup's slots.
template <class C>
struct Walker {
    int64_t N, groups;
    unsigned slot;
    // first token of the slot
    __device__ __forceinline__ int64_t token(int64_t grp) const {
        return grp * C::G + slot * C::kPair;
    }
    __device__ __forceinline__ int64_t row(int64_t grp) const {       // clamped: always a valid row
        const int64_t tok = token(grp);
        return tok < N ? tok : N - 1;
    }
    // From the first row of a slot to its second, where it has two: 0 past the last token, so that the first
    // is read again.
    __device__ __forceinline__ unsigned next_row(int64_t grp) const {
        if constexpr (C::kPair == 2)
            return grp * C::G + 2 * (unsigned)__builtin_amdgcn_readfirstlane(slot) + 1 < N ? C::kRow : 0u;
        else return 0u;
    }
    // Whether the slot fetches anything for group grp (matrix-core schedule: a slot is whole waves).  The
    // clamped row of a slot without a token is another slot's, which the backward pass may overwrite (dx may
    // alias x or dy); where no barrier keeps that store behind this read, the slot reads nothing.
    __device__ __forceinline__ bool fetches(int64_t grp) const {
        if constexpr (C::G == 1 || C::P > 1) return true;
        else return grp * C::G + C::kPair * (unsigned)__builtin_amdgcn_readfirstlane(slot) < N;
    }
};

// Global -> LDS staging -> registers.  x and dy are fetched with LDS-direct loads (the data goes
// from memory into LDS without passing through registers), a whole iteration before they are used,
// so that tens of KiB per workgroup are in flight at all times at no register cost.  An LDS-direct
// load of 16 bytes writes lane l's vector to (wave-uniform base) + 16*l: every wave owns a private
// 1 KiB slot per vector, reads back exactly what it fetched, and needs no workgroup barrier --
// only its own vmcnt (loads return in issue order) and lgkmcnt waits, which are written out here
// because the compiler does not track the dependence between an LDS-direct load and a later LDS read.
typedef const __attribute__((address_space(1))) void* global_cptr;
typedef __attribute__((address_space(3))) void* lds_ptr;

template <class C, int PH>
__device__ __forceinline__ void stage_issue(unsigned char* wave_slot, const typename C::io::elem_t* tensor,
                                            const Walker<C>& wk, int64_t grp, const ThreadMap<C>& tm) {
    const typename C::io::elem_t* row = tensor + wk.row(grp) * C::kRow;
    const unsigned next = wk.next_row(grp);
    static_for<0, C::NV>([&](auto c) {
        constexpr int Cc = decltype(c)::value;
        const typename C::io::elem_t* p = row + vector_offset<C, PH, Cc>(tm, next);
        // (the builtin takes a literal)
        if constexpr (C::kKeep) __builtin_amdgcn_global_load_lds((global_cptr)p, (lds_ptr)(wave_slot + Cc * 1024), 16, 0, 0);
        else __builtin_amdgcn_global_load_lds((global_cptr)p, (lds_ptr)(wave_slot + Cc * 1024), 16, 0, kStreamPolicy);
    });
}

// Read the staged vectors back.  Written as inline assembly on purpose: for a compiler-visible
// LDS load the waitcnt insertion would wait for *every* LDS-direct load in flight (vmcnt(0)),
// including the next group's prefetch issued moments ago.  Which loads must have landed is known
// here (wait_vmem below, issued by the caller first); the reads' own completion is awaited inside
// this function, with the values tied to the wait so that no use can be scheduled before it.
//   OWN: the slot was filled by this wave's own loads and nobody else reads it (poisoned after the
//   read in the debug build); false for a slot that another wave fetched or also reads.
template <class C, bool OWN = true>
__device__ __forceinline__ void stage_read(uint4 (&raw)[C::NV], const unsigned char* wave_slot) {
    static_assert(C::NV <= 4 || C::NV == 8, "unexpected vector count");
    const unsigned addr = lds_byte_address(wave_slot) + (threadIdx.x & 63u) * 16u;
    u32x4 v[C::NV];
#pragma unroll
    for (int c = 0; c < C::NV; ++c) {
        const unsigned a = addr + c * 1024;
        asm volatile("ds_read_b128 %0, %1" : "=&v"(v[c]) : "v"(a) : "memory");
    }
    if constexpr (C::NV == 1)
        asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(v[0]) : : "memory");
    else if constexpr (C::NV == 2)
        asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(v[0]), "+v"(v[1]) : : "memory");
    else if constexpr (C::NV == 3)
        asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(v[0]), "+v"(v[1]), "+v"(v[2]) : : "memory");
    else if constexpr (C::NV == 4)
        asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(v[0]), "+v"(v[1]), "+v"(v[2]), "+v"(v[3]) : : "memory");
    else
        asm volatile("s_waitcnt lgkmcnt(0)"
                     : "+v"(v[0]), "+v"(v[1]), "+v"(v[2]), "+v"(v[3]), "+v"(v[4]), "+v"(v[5]), "+v"(v[6]), "+v"(v[7])
                     : : "memory");
#pragma unroll
    for (int c = 0; c < C::NV; ++c) raw[c] = make_uint4(v[c].x, v[c].y, v[c].z, v[c].w);
    if constexpr (kPoisonLds && OWN) {
        const u32x4 nan = {0x7fc07fc0u, 0x7fc07fc0u, 0x7fc07fc0u, 0x7fc07fc0u};   // NaN as bf16 pairs and as f32
#pragma unroll
        for (int c = 0; c < C::NV; ++c) {
            const unsigned a = addr + c * 1024;
            asm volatile("ds_write_b128 %0, %1" : : "v"(a), "v"(nan) : "memory");
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    }
}

// Rows of 768, two tokens to a wave: zeros in the wave's stage slot for the tokens that a ragged last group does
// not have.  (Zeros in the registers instead cost 44 moves per iteration, ragged or not.)
template <class C>
__device__ __forceinline__ void zero_missing(unsigned char* wave_slot, const Walker<C>& wk, int64_t grp, const ThreadMap<C>& tm) {
    if constexpr (C::kPair == 2) {
        const int64_t left = wk.N - (grp * C::G + 2 * (unsigned)__builtin_amdgcn_readfirstlane(wk.slot));
        if (left < 2) {
            const u32x4 zero = {0u, 0u, 0u, 0u};
            const unsigned addr = lds_byte_address(wave_slot) + (threadIdx.x & 63u) * 16u;
            if (left < 1) asm volatile("ds_write_b128 %0, %1" : : "v"(addr), "v"(zero) : "memory");
            asm volatile("ds_write_b128 %0, %1 offset:1024" : : "v"(addr), "v"(zero) : "memory");
            if (left < 1 || tm.second) asm volatile("ds_write_b128 %0, %1 offset:2048" : : "v"(addr), "v"(zero) : "memory");
        }
    }
}

// Wait until at most PENDING of this wave's vector-memory operations are outstanding.
template <int PENDING>
__device__ __forceinline__ void wait_vmem() {
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(PENDING) : "memory");
}
template <class C>
__device__ __forceinline__ void unpack_all(float (&r)[C::E], const uint4 (&raw)[C::NV]) {
    static_for<0, C::NV>([&](auto c) {
        constexpr int Cc = decltype(c)::value;
        C::io::unpack(raw[Cc], &r[Cc * C::V]);
    });
}

// The rows that a wave stores: up to PER tokens from its first one on, none past the last token.
template <class C>
struct OutRows {
    static constexpr int PER = C::TPT < 64 ? 64 / C::TPT : C::kPair;
    static constexpr unsigned kRowBytes = C::kRow * (unsigned)sizeof(typename C::io::elem_t);
    rsrc_t to;
    unsigned lane_row;              // this lane's row from there, in elements
    __device__ __forceinline__ OutRows(typename C::io::elem_t* tensor, int64_t grp, int64_t N, unsigned slot) {
        const unsigned first_slot = __builtin_amdgcn_readfirstlane(slot);
        const int64_t first = grp * C::G + first_slot * C::kPair, left = N - first;
        to = make_rsrc(tensor + first * C::kRow, (left < 0 ? 0u : left < PER ? (unsigned)left : (unsigned)PER) * kRowBytes);
        lane_row = C::TPT < 64 ? (slot - first_slot) * C::kRow : 0u;
    }
};

// Registers in the layout of phase PH -> the rows of the tokens that exist, through L2 ...
template <class C, int PH>
__device__ __forceinline__ void global_put_through(const float (&r)[C::E], typename C::io::elem_t* tensor,
                                                   unsigned slot, int64_t N, int64_t grp, const ThreadMap<C>& tm) {
    const OutRows<C> rows(tensor, grp, N, slot);
    static_for<0, C::NV>([&](auto c) {
        constexpr int Cc = decltype(c)::value;
        const unsigned at = rows.lane_row + vector_offset<C, PH, Cc>(tm, C::kRow);
        store16_through(rows.to, at * (unsigned)sizeof(typename C::io::elem_t), C::io::pack(&r[Cc * C::V]));
    });
}
// ... or with plain or (STREAM) non-temporal stores.
template <class C, int PH, bool STREAM>
__device__ __forceinline__ void global_put(const float (&r)[C::E], typename C::io::elem_t* tensor,
                                           unsigned slot, int64_t N, int64_t grp, const ThreadMap<C>& tm) {
    const int64_t tok = grp * C::G + slot * C::kPair;
    typename C::io::elem_t* row = tensor + tok * C::kRow;
    static_for<0, C::NV>([&](auto c) {
        constexpr int Cc = decltype(c)::value;
        bool active = C::G == 1 || tok < N;
        if constexpr (C::kPair == 2) active = tok + (Cc == 2 ? (tm.second ? 1 : 0) : Cc) < N;
        if (active) {
            typename C::io::elem_t* p = row + vector_offset<C, PH, Cc>(tm, C::kRow);
            if constexpr (STREAM) stream_store16(p, C::io::pack(&r[Cc * C::V]));
            else *reinterpret_cast<uint4*>(p) = C::io::pack(&r[Cc * C::V]);
        }
    });
}
// The persistent kernels' y and dx.
template <class C, int PH, bool THROUGH>
__device__ __forceinline__ void put_output(const float (&r)[C::E], typename C::io::elem_t* tensor, unsigned slot,
                                           int64_t N, int64_t grp, const ThreadMap<C>& tm) {
    if constexpr (THROUGH) global_put_through<C, PH>(r, tensor, slot, N, grp, tm);
    else global_put<C, PH, true>(r, tensor, slot, N, grp, tm);
}

template <class C>
__device__ __forceinline__ float inv_sqrt_d() {
    if constexpr (C::kTwelve) {
        // d = 3 * 2^(n-2): 1/sqrt(3) or 1/sqrt(6), rounded once, times a power of two
        return ((C::n - 2) % 2 == 0) ? 0.57735026918962576451f / float(1 << ((C::n - 2) / 2))
                                     : 0.40824829046386301637f / float(1 << ((C::n - 2) / 2));
    }
    // exact power of two for even log2 d; one rounding of 1/sqrt(2) * 2^-k otherwise
    return (C::n % 2 == 0) ? 1.0f / float(1 << (C::n / 2))
                           : 0.70710678118654752440f / float(1 << (C::n / 2));
}

// float32 parameter vector -> registers in the layout of the last phase.
template <class C>
__device__ __forceinline__ void param_load(float (&r)[C::E], const float* p, const ThreadMap<C>& tm) {
    static_for<0, C::E / 4>([&](auto i) {
        constexpr int I = decltype(i)::value * 4, VEC = I / C::V;
        if constexpr (C::kPair == 2 && VEC == 1) {                     // the same columns as vector 0
            for (int k = 0; k < 4; ++k) r[I + k] = r[I - C::V + k];
        } else {
            const float4 q = *reinterpret_cast<const float4*>(p + vector_offset<C, C::P - 1, VEC>(tm, 0u) + I % C::V);
            r[I] = q.x; r[I + 1] = q.y; r[I + 2] = q.z; r[I + 3] = q.w;
        }
    });
}
// alpha / sqrt d, with the signs that the last layout carries.
template <class C>
__device__ __forceinline__ void scale_alpha(float (&a)[C::E], const ThreadMap<C>& tm) {
    const float s = inv_sqrt_d<C>() * tm.sign;
#pragma unroll
    for (int i = 0; i < C::E; ++i) a[i] *= s;
}
template <class C>
__device__ __forceinline__ void alpha_get(float (&a)[C::E], const float* p, const ThreadMap<C>& tm) {
    param_load<C>(a, p, tm);
    scale_alpha<C>(a, tm);
}

// ------------------------------------------------------------------------------------------------
// matrix-core rounds: H_32 along five element bits as a 32x32x32 product with a +-1 matrix
//
// v_mfma_f32_32x32x16_bf16 operand layout (two instructions cover K = 32):
//   A[i][k]: lane = i + 32*(k/8 % 2), element k%8 of the lane's 8 bf16, instruction k/16
//   B[k][j]: lane = j + 32*(k/8 % 2), element k%8, instruction k/16
//   D[i][j]: lane = j + 32*(i/4 % 2), register 4*(i/8) + i%4
// With B[k][j] = (-1)^popcount(k & swap23(j)) (bits 2 and 3 of j exchanged) the accumulator of a
// round is again an A operand for the next one -- rows <-> the previous round's outputs, K <-> the
// previous round's rows -- and after two rounds each lane holds, in register order, the 8 + 8
// consecutive elements it loaded.

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

struct HadamardB {
    bf16x8 k_lo, k_hi;      // B operand of the first / second K-half
};

__device__ __forceinline__ HadamardB make_hadamard_b() {
    const unsigned lane = threadIdx.x & 63u;
    const unsigned j = lane & 31u, kg = lane >> 5;
    const unsigned js = (j & 0x13u) | ((j & 4u) << 1) | ((j & 8u) >> 1);
    uint32_t w[2][4];
#pragma unroll
    for (int half = 0; half < 2; ++half)
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            const unsigned k0 = (2u * p) | (kg << 3) | ((unsigned)half << 4), k1 = k0 | 1u;
            const uint32_t lo = (__popc(k0 & js) & 1) ? 0xBF80u : 0x3F80u;     // bf16 -1 : +1
            const uint32_t hi = (__popc(k1 & js) & 1) ? 0xBF80u : 0x3F80u;
            w[half][p] = lo | (hi << 16);
        }
    HadamardB b;
    b.k_lo = __builtin_bit_cast(bf16x8, make_uint4(w[0][0], w[0][1], w[0][2], w[0][3]));
    b.k_hi = __builtin_bit_cast(bf16x8, make_uint4(w[1][0], w[1][1], w[1][2], w[1][3]));
    return b;
}

// One round on bfloat16 data straight from memory: products and sums are exact up to the
// accumulator's float32 rounding.
__device__ __forceinline__ f32x16 hadamard_round_bf16(const uint4& a_lo, const uint4& a_hi,
                                                      const HadamardB& b) {
    f32x16 acc = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a_lo), b.k_lo, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a_hi), b.k_hi, acc, 0, 0, 0);
    return acc;
}

// float32 values as bf16 hi + bf16 lo (hi = RNE(v), lo = RNE(v - hi); v - hi is exact, so |v - hi - lo|
// <= 2^-17 |v|): both parts go through the same +-1 product, accumulated in float32.  v - hi is formed with plain vector instructions (widen hi by
// a shift / a mask, subtract): the bf16 dot-product instruction would do it in one, but it executes
// on the matrix pipeline and stalls behind the rounds' own MFMAs (measured: 20 cycles per dot
// instruction next to back-to-back MFMAs, against 4.4 alone).
template <int PAIRS>
__device__ __forceinline__ void split_bf16(const float* v, uint32_t* hi, uint32_t* lo) {
#pragma unroll
    for (int p = 0; p < PAIRS; ++p) {
        const uint32_t h = IoBF16::pack2(v[2 * p], v[2 * p + 1]);
        const float l0 = v[2 * p] - __uint_as_float(h << 16);
        const float l1 = v[2 * p + 1] - __uint_as_float(h & 0xffff0000u);
        hi[p] = h;
        lo[p] = IoBF16::pack2(l0, l1);
    }
}

// One round on float32 data.
__device__ __forceinline__ f32x16 hadamard_round_f32(const float* v, const HadamardB& b) {
    uint32_t hi[8], lo[8];
    split_bf16<8>(v, hi, lo);
    f32x16 acc = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    const bf16x8 lo0 = __builtin_bit_cast(bf16x8, make_uint4(lo[0], lo[1], lo[2], lo[3]));
    const bf16x8 lo1 = __builtin_bit_cast(bf16x8, make_uint4(lo[4], lo[5], lo[6], lo[7]));
    const bf16x8 hi0 = __builtin_bit_cast(bf16x8, make_uint4(hi[0], hi[1], hi[2], hi[3]));
    const bf16x8 hi1 = __builtin_bit_cast(bf16x8, make_uint4(hi[4], hi[5], hi[6], hi[7]));
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lo0, b.k_lo, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lo1, b.k_hi, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(hi0, b.k_lo, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(hi1, b.k_hi, acc, 0, 0, 0);
    return acc;
}

// Rows of 12 * 2^m elements: the two rounds of wht_plan.h on v_mfma_f32_16x16x32_bf16,
//   A[i][k]: lane = i + 16*(k/8), element k%8;   B[k][j]: lane = j + 16*(k/8), element k%8;
//   D[i][j]: lane = j + 16*(i/4), register i%4.
// What bounds them is the two-term split of round 2's input, 3 vector instructions per value; the products are
// 22 (from bfloat16) or 28 of 16 cycles per wave.
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x8 __attribute__((ext_vector_type(8)));

struct TwelveB {
    bf16x8 b1[2];                   // round 1, by output half
    bf16x8 main[2], shared[2];      // round 2, by pair: results for vector `pair`, for vector 2
};
template <class C>
__device__ __forceinline__ TwelveB make_twelve_b() {
    const unsigned lane = threadIdx.x & 63u;
    auto words = [](auto f) { return __builtin_bit_cast(bf16x8, make_uint4(f(0), f(1), f(2), f(3))); };
    TwelveB b;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        b.b1[i] = words([&](int word) { return twelve_round1_word(lane, i, word); });
        b.main[i] = words([&](int word) { return twelve_round2_word(lane, i, false, word, C::m); });
        b.shared[i] = words([&](int word) { return twelve_round2_word(lane, i, true, word, C::m); });
    }
    return b;
}
__device__ __forceinline__ f32x4 product16(const bf16x8& a, const bf16x8& b, const f32x4& acc) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, acc, 0, 0, 0);
}

template <class C>
__device__ __forceinline__ void twelve_round2(float (&r)[C::E], const f32x4 (&d1)[3][C::V / 4], const TwelveB& b, bool second) {
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    static_for<0, C::V / 4>([&](auto half) {
        constexpr int H = decltype(half)::value;
        uint32_t hi[3][2], lo[3][2];
#pragma unroll
        for (int v = 0; v < 3; ++v) {
            const float q[4] = {d1[v][H][0], d1[v][H][1], d1[v][H][2], d1[v][H][3]};
            split_bf16<2>(q, hi[v], lo[v]);
        }
        // operands of pair 0 and 1, lo and hi: slices of the registers (0, 2, 1)
        bf16x8 a[2][2];
#pragma unroll
        for (int term = 0; term < 2; ++term) {
            const uint32_t (&q)[3][2] = term == 0 ? lo : hi;
            if constexpr (C::kPair == 2) {
                // two tokens: zeros for the other one's values (a product with zero would let its NaN in)
                const bool upper = (threadIdx.x & 32u) != 0u;
                a[term][0] = __builtin_bit_cast(bf16x8, make_uint4(q[0][0], q[0][1], upper ? 0u : q[2][0], upper ? 0u : q[2][1]));
                a[term][1] = __builtin_bit_cast(bf16x8, make_uint4(upper ? q[2][0] : 0u, upper ? q[2][1] : 0u, q[1][0], q[1][1]));
            } else {
                const u32x8 all = {q[0][0], q[0][1], q[2][0], q[2][1], q[1][0], q[1][1], 0u, 0u};
                a[term][0] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(all, all, 0, 1, 2, 3));
                a[term][1] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(all, all, 2, 3, 4, 5));
            }
        }
        f32x4 out[3];
        out[0] = product16(a[1][0], b.main[0], product16(a[0][0], b.main[0], zero));
        out[1] = product16(a[1][1], b.main[1], product16(a[0][1], b.main[1], zero));
        if constexpr (C::kPair == 2) {
            const f32x4 s0 = product16(a[1][0], b.shared[0], product16(a[0][0], b.shared[0], zero));
            const f32x4 s1 = product16(a[1][1], b.shared[1], product16(a[0][1], b.shared[1], zero));
#pragma unroll
            for (int i = 0; i < 4; ++i) out[2][i] = second ? s1[i] : s0[i];
        } else {
            out[2] = product16(a[0][1], b.shared[1], product16(a[0][0], b.shared[0], zero));
            out[2] = product16(a[1][1], b.shared[1], product16(a[1][0], b.shared[0], out[2]));
        }
#pragma unroll
        for (int v = 0; v < 3; ++v)
#pragma unroll
            for (int i = 0; i < 4; ++i) r[C::V * v + 4 * H + i] = out[v][i];
    });
    if constexpr (C::kPair == 1) {                          // the stage on r6; vector 2's is in the product
#pragma unroll
        for (int i = 0; i < C::V; ++i) {
            const float p = r[i], q = r[C::V + i];
            r[i] = p + q;
            r[C::V + i] = p - q;
        }
    }
}

// The schedule's matrices, and its rounds on a thread's values.
template <class C>
using RoundB = std::conditional_t<C::kTwelve, TwelveB, HadamardB>;
template <class C>
__device__ __forceinline__ RoundB<C> make_round_b() {
    if constexpr (C::kTwelve) return make_twelve_b<C>();
    else return make_hadamard_b();
}

// Both rounds on every tile of the thread: bits 0..9 of the element index.  Round 1 of every tile
// is issued before any round 2, so that one tile's split has the other tile's matrix instructions
// to overlap with.  (Explicit MFMA/VALU interleave hints on top of this measured no gain.)
template <class C>
__device__ __forceinline__ void mfma_round2(float (&r)[C::E], const f32x16 (&d1)[C::T], const HadamardB& b) {
    static_for<0, C::T>([&](auto tile) {
        constexpr int Tl = decltype(tile)::value;
        float v[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) v[i] = d1[Tl][i];
        const f32x16 d2 = hadamard_round_f32(v, b);
#pragma unroll
        for (int i = 0; i < 16; ++i) r[16 * Tl + i] = d2[i];
    });
}
//   from raw bfloat16 (the forward input x): round 1 needs no split
template <class C>
__device__ __forceinline__ void mfma_rounds_from_bf16(float (&r)[C::E], const uint4 (&raw)[C::NV], const RoundB<C>& b,
                                                      const ThreadMap<C>& tm) {
    if constexpr (C::kTwelve) {
        const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
        f32x4 d1[3][C::V / 4];
#pragma unroll
        for (int v = 0; v < 3; ++v)
#pragma unroll
            for (int h = 0; h < C::V / 4; ++h) d1[v][h] = product16(__builtin_bit_cast(bf16x8, raw[v]), b.b1[h], zero);
        twelve_round2<C>(r, d1, b, tm.second);
    } else {
        f32x16 d1[C::T];
        static_for<0, C::T>([&](auto tile) {
            constexpr int Tl = decltype(tile)::value;
            d1[Tl] = hadamard_round_bf16(raw[2 * Tl], raw[2 * Tl + 1], b);
        });
        mfma_round2<C>(r, d1, b);
    }
}
//   from float32 registers in the first layout (the backward pass's alpha' (.) dy): round 1, and both
template <class C>
using Round1 = std::conditional_t<C::kTwelve, f32x4[3][2], f32x16[C::kTwelve ? 1 : C::E / 16]>;
template <class C>
__device__ __forceinline__ void mfma_round1_from_f32(const float (&r)[C::E], Round1<C>& d1, const RoundB<C>& b) {
    if constexpr (C::kTwelve) {
        const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int v = 0; v < 3; ++v) {
            uint32_t hi[4], lo[4];
            split_bf16<4>(&r[8 * v], hi, lo);
            const bf16x8 a_hi = __builtin_bit_cast(bf16x8, make_uint4(hi[0], hi[1], hi[2], hi[3]));
            const bf16x8 a_lo = __builtin_bit_cast(bf16x8, make_uint4(lo[0], lo[1], lo[2], lo[3]));
#pragma unroll
            for (int h = 0; h < 2; ++h) d1[v][h] = product16(a_hi, b.b1[h], product16(a_lo, b.b1[h], zero));
        }
    } else {
        static_for<0, C::T>([&](auto tile) {
            constexpr int Tl = decltype(tile)::value;
            d1[Tl] = hadamard_round_f32(&r[16 * Tl], b);
        });
    }
}
template <class C>
__device__ __forceinline__ void mfma_round2(float (&r)[C::E], const Round1<C>& d1, const RoundB<C>& b, const ThreadMap<C>& tm) {
    if constexpr (C::kTwelve) twelve_round2<C>(r, d1, b, tm.second);
    else mfma_round2<C>(r, d1, b);
}
template <class C>
__device__ __forceinline__ void mfma_rounds_from_f32(float (&r)[C::E], const RoundB<C>& b, const ThreadMap<C>& tm) {
    Round1<C> d1;
    mfma_round1_from_f32<C>(r, d1, b);
    mfma_round2<C>(r, d1, b, tm);
}

// raw x[tok] (first layout) -> H_raw x in the last layout, whichever schedule C is.
template <class C, bool TRAILING_BARRIER>
__device__ __forceinline__ void transform_from_raw(float (&r)[C::E], const uint4 (&raw)[C::NV],
                                                   float* lds, const ThreadMap<C>& tm, const RoundB<C>& b) {
    if constexpr (C::kMfma) {
        mfma_rounds_from_bf16<C>(r, raw, b, tm);
        transform<C, true, TRAILING_BARRIER>(r, lds, tm);
    } else {
        unpack_all<C>(r, raw);
        wave_transform<C, true>(r, lds, tm);
        if constexpr (C::w > 0 && TRAILING_BARRIER) exchange_barrier();
    }
}

// registers in the last layout -> H_raw (.) in the first layout (matrix-core schedule).
template <class C, bool TRAILING_BARRIER = false>
__device__ __forceinline__ void transform_back(float (&r)[C::E], float* lds, const ThreadMap<C>& tm, const RoundB<C>& b) {
    transform<C, false, TRAILING_BARRIER>(r, lds, tm);
    mfma_rounds_from_f32<C>(r, b, tm);
}

// ------------------------------------------------------------------------------------------------
// Kernels.  A workgroup holds G token slots of TPT threads each and strides over token groups
// (persistent grid).  Inputs of group k+1 are in flight (LDS-direct loads) while group k is
// computed.  In a ragged last group a slot without a token re-reads the last token (clamped row), or reads
// nothing where dx could be stored over that row meanwhile; its stores and its sums are left out.

// Four sums of a partial row; with which policy: sums_store (wht_route.h).
template <class C, bool DX>
constexpr int sums_policy() {
    constexpr Store store = sums_store(rows_of<C>(), DX);
    return store == Store::Plain ? 0 : store == Store::Stream ? kStreamPolicy : kThroughPolicy;
}
template <int POLICY>
__device__ __forceinline__ void put_sums(rsrc_t row, unsigned column, const float4& q) {
    const u32x4 v = {__float_as_uint(q.x), __float_as_uint(q.y), __float_as_uint(q.z), __float_as_uint(q.w)};
    __builtin_amdgcn_raw_buffer_store_b128(v, row, column * 4u, 0, POLICY);
}

__device__ __forceinline__ float4 add4(const float4& a, const float4& b) {
    return make_float4(a.x + b.x, a.y + b.y, a.z + b.z, a.w + b.w);
}

// Where a backward kernel's workgroup writes its sums: rows of the workspace ([grid][2][kRow]), or, for a
// single workgroup, dalpha and dbeta themselves.
struct SumRows {
    float* dalpha;
    float* dbeta;
    int stride;                     // floats between the rows of consecutive workgroups
    template <class C>
    __device__ __forceinline__ rsrc_t row(int which) const {
        return make_rsrc((which == 0 ? dalpha : dbeta) + (size_t)blockIdx.x * stride, C::kRow * 4u);
    }
};

// sumsq[tok] = sum of the token's r[i]^2 (the values as they stand, before rounding for the store):
// each thread squares its values, the lanes of a token add up by butterfly shuffles, and a token that
// spans several waves adds the wave sums through `wave_sums` (one float per wave of the workgroup)
// in a fixed order, behind one workgroup barrier that every wave passes.
template <class C>
__device__ __forceinline__ void token_sumsq(const float (&r)[C::E], float* wave_sums, float* __restrict__ sumsq,
                                            int64_t tok, int64_t N, unsigned t, unsigned slot, const ThreadMap<C>& tm) {
    if constexpr (C::kPair == 2) {            // two tokens to a wave
        float sq[2] = {0.0f, 0.0f}, both = 0.0f;
#pragma unroll
        for (int i = 0; i < C::V; ++i) {
            sq[0] = fmaf(r[i], r[i], sq[0]);
            sq[1] = fmaf(r[C::V + i], r[C::V + i], sq[1]);
            both = fmaf(r[2 * C::V + i], r[2 * C::V + i], both);
        }
        sq[0] += tm.second ? 0.0f : both;
        sq[1] += tm.second ? both : 0.0f;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            sq[0] += __shfl_xor(sq[0], off);
            sq[1] += __shfl_xor(sq[1], off);
        }
        if (t < 2 && tok + t < N) sumsq[tok + t] = t == 0 ? sq[0] : sq[1];
        return;
    }
    float sq = 0.0f;
#pragma unroll
    for (int i = 0; i < C::E; ++i) sq = fmaf(r[i], r[i], sq);
    constexpr int kLanes = C::TPT < 64 ? C::TPT : 64;       // lanes of one wave that share a token
#pragma unroll
    for (int off = 1; off < kLanes; off <<= 1) sq += __shfl_xor(sq, off);
    if constexpr (C::TPT <= 64) {
        if (t == 0 && tok < N) sumsq[tok] = sq;
    } else {
        constexpr int kWaves = C::TPT / 64;                 // waves per token
        if ((threadIdx.x & 63u) == 0) wave_sums[threadIdx.x >> 6] = sq;
        exchange_barrier();
        if (t == 0 && tok < N) {
            float total = 0.0f;
#pragma unroll
            for (int wv = 0; wv < kWaves; ++wv) total += wave_sums[slot * kWaves + wv];
            sumsq[tok] = total;
        }
    }
}

// forward:  y = (alpha / sqrt d) (.) (H_raw x) + beta      [+ resid when RESID]
//
// Per iteration k (x(k) [and resid(k)] have landed in their stages):
//   raw <- stage;  issue x(k+1) -> stage;  transform raw;  affine;  wait for everything pending;
//   store y(k).
// The one wait sits just before the stores of y(k): all it can be waiting for is x(k+1), issued a
// whole transform earlier, and the stores of y(k-1), a whole iteration old.  (Loads and stores may
// complete out of order with respect to each other, so a counted wait is only safe when nothing
// but older loads is pending; waiting here, before the new stores, keeps it that way.)
// RESID fuses the attention block's residual add into the epilogue: resid is one more staged
// stream, fetched in the layout y is stored in.
// STATS (with RESID) also writes sumsq[token] = sum_j y[token][j]^2, taken from the float32 values
// before they are rounded for the store: the statistic of an RMS normalisation that follows the
// residual stream.  Each thread squares its values, the lanes of a token add up by butterfly
// shuffles, and a token that spans several waves adds the wave sums through LDS in a fixed order
// (one more workgroup barrier per token; the next write to that LDS array is behind the next
// token's exchange barriers, so nothing else is needed).
template <class C, bool RESID, bool STATS, bool THROUGH>
__global__ __launch_bounds__(C::BT) void forward_kernel(const typename C::io::elem_t* x,
                                                        const float* __restrict__ alpha,
                                                        const float* __restrict__ beta,
                                                        const typename C::io::elem_t* resid,
                                                        typename C::io::elem_t* y,
                                                        float* __restrict__ sumsq,
                                                        int64_t N, int cluster) {
    static_assert(!STATS || RESID, "the statistic belongs to the residual-stream output");
    static_assert(!STATS || C::TPT <= 64 || C::P > 1, "a token of several waves has an exchange");
    __shared__ float wave_sums[STATS ? C::BT / 64 : 1];
    // separate LDS objects: the compiler can then tell that the exchange region's accesses never
    // alias an LDS-direct load in flight, and does not wait for the prefetch before them
    __shared__ __align__(16) float lds[C::kExchangeBytes / 4];
    __shared__ __align__(16) unsigned char stage_buf[C::kStageBytes];
    __shared__ __align__(16) unsigned char stage_r_buf[RESID ? C::kStageBytes : 16];
    constexpr int LAST = C::P - 1;
    const unsigned t = threadIdx.x % C::TPT;
    Walker<C> wk{N, (N + C::G - 1) / C::G, threadIdx.x / C::TPT};
    ThreadMap<C> tm;
    tm.init(t, wk.slot);
    unsigned char* stage = stage_buf + (threadIdx.x >> 6) * (C::NV * 1024);
    unsigned char* stage_r = stage_r_buf + (RESID ? (threadIdx.x >> 6) * (C::NV * 1024) : 0);

    // Token groups are dealt to clusters of `cluster` consecutive workgroups: the token groups are
    // cut into gridDim.x / cluster contiguous regions, and a cluster walks its region interleaved
    // (workgroup j of the cluster takes groups j, j + cluster, ...).  cluster = gridDim.x is the
    // plain interleave over the whole grid.
    const int64_t step = cluster;
    const int64_t nclus = gridDim.x / cluster, clus = blockIdx.x / cluster;
    const int64_t per = (wk.groups + nclus - 1) / nclus;
    int64_t grp = clus * per + blockIdx.x % cluster;
    const int64_t grp_end = (clus + 1) * per < wk.groups ? (clus + 1) * per : wk.groups;
    // first token's fetch goes out before anything else; the parameters load in its shadow
    if (grp < grp_end) {
        stage_issue<C, 0>(stage, x, wk, grp, tm);
        if constexpr (RESID)
            stage_issue<C, LAST>(stage_r, resid, wk, grp, tm);
    }

    float a[C::E], b[C::E];
    alpha_get<C>(a, alpha, tm);
    param_load<C>(b, beta, tm);
    RoundB<C> hb{};
    if constexpr (C::kMfma) hb = make_round_b<C>();
    wait_vmem<0>();
    for (; grp < grp_end; grp += step) {
        const bool more = grp + step < grp_end;
        uint4 raw[C::NV], rraw[RESID ? C::NV : 1];
        stage_read<C>(raw, stage);
        if constexpr (RESID) stage_read<C>(rraw, stage_r);
        if (more) {
            stage_issue<C, 0>(stage, x, wk, grp + step, tm);
            if constexpr (RESID)
                stage_issue<C, LAST>(stage_r, resid, wk, grp + step, tm);
        }
        float r[C::E];
        transform_from_raw<C, true>(r, raw, lds, tm, hb);
        if constexpr (RESID) {
            float res[C::E];
            unpack_all<C>(res, rraw);
#pragma unroll
            for (int i = 0; i < C::E; ++i) r[i] = res[i] + fmaf(r[i], a[i], b[i]);
        } else {
#pragma unroll
            for (int i = 0; i < C::E; ++i) r[i] = fmaf(r[i], a[i], b[i]);
        }
        if constexpr (STATS) token_sumsq<C>(r, wave_sums, sumsq, wk.token(grp), N, t, wk.slot, tm);
        if (more) wait_vmem<0>();
        put_output<C, LAST, THROUGH>(r, y, wk.slot, N, grp, tm);
    }
}

// A row's vectors in the layout of phase PH, straight into registers (cached loads).
template <class C, int PH>
__device__ __forceinline__ void global_get(uint4 (&raw)[C::NV], const typename C::io::elem_t* tensor,
                                           const Walker<C>& wk, int64_t grp, const ThreadMap<C>& tm) {
    const typename C::io::elem_t* row = tensor + wk.row(grp) * C::kRow;
    const unsigned next = wk.next_row(grp);
    static_for<0, C::NV>([&](auto c) {
        constexpr int Cc = decltype(c)::value;
        const typename C::io::elem_t* p = row + vector_offset<C, PH, Cc>(tm, next);
        raw[Cc] = *reinterpret_cast<const uint4*>(p);
    });
}

// Keep a value computed where it stands: the compiler otherwise sinks a sum that the loop only uses in
// its next iteration to the end of the body, and with it everything the sum is made of stays live.
template <int COUNT>
__device__ __forceinline__ void pin(float* r) {
#pragma unroll
    for (int i = 0; i < COUNT; ++i) asm volatile("" : "+v"(r[i]));
}

// forward for a few tokens (decoding, paper Sec. 5: one token per sequence and step): one token
// group (R = 2: two) per workgroup and nothing else.  With so little work a launch is one memory round trip
// long, so everything the group needs -- x, alpha, beta, the residual -- is requested at once,
// straight into registers, before anything is awaited; there is no token loop, no prefetch stage and
// no walk over the grid, whose set-up costs the persistent kernel about a microsecond per launch.
//
// The compiler places these loads by register pressure and not by time: a part of x behind the first products
// (d = 8192), the residual behind the transform, and where the store is conditional (several tokens per workgroup)
// alpha, beta and the arithmetic on them in that condition; each makes the launch another round trip longer.  A
// scheduling barrier behind x, behind x and the residual or behind all of them keeps them in front, and the results of
// a conditional store are then pinned in front of the condition.  It costs registers, and so waves, where a CU has
// several workgroups, and a wait where the products could have covered the loads.  So the place differs; this is the
// one that is no slower than the others, or by little, at few tokens and at the limit, on inputs that come back and on
// inputs from memory.  us per call under graph replay, from memory, compiler's own / x / x and residual / all in front:
//     256 wide, 512 tokens: 2.59 / 2.41 / 2.42 / 2.49, residual 3.70 / 3.04 / 2.84 / 2.95 (but 16384 tokens of 128, float32 6.94 /
//       6.56 / 7.05 / 7.04), statistic 3.07 / 3.40 / 3.07 / 3.18
//     1024 wide, 512 tokens: 2.83 / 2.97 / 2.97 / 2.94, residual 3.76 / 3.94 / 3.26 / 3.01, statistic 3.90 / 3.90 / 3.58 / 3.29
//     4096 wide, 64 tokens, residual: 3.54 / 3.54 / 3.07 / 3.48; 8192 wide, 16 tokens 4.60 / 3.96 / 3.83 / 4.24
//     6144 wide, 85 tokens: 4.30 / 4.41 / 4.41 / 4.70, residual 4.84 / 4.68 / 4.46 / 5.07; 341 of 768, statistic 5.02 / 4.54 / 3.81 / 3.51
// (profiles/wht_affine_one_pass_request_order.txt has all).
enum class Requests { kFree, kX, kInputs, kAll };
template <class C>
constexpr Requests requests_first(bool resid, bool stats) {
    const bool plain_resid = resid && !stats;
    if constexpr (C::kTwelve) return C::m == 6 ? Requests::kAll : resid && C::m < 10 ? Requests::kInputs : Requests::kFree;
    else if constexpr (C::kWave) {
        if (C::v == 3) return stats ? Requests::kFree : plain_resid && C::n == 9 ? Requests::kAll : Requests::kX;
        if (C::n <= 10) return Requests::kX;
        if (C::n == 11) return resid ? Requests::kAll : Requests::kFree;
        return C::n == 13 && plain_resid ? Requests::kInputs : Requests::kFree;
    } else {
        if (C::n == 13 || (C::n == 11 && stats)) return Requests::kX;
        if (C::n <= 11) return resid ? Requests::kAll : Requests::kFree;
        return plain_resid || (C::n == 14 && resid) ? Requests::kInputs : Requests::kFree;
    }
}
// The same where the results are written through (1 MiB and more) by R token groups per workgroup; mean over 1.5 to 6 MiB (one
// group) and 6 to 24 MiB (two) of the time before over the time with kFree / kX / kInputs / kAll: 1024 wide 0.98 0.98 0.97 1.07 and
// 1.15 1.16 1.16 1.16; 2048 wide, residual, 0.98 0.98 1.10 1.06 and 1.06 1.05 1.02 0.99; 4096 1.09 1.08 1.08 1.00; 256 wide 1.05 1.10 1.10
// 1.02; 3072 wide, two groups, 1.15 1.15 1.15 1.07, with the statistic 1.04 1.01 0.97 0.99.
template <class C>
constexpr Requests requests_first_through(bool resid, bool stats, int R) {
    if constexpr (C::kTwelve) {
        if (R == 2) return stats ? Requests::kFree : Requests::kX;
        return C::m == 6 ? Requests::kAll : C::m == 10 && !resid ? Requests::kFree : Requests::kInputs;
    } else if constexpr (C::kWave) {
        if (C::v == 3) return resid && !stats ? Requests::kInputs : Requests::kX;
        if (C::n == 11 && !resid) return Requests::kAll;
        return C::n >= 11 && resid ? Requests::kInputs : Requests::kX;
    } else {
        if (C::n == 10) return Requests::kAll;
        return R == 1 && resid ? Requests::kInputs : Requests::kX;
    }
}

// The end of one token group: the affine part, the statistic and plain stores.
template <class C, bool RESID, bool STATS, bool PIN>
__device__ __forceinline__ void once_finish(float (&r)[C::E], const uint4 (&rraw)[RESID ? C::NV : 1], const float (&a)[C::E],
                                            const float (&b)[C::E], float* wave_sums, typename C::io::elem_t* y, float* sumsq,
                                            const Walker<C>& wk, int64_t N, int64_t grp, unsigned t, const ThreadMap<C>& tm) {
    if constexpr (RESID) {
        float res[C::E];
        unpack_all<C>(res, rraw);
#pragma unroll
        for (int i = 0; i < C::E; ++i) r[i] = res[i] + fmaf(r[i], a[i], b[i]);
    } else {
#pragma unroll
        for (int i = 0; i < C::E; ++i) r[i] = fmaf(r[i], a[i], b[i]);
    }
    if constexpr (PIN) pin<C::E>(r);
    if constexpr (STATS) token_sumsq<C>(r, wave_sums, sumsq, wk.token(grp), N, t, wk.slot, tm);
    global_put<C, C::P - 1, false>(r, y, wk.slot, N, grp, tm);
}

template <class C, bool RESID, bool STATS, bool THROUGH, int R>
__global__ __launch_bounds__(C::BT) void forward_once_kernel(const typename C::io::elem_t* x,
                                                             const float* __restrict__ alpha,
                                                             const float* __restrict__ beta,
                                                             const typename C::io::elem_t* resid,
                                                             typename C::io::elem_t* y,
                                                             float* __restrict__ sumsq, int64_t N) {
    static_assert(!STATS || RESID, "the statistic belongs to the residual-stream output");
    __shared__ float wave_sums[STATS ? C::BT / 64 : 1];
    __shared__ __align__(16) float lds[C::kExchangeBytes / 4];
    constexpr int LAST = C::P - 1;
    const unsigned t = threadIdx.x % C::TPT;
    const Walker<C> wk{N, (N + C::G - 1) / C::G, threadIdx.x / C::TPT};
    ThreadMap<C> tm;
    tm.init(t, wk.slot);
    // One group with plain stores is written out, and not a turn of the loops below: in them the same statements take other registers
    // (float32 2048 wide 110 for 83, four waves per SIMD for five: 25 MiB from memory 14.8 us for 13.1).  The loops' own figures are those
    // of two groups and of stores through L2, where they are as fast as this or faster (11 MiB of float32 2048 from memory by 10 %).
    if constexpr (!THROUGH) {
        static_assert(R == 1);
        constexpr Requests FIRST = requests_first<C>(RESID, STATS);
        const int64_t grp = blockIdx.x;
        uint4 raw[C::NV], rraw[RESID ? C::NV : 1];
        global_get<C, 0>(raw, x, wk, grp, tm);                  // a ragged group re-reads the last token
        if constexpr (FIRST == Requests::kX) __builtin_amdgcn_sched_barrier(0);
        if constexpr (RESID) global_get<C, LAST>(rraw, resid, wk, grp, tm);
        if constexpr (FIRST == Requests::kInputs) __builtin_amdgcn_sched_barrier(0);
        float a[C::E], b[C::E];
        param_load<C>(a, alpha, tm);
        param_load<C>(b, beta, tm);
        if constexpr (FIRST == Requests::kAll) __builtin_amdgcn_sched_barrier(0);
        else scale_alpha<C>(a, tm);
        RoundB<C> hb{};
        if constexpr (C::kMfma) hb = make_round_b<C>();
        float r[C::E];
        transform_from_raw<C, false>(r, raw, lds, tm, hb);
        if constexpr (FIRST == Requests::kAll) scale_alpha<C>(a, tm);          // here, so that nothing before waits for alpha
        once_finish<C, RESID, STATS, (FIRST != Requests::kFree && C::G > 1)>(r, rraw, a, b, wave_sums, y, sumsq, wk, N, grp, t, tm);
    } else {
        constexpr Requests FIRST = requests_first_through<C>(RESID, STATS, R);
        uint4 raw[R][C::NV], rraw[R][RESID ? C::NV : 1];
        auto group = [&](int i) { return (int64_t)blockIdx.x + (int64_t)i * gridDim.x; };
#pragma unroll
        for (int i = 0; i < R; ++i) global_get<C, 0>(raw[i], x, wk, group(i), tm);
        if constexpr (FIRST == Requests::kX) __builtin_amdgcn_sched_barrier(0);
        if constexpr (RESID)
#pragma unroll
            for (int i = 0; i < R; ++i) global_get<C, LAST>(rraw[i], resid, wk, group(i), tm);
        if constexpr (FIRST == Requests::kInputs) __builtin_amdgcn_sched_barrier(0);
        float a[C::E], b[C::E];
        param_load<C>(a, alpha, tm);
        param_load<C>(b, beta, tm);
        if constexpr (FIRST == Requests::kAll) __builtin_amdgcn_sched_barrier(0);
        else scale_alpha<C>(a, tm);
        RoundB<C> hb{};
        if constexpr (C::kMfma) hb = make_round_b<C>();
        static_for<0, R>([&](auto rr) {
            constexpr int I = decltype(rr)::value;
            float r[C::E];
            transform_from_raw<C, I + 1 < R>(r, raw[I], lds, tm, hb);
            if constexpr (FIRST == Requests::kAll && I == 0) scale_alpha<C>(a, tm);
            if constexpr (RESID) {
                float res[C::E];
                unpack_all<C>(res, rraw[I]);
#pragma unroll
                for (int i = 0; i < C::E; ++i) r[i] = res[i] + fmaf(r[i], a[i], b[i]);
            } else {
#pragma unroll
                for (int i = 0; i < C::E; ++i) r[i] = fmaf(r[i], a[i], b[i]);
            }
            if constexpr (STATS) token_sumsq<C>(r, wave_sums, sumsq, wk.token(group(I)), N, t, wk.slot, tm);
            global_put_through<C, LAST>(r, y, wk.slot, N, group(I), tm);
        });
    }
}

// The sums of a workgroup's G token slots (in LDS, one region of kTokenWords floats each) added up, times
// `scale`, to its row: four columns per thread at a time (one where there are more threads than that), the
// slots in up to eight chains that are combined by a fixed tree (short chains: less rounding, LDS reads in
// flight).  Four columns against one, and 16-byte stores against 4-byte ones, at 32768 x 1536: 63.4 against
// 68.7 us for the call.
template <class C, bool DX>
__device__ __forceinline__ void add_token_slots(rsrc_t out, const float* slots, unsigned tid, float scale) {
    constexpr int SLOTS = C::G / C::kPair, CHAINS = SLOTS < 8 ? SLOTS : 8;
    if constexpr (C::D >= 4 * C::BT || C::kTwelve) {
        // unrolled: the reads of one pass do not wait for the stores of the one before
        constexpr int PASSES = (C::D + 4 * C::BT - 1) / (4 * C::BT);
#pragma unroll
        for (int pass = 0; pass < PASSES; ++pass) {
            const unsigned j = 4 * (tid + pass * C::BT);
            if (C::D % (4 * C::BT) != 0 && j >= (unsigned)C::D) break;
            float4 acc[CHAINS];
#pragma unroll
            for (int g = 0; g < SLOTS; ++g) {
                const float4 q = *reinterpret_cast<const float4*>(slots + g * C::kTokenWords + C::phys(j));
                acc[g % CHAINS] = g < CHAINS ? q : add4(acc[g % CHAINS], q);
            }
#pragma unroll
            for (int half = CHAINS / 2; half >= 1; half /= 2)
#pragma unroll
                for (int c = 0; c < half; ++c) acc[c] = add4(acc[c], acc[c + half]);
            put_sums<sums_policy<C, DX>()>(out, j, make_float4(acc[0].x * scale, acc[0].y * scale, acc[0].z * scale, acc[0].w * scale));
        }
    } else {
        for (unsigned j = tid; j < (unsigned)C::D; j += C::BT) {
            float acc[CHAINS];
#pragma unroll
            for (int g = 0; g < SLOTS; ++g) {
                const float q = slots[g * C::kTokenWords + C::phys(j)];
                acc[g % CHAINS] = g < CHAINS ? q : acc[g % CHAINS] + q;
            }
#pragma unroll
            for (int half = CHAINS / 2; half >= 1; half /= 2)
#pragma unroll
                for (int c = 0; c < half; ++c) acc[c] += acc[c + half];
            __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(acc[0] * scale), out, j * 4u, 0, sums_policy<C, DX>());
        }
    }
}

// A thread's sums (last layout) to its token's slot for add_token_slots.
template <class C>
__device__ __forceinline__ void sums_to_slot(const float (&acc)[C::kSums], float* slots, const ThreadMap<C>& tm) {
    if constexpr (C::kPair == 2) {                          // lanes l and l ^ 8 hold the same columns in vector 2
#pragma unroll
        for (int i = 0; i < C::V; i += 4) {
            float both[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const float v = acc[C::V + i + k];
                both[k] = v + __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x128, 0xf, 0xf, false));   // row_ror:8
            }
            *reinterpret_cast<float4*>(slots + tm.columns + i) = make_float4(acc[i], acc[i + 1], acc[i + 2], acc[i + 3]);
            if (!tm.second) *reinterpret_cast<float4*>(slots + tm.columns2 + i) = make_float4(both[0], both[1], both[2], both[3]);
        }
    } else if constexpr (C::kTwelve) {
        static_for<0, C::E / 4>([&](auto i) {
            constexpr int I = decltype(i)::value * 4, VEC = I / C::V;
            float* at = slots + (VEC == 2 ? tm.columns2 : tm.columns + VEC * 64) + I % C::V;
            *reinterpret_cast<float4*>(at) = make_float4(acc[I], acc[I + 1], acc[I + 2], acc[I + 3]);
        });
    } else {
        lds_put<C, C::P - 1>(acc, slots + tm.lds_off[C::P - 1]);
    }
}

// A thread's sums (last layout) times `scale` straight to the row, where the workgroup has one token.
template <class C, bool DX>
__device__ __forceinline__ void put_thread_sums(const float (&acc)[C::E], rsrc_t out, float scale, const ThreadMap<C>& tm) {
    static_for<0, C::E / 4>([&](auto i) {
        constexpr int I = decltype(i)::value * 4;
        put_sums<sums_policy<C, DX>()>(out, vector_offset<C, C::P - 1, I / C::V>(tm, 0u) + I % C::V,
                          make_float4(acc[I] * scale, acc[I + 1] * scale, acc[I + 2] * scale, acc[I + 3] * scale));
    });
}
// dalpha without the signs that the last layout carries in z.
template <class C>
__device__ __forceinline__ void unsign_sums(float (&da)[C::kSums], const ThreadMap<C>& tm) {
    if constexpr (C::kWave || (C::kTwelve && C::P > 1)) {
#pragma unroll
        for (int i = 0; i < C::E; ++i) da[i] *= tm.sign;
    }
}

// backward:  z = H x (recomputed);  dalpha += dy z;  dbeta += dy;  dx = H_raw((alpha/sqrt d) dy)
// Each workgroup keeps its dalpha/dbeta sums in registers and at the end writes one row of partial
// sums; reduce_partials_kernel adds the rows in a fixed order, so the result does not depend on
// scheduling.
//
// Per iteration k (x(k) and dy(k) have landed in their stages):
//   raw <- stage X;  graw <- stage DY;  issue x(k+1), dy(k+1);  z = transform(raw);  sums;
//   g = alpha' dy;  transform back;  wait for everything pending;  store dx(k).
// As in the forward kernel the single wait precedes the stores and only covers loads issued a whole
// iteration earlier (and the previous token's stores).
//
// GRADS / DX select the outputs: without GRADS x is never read and no sums are kept (dx only, the
// traffic of a forward pass); without DX nothing is transformed back or stored.  With only one of
// the two, consecutive transforms run in the same order and need the trailing barrier again.
template <class C, bool GRADS, bool DX, bool THROUGH>
__global__ __launch_bounds__(C::BT, C::kBwdWavesPerSimd) void backward_kernel(const typename C::io::elem_t* dy,
                                                         const typename C::io::elem_t* x,
                                                         const float* __restrict__ alpha,
                                                         typename C::io::elem_t* dx,
                                                         SumRows sums,
                                                         int64_t N) {
    static_assert(C::kMfma && (GRADS || DX), "matrix-core schedule; something to compute");
    __shared__ __align__(16) float lds[C::kExchangeBytes / 4];
    __shared__ __align__(16) unsigned char stage_x_buf[GRADS ? C::kStageBytes : 16];
    __shared__ __align__(16) unsigned char stage_g_buf[C::kStageBytes];
    constexpr int LAST = C::P - 1;
    constexpr bool BOTH = GRADS && DX;
    const unsigned t = threadIdx.x % C::TPT;
    Walker<C> wk{N, (N + C::G - 1) / C::G, threadIdx.x / C::TPT};
    ThreadMap<C> tm;
    tm.init(t, wk.slot);
    unsigned char* stage_x = stage_x_buf + (GRADS ? (threadIdx.x >> 6) * (C::NV * 1024) : 0);
    unsigned char* stage_g = stage_g_buf + (threadIdx.x >> 6) * (C::NV * 1024);

    const int64_t step = gridDim.x;
    int64_t grp = blockIdx.x;
    if (grp < wk.groups && wk.fetches(grp)) {
        if constexpr (GRADS) stage_issue<C, 0>(stage_x, x, wk, grp, tm);
        stage_issue<C, LAST>(stage_g, dy, wk, grp, tm);
    }

    float a[DX ? C::E : 1], da[GRADS ? C::kSums : 1], db[GRADS ? C::kSums : 1];
    if constexpr (DX) alpha_get<C>(a, alpha, tm);
    if constexpr (GRADS) {
#pragma unroll
        for (int i = 0; i < C::kSums; ++i) { da[i] = 0.0f; db[i] = 0.0f; }
    }
    const RoundB<C> hb = make_round_b<C>();
    wait_vmem<0>();
    for (; grp < wk.groups; grp += step) {
        const bool more = grp + step < wk.groups;
        uint4 raw[GRADS ? C::NV : 1], graw[C::NV];
        if constexpr (GRADS) {
            zero_missing<C>(stage_x, wk, grp, tm);
            zero_missing<C>(stage_g, wk, grp, tm);
            stage_read<C>(raw, stage_x);
        }
        stage_read<C>(graw, stage_g);
        if (more && wk.fetches(grp + step)) {
            if constexpr (GRADS)
                stage_issue<C, 0>(stage_x, x, wk, grp + step, tm);
            stage_issue<C, LAST>(stage_g, dy, wk, grp + step, tm);
        }
        float g[C::E];
        // one slot per workgroup: never ragged; two tokens per slot: zero_missing
        const bool active = C::G == 1 || C::kPair == 2 || wk.token(grp) < N;
        if constexpr (GRADS) {
            float r[C::E];
            transform_from_raw<C, !BOTH>(r, raw, lds, tm, hb);   // r = H_raw x, last layout
            unpack_all<C>(g, graw);
            // a slot of a ragged last group that has no token adds nothing, whatever its stage holds (a
            // product with zero would do for finite values only)
            if (active) {
#pragma unroll
                for (int i = 0; i < C::E; ++i) {
                    const int at = C::kPair == 2 && i >= C::V ? i - C::V : i;
                    da[at] = fmaf(g[i], r[i], da[at]);        // 1/sqrt d applied once at the end
                    db[at] += g[i];
                }
            }
        } else {
            unpack_all<C>(g, graw);
        }
        if constexpr (DX) {
#pragma unroll
            for (int i = 0; i < C::E; ++i) g[i] *= a[i];
            transform_back<C, !BOTH>(g, lds, tm, hb);    // g = H_raw(alpha' dy), first layout
            if (more) wait_vmem<0>();
            put_output<C, 0, THROUGH>(g, dx, wk.slot, N, grp, tm);
        } else {
            if (more) wait_vmem<0>();
        }
    }
    if constexpr (GRADS) {
    // Sum the G token slots of this workgroup through LDS, then write the workgroup's row.
    const float s = inv_sqrt_d<C>();
    unsign_sums<C>(da, tm);
#pragma unroll
    for (int which = 0; which < 2; ++which) {
        __syncthreads();                          // the last exchange, or the first sums, have been read everywhere
        sums_to_slot<C>(which == 0 ? da : db, lds, tm);
        __syncthreads();
        add_token_slots<C, DX>(sums.row<C>(which), lds, threadIdx.x, which == 0 ? s : 1.0f);
    }
    }   // GRADS
}

// Read COUNT (1, 2 or 4) of the staged vectors, starting with vector FIRST; reads and wait in one block.
template <class C, int FIRST, int COUNT>
__device__ __forceinline__ void stage_read_some(uint4 (&raw)[COUNT], const unsigned char* wave_slot) {
    static_assert(COUNT == 1 || COUNT == 2 || COUNT == 4, "unexpected vector count");
    const unsigned addr = lds_byte_address(wave_slot) + (threadIdx.x & 63u) * 16u;
    u32x4 v[COUNT];
    if constexpr (COUNT == 1)
        asm volatile("ds_read_b128 %0, %1 offset:%2\n\ts_waitcnt lgkmcnt(0)"
                     : "=&v"(v[0]) : "v"(addr), "n"(FIRST * 1024) : "memory");
    else if constexpr (COUNT == 2)
        asm volatile("ds_read_b128 %0, %2 offset:%3\n\tds_read_b128 %1, %2 offset:%4\n\ts_waitcnt lgkmcnt(0)"
                     : "=&v"(v[0]), "=&v"(v[1]) : "v"(addr), "n"(FIRST * 1024), "n"(FIRST * 1024 + 1024) : "memory");
    else
        asm volatile("ds_read_b128 %0, %4 offset:%5\n\tds_read_b128 %1, %4 offset:%6\n\t"
                     "ds_read_b128 %2, %4 offset:%7\n\tds_read_b128 %3, %4 offset:%8\n\ts_waitcnt lgkmcnt(0)"
                     : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]), "=&v"(v[3])
                     : "v"(addr), "n"(FIRST * 1024), "n"(FIRST * 1024 + 1024), "n"(FIRST * 1024 + 2048),
                       "n"(FIRST * 1024 + 3072) : "memory");
#pragma unroll
    for (int c = 0; c < COUNT; ++c) raw[c] = make_uint4(v[c].x, v[c].y, v[c].z, v[c].w);
    if constexpr (kPoisonLds) {
        const u32x4 nan = {0x7fc07fc0u, 0x7fc07fc0u, 0x7fc07fc0u, 0x7fc07fc0u};
#pragma unroll
        for (int c = 0; c < COUNT; ++c) {
            const unsigned a = addr + (FIRST + c) * 1024;
            asm volatile("ds_write_b128 %0, %1" : : "v"(a), "v"(nan) : "memory");
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    }
}

// The rows of one wave's tokens: a wave-uniform base and a 32-bit offset per lane, so that an address
// costs the vector unit nothing (loads and stores take base, offset and an immediate).
template <class C>
struct WaveRows {
    static constexpr int W = C::TPT < 64 ? 64 / C::TPT : 1;     // tokens per wave
    int64_t base;                                   // element index of the wave's first row (clamped to a valid row)
    unsigned rel;                                   // this lane's row from there, in elements (clamped)
    bool active;                                    // this lane's token exists
    bool any;                                       // the wave has a token (wave-uniform)
    bool whole;                                     // all W tokens of the wave exist (wave-uniform)
    __device__ __forceinline__ WaveRows(int64_t grp, int64_t N, unsigned wave, unsigned lane) {
        const int64_t tok0 = grp * C::G + (C::w > 0 ? wave >> C::w : wave * W);
        const int64_t left = N - tok0;              // tokens from the wave's first on, <= 0 past the end
        const unsigned sl = C::TPT < 64 ? lane / C::TPT : 0u;
        any = left > 0;
        whole = left >= W;
        base = (left > 0 ? tok0 : N - 1) * C::kRow;
        const unsigned last = left >= W ? W - 1 : (left > 0 ? (unsigned)left - 1u : 0u);
        rel = (sl < last ? sl : last) * C::kRow;
        active = (int64_t)sl < left;
    }
};

template <class C, int PH>
__device__ __forceinline__ void wave_issue(unsigned char* wave_slot, const typename C::io::elem_t* tensor,
                                           const WaveRows<C>& rows, unsigned thread_elem) {
    const unsigned char* base = reinterpret_cast<const unsigned char*>(tensor + rows.base);
    const unsigned off = (rows.rel + thread_elem) * (unsigned)sizeof(typename C::io::elem_t);
    static_for<0, C::NV>([&](auto c) {
        constexpr int Cc = decltype(c)::value;
        constexpr unsigned elem = reg_elem_offset(C::plan.ph[PH], C::e, Cc * C::V);
        __builtin_amdgcn_global_load_lds((global_cptr)(base + elem * sizeof(typename C::io::elem_t) + off),
                                         (lds_ptr)(wave_slot + Cc * 1024), 16, 0, kStreamPolicy);
    });
}

// Registers in the first layout -> the rows, streamed.  With global_put's 64-bit address of a row per lane the kernels for dx take 4
// to 8 registers more, and are up to 6 % slower (float32 2048 wide, 24 to 50 MiB).
template <class C>
__device__ __forceinline__ void wave_put(const float (&r)[C::E], typename C::io::elem_t* tensor, const WaveRows<C>& rows,
                                         unsigned thread_elem) {
    unsigned char* base = reinterpret_cast<unsigned char*>(tensor + rows.base);
    const unsigned off = (rows.rel + thread_elem) * (unsigned)sizeof(typename C::io::elem_t);
    if (rows.active)
        static_for<0, C::NV>([&](auto c) {
            constexpr int Cc = decltype(c)::value;
            constexpr unsigned elem = reg_elem_offset(C::plan.ph[0], C::e, Cc * C::V);
            stream_store16(base + elem * sizeof(typename C::io::elem_t) + off, C::io::pack(&r[Cc * C::V]));
        });
}

// Zeros for this lane's vectors of a wave's stage slot.
template <class C>
__device__ __forceinline__ void zero_stage(const unsigned char* wave_slot) {
    const u32x4 zero = {0u, 0u, 0u, 0u};
    const unsigned addr = lds_byte_address(wave_slot) + (threadIdx.x & 63u) * 16u;
#pragma unroll
    for (int c = 0; c < C::NV; ++c)
        asm volatile("ds_write_b128 %0, %1 offset:%2" : : "v"(addr), "v"(zero), "n"(c * 1024) : "memory");
}

// alpha' dy and the first stage back in one, on COUNT of a thread's values: a product and two multiply-adds per pair.
template <class C, int COUNT>
__device__ __forceinline__ void first_stage_back(float* r, const float* g, const float* a) {
    constexpr int Q = wave_first_back_reg<C>();
    static_assert((2 << Q) <= COUNT, "a pair lies in one piece");
#pragma unroll
    for (int i = 0; i < COUNT; ++i)
        if (!((i >> Q) & 1)) {
            const int j = i | (1 << Q);
            const float p = g[j] * a[j], q = g[i];
            r[i] = fmaf(q, a[i], p);
            r[j] = fmaf(q, a[i], -p);
        }
}

// backward of the wave schedule, which took the place of butterflies re-dealt two or three times through
// LDS per transform (two one-word passes at d = 256; one wave per SIMD waiting on conflicting LDS accesses
// at float32 d = 4096).  Bound by memory (vector issue 41 and 39 % of the SIMD cycles, no bank conflict in
// the loop): median kernel time 16384 x 4096 float32 136 us where the plain copy's rate would take 130 (was
// 181), 65537 x 256 bfloat16 19.2 us against 16 (was 27.0); a stage costs one vector instruction per value,
// between lanes as in registers.  With tokens inside a wave the four waves of a workgroup walk their
// own tokens and never wait for one another: the loop has no barrier, and the transforms touch no LDS.
// A wave past the last token therefore fetches nothing: the last row is another wave's, and that wave may
// have stored dx over it (dx may alias x or dy).
// A token of two or four waves is the workgroup's only one and has one exchange per transform.
//
// Per iteration k (x(k) and dy(k) have landed in the wave's stage slots):
//   r <- stage X;  issue x(k+1);  r = H_raw x;  dy(k) from the stage, a few vectors at a time:
//   sums, and r <- alpha' dy (and its first stage) in place of the z that has been used;  issue dy(k+1);  transform back;
//   wait for everything pending;  store dx(k).
// Taking dy in pieces keeps one set of 2^e values live besides the sums and alpha'.
template <class C, bool GRADS, bool DX, bool THROUGH>
__global__ __launch_bounds__(C::BT, C::kBwdWavesPerSimd)
void backward_wave_kernel(const typename C::io::elem_t* dy, const typename C::io::elem_t* x,
                          const float* __restrict__ alpha, typename C::io::elem_t* dx,
                          SumRows sums,
                          int64_t N) {
    static_assert(GRADS || DX, "nothing to compute");
    constexpr int LAST = C::P - 1;
    constexpr int Q = wave_first_back_reg<C>();
    // vectors of dy taken at a time: 16 values, and the pairs of the first stage back together
    constexpr int CH16 = C::NV * C::V < 16 ? C::NV : 16 / C::V, CH = CH16 * C::V < (2 << Q) ? (2 << Q) / C::V : CH16;
    // separate LDS objects where there is an exchange: its accesses then do not wait for the prefetches
    constexpr bool SPLIT = C::w > 0;
    // two-wave tokens: filled up to 64 KiB per workgroup, so that the grid's two workgroups per CU
    // cannot land as three on some CUs and one on others (135 against 139 us, 16384 x 4096 float32)
    constexpr unsigned kFill = GRADS && C::w == 1 ? 65536u - 2u * C::kStageBytes : 0u;
    __shared__ __align__(16) float lds[(kFill > C::kExchangeBytes ? kFill : C::kExchangeBytes) / 4];
    __shared__ __align__(16) unsigned char stage_buf[(GRADS && !SPLIT ? 2 : 1) * C::kStageBytes];
    __shared__ __align__(16) unsigned char stage_x_buf[GRADS && SPLIT ? C::kStageBytes : 16];
    const unsigned wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63u;
    ThreadMap<C> tm;
    tm.init(threadIdx.x % C::TPT, threadIdx.x / C::TPT);
    unsigned char* stage_g = stage_buf + wave * (C::NV * 1024);
    unsigned char* stage_x = SPLIT ? stage_x_buf + (GRADS ? wave * (C::NV * 1024) : 0)
                                   : stage_buf + (GRADS ? C::kStageBytes : 0) + wave * (C::NV * 1024);

    const int64_t groups = (N + C::G - 1) / C::G, step = gridDim.x;
    int64_t grp = blockIdx.x;
    if (grp < groups) {
        const WaveRows<C> rows(grp, N, wave, lane);
        if (rows.any) {
            if constexpr (GRADS) wave_issue<C, 0>(stage_x, x, rows, tm.first_elem);
            wave_issue<C, LAST>(stage_g, dy, rows, tm.last_elem);
        }
    }
    float a[DX ? C::E : 1], da[GRADS ? C::E : 1], db[GRADS ? C::E : 1];
    if constexpr (DX) alpha_get<C>(a, alpha, tm);      // with the sign of dx's input and of z
    if constexpr (GRADS) {
#pragma unroll
        for (int i = 0; i < C::E; ++i) { da[i] = 0.0f; db[i] = 0.0f; }
    }
    wait_vmem<0>();
    for (; grp < groups; grp += step) {
        const bool more = grp + step < groups;
        const WaveRows<C> rows(grp, N, wave, lane), next(more ? grp + step : grp, N, wave, lane);
        if (C::G > 1 && !rows.whole && !rows.active) {
            // ragged last group: zeros for the missing tokens' x and dy, so that they add nothing to the sums
            // (dy alone would do for finite x only)
            zero_stage<C>(stage_g);
            if constexpr (GRADS) zero_stage<C>(stage_x);
        }
        float r[C::E];
        if constexpr (GRADS) {
            uint4 raw[C::NV];
            stage_read<C>(raw, stage_x);
            if (more && next.any) wave_issue<C, 0>(stage_x, x, next, tm.first_elem);
            unpack_all<C>(r, raw);
            wave_transform<C, true>(r, lds, tm);
            pin<C::E>(r);
        }
        static_for<0, C::NV / CH>([&](auto c) {
            constexpr int FIRST = decltype(c)::value * CH, B = FIRST * C::V, COUNT = CH * C::V;
            uint4 graw[CH];
            stage_read_some<C, FIRST, CH>(graw, stage_g);
            float g[COUNT];
#pragma unroll
            for (int i = 0; i < CH; ++i) C::io::unpack(graw[i], &g[i * C::V]);
            if constexpr (GRADS) {
#pragma unroll
                for (int i = 0; i < COUNT; ++i) {
                    da[B + i] = fmaf(g[i], r[B + i], da[B + i]);
                    db[B + i] += g[i];
                }
                pin<COUNT>(da + B);
                pin<COUNT>(db + B);
            }
            if constexpr (DX) {
                first_stage_back<C, COUNT>(r + B, g, a + B);
                pin<COUNT>(r + B);
            }
        });
        if (more && next.any) wave_issue<C, LAST>(stage_g, dy, next, tm.last_elem);
        if constexpr (DX) {
            wave_transform<C, false, wave_first_back_bit<C>()>(r, lds, tm);
            pin<C::E>(r);
        }
        // The exchange region: with both transforms each one's put goes, thread by thread, to the words
        // that this thread's last get has read; with one alone the next put needs a barrier.
        if constexpr (C::w > 0 && GRADS != DX) exchange_barrier();
        if (more) wait_vmem<0>();
        if constexpr (DX) {
            if constexpr (THROUGH) global_put_through<C, 0>(r, dx, threadIdx.x / C::TPT, N, grp, tm);
            else wave_put<C>(r, dx, rows, tm.first_elem);
        }
    }
    if constexpr (GRADS) {
        // the token slots of the workgroup, added in slot order through LDS that is idle now
        float* slots = SPLIT ? lds : reinterpret_cast<float*>(stage_buf);
        const float s = inv_sqrt_d<C>();
#pragma unroll
        for (int which = 0; which < 2; ++which) {
            const rsrc_t row = sums.row<C>(which);
            if (which == 0) unsign_sums<C>(da, tm);
            if constexpr (C::G == 1) {                         // one token per workgroup: straight to the row
                put_thread_sums<C, DX>(which == 0 ? da : db, row, which == 0 ? s : 1.0f, tm);
                continue;
            }
            __syncthreads();
            sums_to_slot<C>(which == 0 ? da : db, slots, tm);
            __syncthreads();
            add_token_slots<C, DX>(row, slots, threadIdx.x, which == 0 ? s : 1.0f);
        }
    }
}

// One team's per-thread sums (last layout) -> the workgroup's row out[kRow], times `scale`, through `slots`
// (an idle region of G * kTokenWords floats): with one workgroup barrier, which every wave passes.
template <class C>
__device__ __forceinline__ void write_partial_row(const float (&acc)[C::E], float* slots, rsrc_t out,
                                                  float scale, unsigned tid, const ThreadMap<C>& tm) {
    sums_to_slot<C>(acc, slots, tm);
    __syncthreads();
    add_token_slots<C, true>(out, slots, tid, scale);
}

// backward (all three outputs) on three teams of waves per workgroup, 3 * C::BT threads, for the
// schedules with one LDS exchange per transform.  Wave w of every team holds the same elements of
// the token, so each SIMD runs one wave of each team and their matrix-core, vector and LDS phases
// overlap; one workgroup per CU keeps one token group per CU in flight.
//   X  waves: z = H_raw x (recomputed) and the dalpha sums
//   Y1 waves: fetch dy, the dbeta sums, alpha' dy, the stages before the exchange
//   Y2 waves: the stages after the exchange, the matrix-core rounds, store dx -- one token group
//             behind the other two teams
// Every wave passes two barriers per token group k, B1(k) and B2(k):
//   X (k) : [wait x(k); raw <- stage X; issue x(k+1); rounds; register stage; put X]  B1(k)
//           [get X; last stages; graw <- stage DY[k%2]; sums]                         B2(k)
//   Y1(k) : [wait dy(k); graw <- stage DY[k%2]; issue dy(k+1) -> DY[(k+1)%2]; sums; alpha'; stages]  B1(k)
//           [put Y]                                                                   B2(k)
//   Y2(k) : [get Y of group k-1; register stage; round 1]  B1(k)  [round 2; store dx(k-1)]  B2(k)
// and Y2 finishes the last group after the last barrier.  What the barriers order:
//   exchange region X: put before B1(k), get between B1(k) and B2(k), next put after B2(k);
//   exchange region Y: put between B1(k) and B2(k), get between B2(k) and B1(k+1);
//   stage DY[k%2]: filled by the Y1 waves' own loads (awaited before B1(k)), read by the X waves
//   between B1(k) and B2(k), refilled with dy(k+2) after B2(k).
// All teams run the same number of iterations, so they pass the same number of barriers.
// dx(k) is stored after x(k) and dy(k) have been read in full, so dx may alias either exactly.
template <class C, bool THROUGH>
__global__ __launch_bounds__(3 * C::BT) void backward_teams_kernel(const typename C::io::elem_t* dy,
                                                                   const typename C::io::elem_t* x,
                                                                   const float* __restrict__ alpha,
                                                                   typename C::io::elem_t* dx,
                                                                   SumRows sums,
                                                                   int64_t N) {
    static_assert(3 * C::BT <= 1024, "three teams must fit one workgroup");
    static_assert(C::kMfma && C::P == 2, "one exchange per transform");
    __shared__ __align__(16) float lds_x[C::kExchangeBytes / 4];
    __shared__ __align__(16) float lds_g[C::kExchangeBytes / 4];
    __shared__ __align__(16) unsigned char stage_x_buf[C::kStageBytes];
    // two buffers; at the end the dbeta sums of the token slots
    constexpr unsigned kSlotBytes = C::G / C::kPair * C::kTokenWords * 4u;
    __shared__ __align__(16) unsigned char stage_g_buf[kSlotBytes > 2u * C::kStageBytes ? kSlotBytes : 2u * C::kStageBytes];
    constexpr int LAST = 1;
    const unsigned team = threadIdx.x / C::BT;                // wave-uniform: BT is a multiple of 64
    const unsigned tid = threadIdx.x % C::BT;
    const unsigned t = tid % C::TPT;
    Walker<C> wk{N, (N + C::G - 1) / C::G, tid / C::TPT};
    ThreadMap<C> tm;
    tm.init(t, wk.slot);
    const unsigned wave_off = (tid >> 6) * (C::NV * 1024);
    unsigned char* stage_x = stage_x_buf + wave_off;
    unsigned char* stage_g0 = stage_g_buf + wave_off;
    unsigned char* stage_g1 = stage_g_buf + C::kStageBytes + wave_off;

    const int64_t step = gridDim.x;
    int64_t grp = blockIdx.x;

    if (team == 0) {
        // (before the first fetch: with it behind, the compiler waits for the prefetch at every exchange, 284 against
        // 270 us at 32768 x 8192; not so for rows of 12 * 2^m elements)
        if (C::kTwelve && grp < wk.groups) stage_issue<C, 0>(stage_x, x, wk, grp, tm);
        const RoundB<C> hb = make_round_b<C>();
        if (!C::kTwelve && grp < wk.groups) stage_issue<C, 0>(stage_x, x, wk, grp, tm);
        float da[C::E];
#pragma unroll
        for (int i = 0; i < C::E; ++i) da[i] = 0.0f;
        for (int par = 0; grp < wk.groups; grp += step, par ^= 1) {
            const bool more = grp + step < wk.groups;
            uint4 raw[C::NV], graw[C::NV];
            wait_vmem<0>();                                     // x(k) has landed
            stage_read<C>(raw, stage_x);
            if (more) stage_issue<C, 0>(stage_x, x, wk, grp + step, tm);
            float r[C::E], g[C::E];
            mfma_rounds_from_bf16<C>(r, raw, hb, tm);
            if constexpr (!C::kTwelve) run_stages<C, 0>(r);
            lds_put<C, 0>(r, lds_x + tm.lds_off[0]);
            exchange_barrier();                                 // B1(k)
            lds_get<C, LAST>(r, lds_x + tm.lds_off[LAST]);
            stage_read<C, false>(graw, par ? stage_g1 : stage_g0);     // fetched by the Y1 waves, read by both
            if constexpr (C::kTwelve) wave_bit_stages<C, false>(r, tm);
            else run_stages<C, LAST>(r);
            unpack_all<C>(g, graw);
            if (C::G == 1 || wk.token(grp) < N) {               // a ragged last group's clamped rows add nothing
#pragma unroll
                for (int i = 0; i < C::E; ++i) da[i] = fmaf(g[i], r[i], da[i]);
            }
            exchange_barrier();                                 // B2(k)
        }
        unsign_sums<C>(da, tm);
        write_partial_row<C>(da, lds_x, sums.row<C>(0), inv_sqrt_d<C>(), tid, tm);
    } else if (team == 1) {
        if (grp < wk.groups) stage_issue<C, LAST>(stage_g0, dy, wk, grp, tm);
        float a[C::E], db[C::E];
        alpha_get<C>(a, alpha, tm);
#pragma unroll
        for (int i = 0; i < C::E; ++i) db[i] = 0.0f;
        for (int par = 0; grp < wk.groups; grp += step, par ^= 1) {
            const bool more = grp + step < wk.groups;
            uint4 graw[C::NV];
            wait_vmem<0>();                                     // dy(k) has landed
            stage_read<C, false>(graw, par ? stage_g1 : stage_g0);
            if (more) stage_issue<C, LAST>(par ? stage_g0 : stage_g1, dy, wk, grp + step, tm);
            float g[C::E];
            unpack_all<C>(g, graw);
            if (C::G == 1 || wk.token(grp) < N) {               // a ragged last group's clamped rows add nothing
#pragma unroll
                for (int i = 0; i < C::E; ++i) db[i] += g[i];
            }
#pragma unroll
            for (int i = 0; i < C::E; ++i) g[i] *= a[i];
            if constexpr (C::kTwelve) wave_bit_stages<C, true>(g, tm);
            else run_stages<C, LAST>(g);
            exchange_barrier();                                 // B1(k): the Y2 waves have read token k-1
            lds_put<C, LAST>(g, lds_g + tm.lds_off[LAST]);
            exchange_barrier();                                 // B2(k)
        }
        // the stage buffers are idle now
        write_partial_row<C>(db, reinterpret_cast<float*>(stage_g_buf), sums.row<C>(1), 1.0f, tid, tm);
    } else {
        const RoundB<C> hb = make_round_b<C>();
        int64_t prev = -1;                                      // token group whose Y data is in the exchange region
        auto first_half = [&](float (&g)[C::E], Round1<C>& d1) {
            lds_get<C, 0>(g, lds_g + tm.lds_off[0]);
            if constexpr (!C::kTwelve) run_stages<C, 0>(g);
            mfma_round1_from_f32<C>(g, d1, hb);
        };
        auto second_half = [&](float (&g)[C::E], const Round1<C>& d1, int64_t grp_done) {
            mfma_round2<C>(g, d1, hb, tm);
            put_output<C, 0, THROUGH>(g, dx, wk.slot, N, grp_done, tm);
        };
        for (; grp < wk.groups; grp += step) {
            float g[C::E];
            Round1<C> d1;
            if (prev >= 0) first_half(g, d1);
            exchange_barrier();                                 // B1(k)
            if (prev >= 0) second_half(g, d1, prev);
            exchange_barrier();                                 // B2(k): token k is in the exchange region
            prev = grp;
        }
        exchange_barrier();                                     // the barrier of the other teams' row writes
        if (prev >= 0) {
            float g[C::E];
            Round1<C> d1;
            first_half(g, d1);
            second_half(g, d1, prev);
        }
    }
}

// ------------------------------------------------------------------------------------------------
// backward for a few tokens: one launch, no partial rows
//
// dalpha and dbeta are sums over all tokens, so the other kernels end in rows of partial sums and a second launch.
// Here a workgroup has 64 columns instead (a "slice") and takes every token: of z it needs the 64 values of its slice,
//     z[64 j + lo] = H_64 along lo of  sum over k of +-x[64 k + lo],   the sign that of row j, column k of H_raw's upper factor,
// one multiply-add per element of x and 64-point butterflies, and nothing of what other workgroups compute.  Every such
// workgroup reads all of x; that is the price, and why this is for calls of few elements.  Further workgroups make dx,
// one token group each.
// A wave takes every 16th token.  Its lanes hold 16-byte vectors of V elements, 64 / V lanes to the 64 columns of one k
// and V consecutive k to a load; the V k's sums of each column are then brought together, half of the values at a time, by
// lane swaps, which leaves one column per lane.
// Bound by vector issue: 18 instructions per load (bfloat16: 8 values, widen, multiply-add, sign) and about 36 per token behind them,
// on the 16 waves of one CU, 1.1 to 2 us per 2^15 to 2^16 elements; 64 columns because a line of dy has them.  The table at
// few_backward_elements (wht_affine.hip) has the times.
constexpr int kFewThreads = 1024, kFewWaves = kFewThreads / 64;

template <class C>
struct FewSlices {
    static constexpr int V = 16 / (int)sizeof(typename C::io::elem_t), LANES = 64 / V;
    static constexpr int A = C::kRow / 64;                          // slices, and values of k
    static constexpr int LOADS = (A + V - 1) / V;
    static constexpr int TOKENS = LOADS >= 8 ? 1 : LOADS >= 4 ? 2 : 4, CHUNK = LOADS < 8 ? LOADS : LOADS % 8 == 0 ? 8 : 6;
    static_assert(C::kRow % 64 == 0 && A >= V && LOADS <= 32 && LOADS % CHUNK == 0, "a load is V values of k, one sign bit each");
    // float32 rows of 2048 on add the loads of a chunk in pairs, as the butterflies do.  dalpha of one token against 64 bits, in one
    // chain over the loads / in pairs / by butterflies: 8192 wide 1.37e-7 / 1.07e-7 / 1.07e-7, 4096 1.11e-7 / 0.97e-7 / 0.97e-7, 2048
    // 1.04e-7 / 0.99e-7 / 0.98e-7; up to 1024 the chain is short (0.90e-7).  It takes half as many instructions again per load: 0.04 to 0.1 us
    // of a call.  bfloat16 keeps the chain: the kernels of more tokens carry z in two bfloat16 terms (2^-17).
    static constexpr bool PAIRS = V == 4 && LOADS >= 8;
    static_assert(!PAIRS || (CHUNK & (CHUNK - 1)) == 0, "pairs of pairs");
    // whether row j, column k of the upper factor is -1
    static __device__ __forceinline__ unsigned minus(unsigned j, unsigned k) {
        if constexpr (C::kTwelve) {
            constexpr unsigned mid = C::m - 6;
            return ((paley12_minus_row(j >> mid) >> (k >> mid)) ^ __popc(j & k & ((1u << mid) - 1u))) & 1u;
        } else return __popc(j & k) & 1u;
    }
};

// z <- its 64-point transform across the lanes of the wave.
__device__ __forceinline__ float lanes_transform(float z, unsigned lane) {
    auto dpp = [](float v, auto ctrl) {
        return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), decltype(ctrl)::value, 0xf, 0xf, false));
    };
    auto stage = [&](float partner, unsigned bit) { z = fmaf(z, lane & bit ? -1.0f : 1.0f, partner); };
    stage(dpp(z, std::integral_constant<int, 0xB1>{}), 1u);                                     // quad_perm [1,0,3,2]
    stage(dpp(z, std::integral_constant<int, 0x4E>{}), 2u);                                     // quad_perm [2,3,0,1]
    stage(dpp(dpp(z, std::integral_constant<int, 0x141>{}), std::integral_constant<int, 0x1B>{}), 4u);     // l ^ 7, then ^ 3
    stage(dpp(z, std::integral_constant<int, 0x128>{}), 8u);                                    // row_ror:8
    const auto s16 = __builtin_amdgcn_permlane16_swap(__float_as_uint(z), __float_as_uint(z), false, false);
    z = fmaf(__uint_as_float(s16[1]), lane & 16u ? -1.0f : 1.0f, __uint_as_float(s16[0]));
    const auto s32 = __builtin_amdgcn_permlane32_swap(__float_as_uint(z), __float_as_uint(z), false, false);
    return fmaf(__uint_as_float(s32[1]), lane & 32u ? -1.0f : 1.0f, __uint_as_float(s32[0]));
}

// dalpha and dbeta of slice j.
template <class C>
__device__ __forceinline__ void few_sums(const typename C::io::elem_t* dy, const typename C::io::elem_t* x, float* dalpha,
                                         float* dbeta, int64_t N, unsigned j) {
    using F = FewSlices<C>;
    using T = typename C::io::elem_t;
    __shared__ float part[2][kFewWaves][64];
    const unsigned wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63u;
    const unsigned group = lane / F::LANES;
    uint32_t minus = 0;
#pragma unroll
    for (int l = 0; l < F::LOADS; ++l) minus |= F::minus(j, l * F::V + group) << l;
    // the column that ends up in this lane
    const unsigned value = F::V == 8 ? ((lane >> 5) << 2) | (((lane >> 4) & 1u) << 1) | ((lane >> 3) & 1u)
                                     : ((lane >> 5) << 1) | ((lane >> 4) & 1u);
    const unsigned column = 64u * j + (lane % F::LANES) * F::V + value;
    float da = 0.0f, db = 0.0f;
    for (int64_t n = wave; n < N; n += kFewWaves * F::TOKENS) {
        float acc[F::TOKENS][F::V], g[F::TOKENS];
#pragma unroll
        for (int u = 0; u < F::TOKENS; ++u) {
            const int64_t tok = n + u * kFewWaves, row = (tok < N ? tok : N - 1) * C::kRow;
            if constexpr (sizeof(T) == 2) g[u] = __uint_as_float((uint32_t)dy[row + column] << 16);
            else g[u] = dy[row + column];
#pragma unroll
            for (int i = 0; i < F::V; ++i) acc[u][i] = 0.0f;
        }
#pragma unroll 1
        for (int l0 = 0; l0 < F::LOADS; l0 += F::CHUNK) {
            uint4 raw[F::TOKENS][F::CHUNK];
#pragma unroll
            for (int u = 0; u < F::TOKENS; ++u) {
                const int64_t tok = n + u * kFewWaves;
                const T* row = x + (tok < N ? tok : N - 1) * C::kRow;
#pragma unroll
                for (int l = 0; l < F::CHUNK; ++l) {
                    const unsigned at = ((l0 + l) * 64u + lane) * F::V;
                    // rows of 768: the second half of the last load lies past the row
                    raw[u][l] = F::A % F::V == 0 || at < (unsigned)C::kRow ? *reinterpret_cast<const uint4*>(row + at) : make_uint4(0u, 0u, 0u, 0u);
                }
            }
            auto sign = [&](int l) { return __uint_as_float(0x3F800000u | ((minus >> (l0 + l)) << 31)); };
#pragma unroll
            for (int u = 0; u < F::TOKENS; ++u) {
                if constexpr (F::PAIRS) {
                    float v[F::CHUNK][F::V];
#pragma unroll
                    for (int l = 0; l < F::CHUNK; ++l) C::io::unpack(raw[u][l], v[l]);
#pragma unroll
                    for (int l = 0; l < F::CHUNK; l += 2)
#pragma unroll
                        for (int i = 0; i < F::V; ++i) v[l][i] = fmaf(v[l + 1][i], sign(l + 1), v[l][i] * sign(l));
#pragma unroll
                    for (int step = 2; step < F::CHUNK; step *= 2)
#pragma unroll
                        for (int l = 0; l < F::CHUNK; l += 2 * step)
#pragma unroll
                            for (int i = 0; i < F::V; ++i) v[l][i] += v[l + step][i];
#pragma unroll
                    for (int i = 0; i < F::V; ++i) acc[u][i] += v[0][i];
                } else {
#pragma unroll
                    for (int l = 0; l < F::CHUNK; ++l) {
                        float v[F::V];
                        C::io::unpack(raw[u][l], v);
#pragma unroll
                        for (int i = 0; i < F::V; ++i) acc[u][i] = fmaf(v[i], sign(l), acc[u][i]);
                    }
                }
            }
        }
#pragma unroll
        for (int u = 0; u < F::TOKENS; ++u) {
            float (&r)[F::V] = acc[u];
#pragma unroll
            for (int i = 0; i < F::V / 2; ++i) {
                const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(r[i]), __float_as_uint(r[i + F::V / 2]), false, false);
                r[i] = __uint_as_float(sw[0]) + __uint_as_float(sw[1]);
            }
#pragma unroll
            for (int i = 0; i < F::V / 4; ++i) {
                const auto sw = __builtin_amdgcn_permlane16_swap(__float_as_uint(r[i]), __float_as_uint(r[i + F::V / 4]), false, false);
                r[i] = __uint_as_float(sw[0]) + __uint_as_float(sw[1]);
            }
            if constexpr (F::V == 8) {
                const bool upper = (lane & 8u) != 0u;
                const float keep = upper ? r[1] : r[0], send = upper ? r[0] : r[1];
                r[0] = keep + __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(send), 0x128, 0xf, 0xf, false));   // row_ror:8
            }
            const float z = lanes_transform(r[0], lane);
            if (n + u * kFewWaves < N) {
                da = fmaf(g[u], z, da);
                db += g[u];
            }
        }
    }
    part[0][wave][lane] = da;
    part[1][wave][lane] = db;
    __syncthreads();
    if (wave < 2) {
        float s[kFewWaves];
#pragma unroll
        for (int w = 0; w < kFewWaves; ++w) s[w] = part[wave][w][lane];
#pragma unroll
        for (int half = kFewWaves / 2; half >= 1; half /= 2)
#pragma unroll
            for (int w = 0; w < half; ++w) s[w] += s[w + half];
        if (wave == 0) dalpha[column] = s[0] * inv_sqrt_d<C>();
        else dbeta[column] = s[0];
    }
}

// dx of token group grp, by the first C::BT threads: the arithmetic of the other backward kernels.
template <class C>
__device__ __forceinline__ void few_dx(const typename C::io::elem_t* dy, const float* __restrict__ alpha, typename C::io::elem_t* dx,
                                       int64_t N, int64_t grp) {
    __shared__ __align__(16) float lds[C::kExchangeBytes / 4];
    constexpr int LAST = C::P - 1;
    if (threadIdx.x >= C::BT) return;               // whole waves; a barrier counts the waves that are left
    const Walker<C> wk{N, (N + C::G - 1) / C::G, threadIdx.x / C::TPT};
    ThreadMap<C> tm;
    tm.init(threadIdx.x % C::TPT, wk.slot);
    uint4 graw[C::NV];
    global_get<C, LAST>(graw, dy, wk, grp, tm);     // a ragged group re-reads the last token
    float a[C::E], r[C::E];
    alpha_get<C>(a, alpha, tm);
    unpack_all<C>(r, graw);
    if constexpr (C::kMfma) {
        const RoundB<C> hb = make_round_b<C>();
#pragma unroll
        for (int i = 0; i < C::E; ++i) r[i] *= a[i];
        transform_back<C>(r, lds, tm, hb);
    } else {
        first_stage_back<C, C::E>(r, r, a);
        wave_transform<C, false, wave_first_back_bit<C>()>(r, lds, tm);
    }
    global_put<C, 0, false>(r, dx, wk.slot, N, grp, tm);
}

// Workgroups 0 .. slices - 1: dalpha and dbeta; the others, where dx is wanted: its token groups.  dx must not lie over x or dy.
template <class C>
__global__ __launch_bounds__(kFewThreads) void backward_few_kernel(const typename C::io::elem_t* dy, const typename C::io::elem_t* x,
                                                                   const float* __restrict__ alpha, typename C::io::elem_t* dx,
                                                                   float* dalpha, float* dbeta, int64_t N) {
    if (blockIdx.x < (unsigned)FewSlices<C>::A) few_sums<C>(dy, x, dalpha, dbeta, N, blockIdx.x);
    else few_dx<C>(dy, alpha, dx, N, blockIdx.x - FewSlices<C>::A);
}

// out[which][j] = sum over rows of partials[row][which][j].  Workgroup = CG float4 columns x
// (512 / CG) row lanes: lane r adds rows r, r + lanes, ..., four requested before the first is used and
// added in pairs; the row lanes of a wave add up by butterfly shuffles, the waves' sums through LDS by a
// fixed binary tree -- one association, independent of scheduling, so the result is bit-reproducible.
// All latency: a launch, one round to memory, the tree.  Measured under graph replay (rows x d), with 1024
// threads, 8 barriers and no loads in flight ahead / now: 256 x 4096 3.15 / 2.54 us, 512 x 1024 3.04 / 2.34,
// 512 x 256 2.43 / 2.17, 256 x 8192 4.53 / 4.23.  CG: 64-byte pieces of a row while
// the grid is small, 256-byte pieces once there are enough of them (CG = 4 / 8 / 16 at 512 x 768 2.27 / 2.32
// / 2.65, at 256 x 2048 2.60 / 2.15 / 2.22, at 256 x 6144 5.89 / 3.97 / 3.73).
constexpr int kReduceThreads = 512;
constexpr int reduce_columns(int d) { return d >= 6144 ? 16 : (d >= 1024 ? 8 : 4); }

template <int CG>
__global__ __launch_bounds__(kReduceThreads) void reduce_partials_kernel(const float* __restrict__ partials,
                                                                         int rows, int d,
                                                                         float* __restrict__ dalpha,
                                                                         float* __restrict__ dbeta) {
    constexpr int LANES = kReduceThreads / CG, WAVES = kReduceThreads / 64;
    __shared__ float4 part[WAVES][CG];
    const int cg = threadIdx.x % CG, lane_row = threadIdx.x / CG;
    const int col = (blockIdx.x * CG + cg) * 4;           // first of this thread's 4 columns
    const int which = blockIdx.y;
    const float* base = partials + (size_t)which * d + (col < d ? col : 0);
    auto at = [&](int r) { return *reinterpret_cast<const float4*>(base + (size_t)r * 2 * d); };
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    int r = lane_row;
    for (; r + 3 * LANES < rows; r += 4 * LANES) {
        const float4 q0 = at(r), q1 = at(r + LANES), q2 = at(r + 2 * LANES), q3 = at(r + 3 * LANES);
        acc = add4(acc, add4(add4(q0, q1), add4(q2, q3)));
    }
    for (; r < rows; r += LANES) acc = add4(acc, at(r));
#pragma unroll
    for (int off = CG; off < 64; off <<= 1)
        acc = add4(acc, make_float4(__shfl_xor(acc.x, off), __shfl_xor(acc.y, off), __shfl_xor(acc.z, off),
                                    __shfl_xor(acc.w, off)));
    if ((threadIdx.x & 63) < CG) part[threadIdx.x >> 6][cg] = acc;
    __syncthreads();
    if (threadIdx.x < CG && col < d) {
        float4 s[WAVES];
#pragma unroll
        for (int i = 0; i < WAVES; ++i) s[i] = part[i][cg];
#pragma unroll
        for (int half = WAVES / 2; half >= 1; half /= 2)
#pragma unroll
            for (int i = 0; i < half; ++i) s[i] = add4(s[i], s[i + half]);
        *reinterpret_cast<float4*>((which == 0 ? dalpha : dbeta) + col) = s[0];
    }
}

__global__ void zero_kernel(float* a, float* b, int d) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < d) { a[i] = 0.0f; b[i] = 0.0f; }
}

}  // namespace wht
