// Device helpers shared by the libechoattn kernels (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace echo {

// bf16 storage: the upper 16 bits of an IEEE float.
struct bf16_t { uint16_t bits; };

template <typename T> __device__ __forceinline__ float ld(const T *p, size_t i);
template <> __device__ __forceinline__ float ld<float>(const float *p, size_t i) { return p[i]; }
template <> __device__ __forceinline__ float ld<bf16_t>(const bf16_t *p, size_t i) {
    return __uint_as_float(static_cast<uint32_t>(p[i].bits) << 16);
}

// Four consecutive elements starting at a multiple of four (16-byte / 8-byte aligned).
__device__ __forceinline__ float4 ld4(const float *p, size_t i) {
    return *reinterpret_cast<const float4 *>(p + i);
}
__device__ __forceinline__ float4 ld4(const bf16_t *p, size_t i) {
    uint2 u = *reinterpret_cast<const uint2 *>(p + i);
    float4 r;
    r.x = __uint_as_float(u.x << 16);
    r.y = __uint_as_float(u.x & 0xffff0000u);
    r.z = __uint_as_float(u.y << 16);
    r.w = __uint_as_float(u.y & 0xffff0000u);
    return r;
}
// The same in two steps, for loads that wait in registers: four elements as they stand in memory, and their values.
template <typename T> using Raw4 = std::conditional_t<sizeof(T) == 4, float4, uint2>;
template <typename T> __device__ __forceinline__ Raw4<T> ld4_raw(const T *p, size_t i) {
    return *reinterpret_cast<const Raw4<T> *>(p + i);
}
__device__ __forceinline__ float4 value4(float4 x) { return x; }
__device__ __forceinline__ float4 value4(uint2 u) {
    asm volatile("" : "+v"(u.x), "+v"(u.y));      // the conversion stays behind whatever barrier precedes the call
    return make_float4(__uint_as_float(u.x << 16), __uint_as_float(u.x & 0xffff0000u), __uint_as_float(u.y << 16),
                       __uint_as_float(u.y & 0xffff0000u));
}

// An element as loaded, and the number it stands for, as two steps: a load that sits in a guarded branch together
// with the first operation on its value (for bf16 the shift that widens it) makes the compiler wait for the load
// inside that branch, one trip to memory per load.  The raw form is what the load instruction delivers (bf16: the
// 16 bits, zero-extended); zero stands for zero in both.
template <typename T> struct RawElem;
template <> struct RawElem<float> {
    typedef float type;
    static __device__ __forceinline__ type load(const float *p, size_t i) { return p[i]; }
    static __device__ __forceinline__ float value(type r) { return r; }
};
template <> struct RawElem<bf16_t> {
    typedef unsigned type;
    static __device__ __forceinline__ type load(const bf16_t *p, size_t i) { return p[i].bits; }
    static __device__ __forceinline__ float value(type r) { return __uint_as_float(r << 16); }
};

// Four consecutive elements of a row exactly as they were loaded: one 16- or 8-byte register group that stays
// whole from the load to pin().  The forward's row mode, for one, loads its keys under uniform branches (a wave requests only its own
// keys); if the loaded value were taken apart or converted right away, the compiler would merge those pieces with
// the other branch's zeros inside the branch and wait for every key in turn behind its load: one trip to memory per
// key instead of one for all.  pin() marks the place from where the value may be used.
// Loads need no more than the element's own alignment, so that rows of any H take the same kernels.
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));
typedef unsigned u32x2_any __attribute__((ext_vector_type(2), aligned(2)));
__device__ __forceinline__ float4 ld4_any(const float *p, size_t i) {
    const f32x4 v = *reinterpret_cast<const f32x4_any *>(p + i);
    return make_float4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ float4 ld4_any(const bf16_t *p, size_t i) {
    const u32x2 v = *reinterpret_cast<const u32x2_any *>(p + i);
    return make_float4(__uint_as_float(v.x << 16), __uint_as_float(v.x & 0xffff0000u), __uint_as_float(v.y << 16),
                       __uint_as_float(v.y & 0xffff0000u));
}
template <typename T> struct RawKey;
template <> struct RawKey<float> {
    f32x4 v;
    __device__ __forceinline__ void load(const float *p, size_t i) { v = *reinterpret_cast<const f32x4_any *>(p + i); }
    // the first n elements (any n), zeros behind them
    __device__ __forceinline__ void load_some(const float *p, int n) {
        v = f32x4{n > 0 ? p[0] : 0.f, n > 1 ? p[1] : 0.f, n > 2 ? p[2] : 0.f, n > 3 ? p[3] : 0.f};
    }
    __device__ __forceinline__ void zero() { v = f32x4{0.f, 0.f, 0.f, 0.f}; }
    __device__ __forceinline__ void pin() { asm("" : "+v"(v)); }
    __device__ __forceinline__ float4 get() const { return make_float4(v.x, v.y, v.z, v.w); }
};
template <> struct RawKey<bf16_t> {
    u32x2 v;
    __device__ __forceinline__ void load(const bf16_t *p, size_t i) { v = *reinterpret_cast<const u32x2_any *>(p + i); }
    __device__ __forceinline__ void load_some(const bf16_t *p, int n) {
        v = u32x2{(n > 0 ? (unsigned)p[0].bits : 0u) | (n > 1 ? (unsigned)p[1].bits << 16 : 0u),
                  (n > 2 ? (unsigned)p[2].bits : 0u) | (n > 3 ? (unsigned)p[3].bits << 16 : 0u)};
    }
    __device__ __forceinline__ void zero() { v = u32x2{0u, 0u}; }
    __device__ __forceinline__ void pin() { asm("" : "+v"(v)); }
    __device__ __forceinline__ float4 get() const {
        return make_float4(__uint_as_float(v.x << 16), __uint_as_float(v.x & 0xffff0000u),
                           __uint_as_float(v.y << 16), __uint_as_float(v.y & 0xffff0000u));
    }
};

// Rows of a matrix read through a buffer descriptor: element address = base + vector byte offset + scalar byte offset,
// both 32-bit, range-checked by the hardware against the n_elems elements the descriptor covers (a load past them
// returns zero).  The descriptor's last word is the raw 32-bit data format of this architecture family.
template <typename T> struct BufferRows {
    __amdgpu_buffer_rsrc_t rsrc;
    __device__ __forceinline__ BufferRows(const T *base, unsigned n_elems)
        : rsrc(__builtin_amdgcn_make_buffer_rsrc(const_cast<T *>(base), 0, (int)(n_elems * (unsigned)sizeof(T)),
                                                  0x00020000)) {}
    // the element as loaded (16-bit types: the bits, zero-extended); value() turns it into the number.  Two steps so
    // that nothing but the load sits where the loads are issued (an operation on the loaded value there makes the
    // compiler wait for every load in turn)
    using Raw = std::conditional_t<sizeof(T) == 4, float, unsigned short>;
    __device__ __forceinline__ Raw load_raw(unsigned v_off, unsigned s_off) const {
        if constexpr (sizeof(T) == 4) {
            return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rsrc, v_off, s_off, 0));
        } else {
            return __builtin_amdgcn_raw_buffer_load_b16(rsrc, v_off, s_off, 0);
        }
    }
    // four consecutive elements (16 or 8 bytes)
    __device__ __forceinline__ Raw4<T> load4_raw(unsigned v_off, unsigned s_off) const {
        if constexpr (sizeof(T) == 4) {
            return __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, v_off, s_off, 0));
        } else {
            return __builtin_bit_cast(uint2, __builtin_amdgcn_raw_buffer_load_b64(rsrc, v_off, s_off, 0));
        }
    }
    // (16-bit types: the empty statement keeps the conversion behind whatever barrier precedes the call)
    static __device__ __forceinline__ float value(Raw raw) {
        if constexpr (sizeof(T) == 4) {
            return raw;
        } else {
            asm volatile("" : "+v"(raw));
            return __uint_as_float((unsigned)raw << 16);
        }
    }
};

// Non-temporal loads, for inputs read once by the whole grid.  Measured: they help the LSTM block (nine input and
// output streams at once, 180 -> 170 us) and hurt a single-stream copy (76 -> 93 us), so only the former uses them
// (in the recompute kernel they cost 1 to 8 %).
__device__ __forceinline__ float4 load4_streaming(const float *p) {
    typedef float f4 __attribute__((ext_vector_type(4)));
    const f4 v = __builtin_nontemporal_load(reinterpret_cast<const f4 *>(p));
    return make_float4(v.x, v.y, v.z, v.w);
}
// Stores of results that this kernel does not read again go out as non-temporal (streaming) stores: they do not
// stay behind as dirty lines for the end of the kernel to write back, which measured 0.3 to 0.6 us per kernel at
// the smallest benchmark workload and 5 % of a pure streaming kernel.
__device__ __forceinline__ void store_streaming(float *p, float x) { __builtin_nontemporal_store(x, p); }
__device__ __forceinline__ void store4_streaming(float *p, float4 x) {
    typedef float f4 __attribute__((ext_vector_type(4)));
    __builtin_nontemporal_store((f4){x.x, x.y, x.z, x.w}, reinterpret_cast<f4 *>(p));
}

// tanh(x) = 1 - 2 / (exp(2x) + 1).  With s = 2*log2(e)*x this is
// 1 - 2*rcp(exp2(s) + 1); exp2 -> inf gives 1, exp2 -> 0 gives -1, no NaN.
constexpr float kTwoLog2e = 2.8853900817779268f;

// exp(2(q+k)) = exp(2q) * exp(2k): the exponentials are taken once per row
// element and the inner loop needs one multiply-add and one reciprocal.  The
// factors stay finite and normal while |x| <= kFactorLimit (|s| <= 115.4), and
// their product then overflows to inf or underflows to 0 exactly where tanh
// has saturated, never to NaN.  Rows with a larger |x| take the exact path,
// which exponentiates the sum.
constexpr float kFactorLimit = 40.0f;

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ __forceinline__ float fast_rcp(float x) { return __builtin_amdgcn_rcpf(x); }

// r = 1 / (exp(2x) + 1) from the two factors:  tanh = 1 - 2r,  1 - tanh^2 = 4 r (1 - r).
__device__ __forceinline__ float r_from_factors(float eq, float ek) {
    return fast_rcp(__builtin_fmaf(eq, ek, 1.0f));
}
// same from the scaled pre-activations sq = c*q, sk = c*k (exact path)
__device__ __forceinline__ float r_from_sum(float sq, float sk) {
    return fast_rcp(fast_exp2(sq + sk) + 1.0f);
}

// A batch of transcendental instructions (reciprocals, exponentials) between these two goes before whatever the other waves of the
// SIMD have to issue.  Measured on small kernels of nothing but the loop bodies, four waves on a SIMD: a
// transcendental instruction holds the vector unit for 8.1 clocks, a plain one takes 2.1 as long as two waves have plain ones to
// issue, but 2.7 to 5.5 next to waves with transcendental ones.  Waves left to themselves drift into that interleaving; with the batches in
// front they run them back to back and then share the plain instructions: the forward's tanh, half a reciprocal each, 12.7 -> 10.0
// clocks per evaluation and wave, the recomputation's 26.0 -> 20.4 (plain instructions in front instead: 12.7 and 28.4).  The
// fences keep the batch between the two priority changes.
__device__ __forceinline__ void trans_begin() {
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_setprio(1);
    __builtin_amdgcn_sched_barrier(0);
}
__device__ __forceinline__ void trans_end() {
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_setprio(0);
    __builtin_amdgcn_sched_barrier(0);
}

__device__ __forceinline__ int lane_id() { return threadIdx.x & 63; }
__device__ __forceinline__ int wave_id() { return __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); }

// Reductions over the 64 lanes, result in every lane.  Within a row of 16 lanes the partners are reached with DPP
// (two quad permutations, then the two mirror patterns); the four row results are then read as scalars.  A dozen
// full-rate instructions, where six general shuffles would each take a trip through the LDS crossbar.
template <int CTRL> __device__ __forceinline__ float dpp_get(float x) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xf, 0xf, false));
}
template <int CTRL> __device__ __forceinline__ uint32_t dpp_get_u32(uint32_t x) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, 0xf, 0xf, false);
}
__device__ __forceinline__ float lane_value(float x, int l) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), l));
}
__device__ __forceinline__ float wave_sum(float x) {
    x += dpp_get<0xB1>(x);      // quad_perm [1,0,3,2]
    x += dpp_get<0x4E>(x);      // quad_perm [2,3,0,1]
    x += dpp_get<0x141>(x);     // row_half_mirror
    x += dpp_get<0x140>(x);     // row_mirror
    return (lane_value(x, 0) + lane_value(x, 16)) + (lane_value(x, 32) + lane_value(x, 48));
}
__device__ __forceinline__ float wave_max(float x) {
    x = fmaxf(x, dpp_get<0xB1>(x));
    x = fmaxf(x, dpp_get<0x4E>(x));
    x = fmaxf(x, dpp_get<0x141>(x));
    x = fmaxf(x, dpp_get<0x140>(x));
    return fmaxf(fmaxf(lane_value(x, 0), lane_value(x, 16)), fmaxf(lane_value(x, 32), lane_value(x, 48)));
}

// ---------------------------------------------------------------------------
// Sum N per-lane arrays over the 64 lanes of a wave at a cost of about one
// exchange per value instead of six.  At each level a lane keeps one half of
// its values and hands the other half to the partner lane `OFF` away (levels
// 32 and 16 with the gfx950 lane-swap instructions, 8 and 4 with DPP row
// shifts selected by bank masks, 2 and 1 with quad permutations); once one value is left the group of
// lanes that shares it is summed with quad permutations and the two mirror patterns (and, for N < 8, lane swaps
// of a value with itself).  On return lane l holds in a[0] the full sum of value
// number l / (64 / N).  N is a power of two <= 64; the order of additions is fixed.
template <int CTRL, int BANK_MASK, bool BOUND>
__device__ __forceinline__ float dpp_mov(float old, float src) {
    return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(old), __float_as_int(src), CTRL, 0xf, BANK_MASK, BOUND));
}

// x = value kept by lanes whose bit OFF is 0, y = value kept by the others.
template <int OFF>
__device__ __forceinline__ float transpose_pair(float x, float y, int lane) {
    if constexpr (OFF == 32) {
        auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false, false);
        return __uint_as_float(r[0]) + __uint_as_float(r[1]);
    } else if constexpr (OFF == 16) {
        auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(y), false, false);
        return __uint_as_float(r[0]) + __uint_as_float(r[1]);
    } else if constexpr (OFF == 8 || OFF == 4) {
        constexpr int SHL = 0x100 + OFF, SHR = 0x110 + OFF;     // row_shl:OFF / row_shr:OFF
        constexpr int LO_BANKS = OFF == 8 ? 0x3 : 0x5;           // lanes of a row whose bit OFF is 0
        const float t_lo = x + dpp_mov<SHL, 0xf, true>(0.f, x);  // x[l] + x[l + OFF]   (right where bit OFF is 0)
        const float t_hi = y + dpp_mov<SHR, 0xf, true>(0.f, y);  // y[l] + y[l - OFF]   (right where bit OFF is 1)
        return dpp_mov<0xE4, LO_BANKS, false>(t_hi, t_lo);       // identity move into the low banks only
    } else {                                                     // partner inside the quad: one quad permutation
        static_assert(OFF == 2 || OFF == 1, "lane offsets are powers of two below 64");
        const bool hi = (lane & OFF) != 0;
        const float keep = hi ? y : x;
        const float send = hi ? x : y;
        return keep + dpp_get<OFF == 2 ? 0x4E : 0xB1>(send);
    }
}

template <int N, int OFF>
struct TransposeSumStep {
    template <int M>
    static __device__ __forceinline__ void run(float (&a)[M], int lane) {
        if constexpr (N == 1) {      // one value left: sum over the group of 2 OFF lanes that share it
            a[0] += dpp_get<0xB1>(a[0]);                              // lanes l ^ 1
            if constexpr (OFF >= 2) a[0] += dpp_get<0x4E>(a[0]);      // l ^ 2: the quad
            if constexpr (OFF >= 4) a[0] += dpp_get<0x141>(a[0]);     // mirror in the half row: the other quad
            if constexpr (OFF >= 8) a[0] += dpp_get<0x140>(a[0]);     // mirror in the row: the other half
            if constexpr (OFF >= 16) a[0] = transpose_pair<16>(a[0], a[0], lane);   // the neighbouring row
            if constexpr (OFF >= 32) a[0] = transpose_pair<32>(a[0], a[0], lane);   // the other half of the wave
        } else {
            constexpr int half = N / 2;
#pragma unroll
            for (int k = 0; k < half; ++k) a[k] = transpose_pair<OFF>(a[k], a[k + half], lane);
            if constexpr (OFF > 1) TransposeSumStep<half, OFF / 2>::run(a, lane);
        }
    }
};

template <int N>
__device__ __forceinline__ float wave_transpose_sum(float (&a)[N]) {
    static_assert(N >= 1 && N <= 64 && (N & (N - 1)) == 0, "N must be a power of two <= 64");
    TransposeSumStep<N, 32>::run(a, lane_id());
    return a[0];
}

// The same within groups of G lanes: lane l of a group ends with the sums of values (N / G) l .. in a[0 .. N / G - 1], or, where
// N < G, of value l / (G / N) in a[0].
template <int N, int G>
__device__ __forceinline__ void group_transpose_sum(float (&a)[N]) {
    static_assert(N >= 1 && N <= 64 && (N & (N - 1)) == 0 && (G == 16 || G == 32 || G == 64), "powers of two");
    TransposeSumStep<N, G / 2>::run(a, lane_id());
}

__device__ __forceinline__ f32x4 mfma16(float a, float b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// Barrier for data exchanged through LDS only: waits for this wave's LDS operations, not for its global
// loads and stores (__syncthreads() would also wait for every prefetch and store in flight).
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// Accesses that other blocks of the same launch must see (or that must see theirs): device-scope relaxed
// atomics, which go through to the memory side of the per-XCD L2 caches instead of staying in one of them.
// Ordering between them is the program order of the issuing wave plus an explicit wait on the memory counter.
__device__ __forceinline__ void store_agent(float *p, float x) {
    __hip_atomic_store(p, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float load_agent(const float *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void store_agent(unsigned long long *p, unsigned long long x) {
    __hip_atomic_store(p, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned long long load_agent(const unsigned long long *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void wait_all_memory_ops() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }
// A wait on another block's flag gives up after this many ticks of the 100 MHz wall clock (2 s), so that every
// wave ends whatever happens; the results of that launch are then marked invalid (NaN).
constexpr long long kSpinLimitTicks = 200000000LL;

__device__ __forceinline__ int clamp_len(int len, int Tk) { return len < 0 ? 0 : (len > Tk ? Tk : len); }

// n items dealt to the 8 waves of a block as contiguous ranges of n / 8 or n / 8 + 1 items: first item of wave w
// (w = 8 gives n).  Waves w and w + 4 run on the same SIMD, so the n % 8 longer ranges go to waves
// 0, 5, 2, 7, 4, 1, 6, 3 in that order: the SIMDs' totals then differ by at most one item, where the plain
// floor(n w / 8) split would hand both longer ranges of n % 8 == 2 to one SIMD.
__device__ __forceinline__ int deal8_begin(int n, int w) {
    // byte e: bit w set if wave w gets a longer range when n % 8 == e (0x00, 0x01, 0x21, 0x25, 0xa5, 0xb5, 0xb7,
    // 0xf7).  Packed into one immediate: as an array the table sits in memory, and the scalar load that fetches
    // it is a trip to memory at the start of a block, right in front of the loads that depend on the ranges.
    constexpr unsigned long long kLonger = 0xf7b7b5a525210100ull;
    const unsigned m = (unsigned)(kLonger >> (8 * (n & 7))) & 0xffu;
    return (n >> 3) * w + __builtin_popcount(m & ((1u << w) - 1u));
}

// Parts of a sum handed by the blocks of a launch to the one that adds them, without a launch of its own: a part is written
// through, its arrival awaited, then flagged with the launch's number; the block that adds, which must have been dispatched
// after all that send, polls the flags (any initial state), reads the parts and sets the flags back to zero, so that a
// captured launch, whose number is fixed, can be replayed.  (A release fence would make every block wait for its XCD's L2 to
// write back everything; slots that carry the number next to every value need no wait at the sender but measured slower, 21.4
// -> 24.0 us per recompute launch at B = 64: four times the bytes, all of them polled past the L2.)
// Sender: the first wave of its block; `on`: this lane has a part.
__device__ __forceinline__ void send_part(float *part, float x, bool on, unsigned long long *flag, unsigned long long epoch) {
    if (on) store_agent(part, x);
    wait_all_memory_ops();
    if (lane_id() == 0) store_agent(flag, epoch);
}
// Receiver: all W waves of a block.  Parts p = 0 .. n - 1 of column h at parts[p * H + h], flagged by flags[p]; skip(p): part p is
// not sent.  HW columns per block: lanes past HW take parts of their own.  Every lane adds its parts in order, then lane groups
// and waves are added in order.  The result is in lanes < HW of wave 0, NaN if a part did not arrive within kSpinLimitTicks.
// s_sum: 64 W floats; s_seen: W words.
template <int HW, int W, typename Skip>
__device__ __forceinline__ float sum_parts(const float *parts, unsigned long long *flags, int n, int H, int h,
                                           unsigned long long epoch, Skip skip, float *s_sum, int *s_seen) {
    constexpr int THREADS = 64 * W, NS = 64 / HW, STEP = W * NS;
    const int lane = lane_id(), w = wave_id();
    const long long t0 = wall_clock64();
    bool seen = true;
    for (int p = threadIdx.x; p < n; p += THREADS) {
        if (skip(p)) continue;
        while (load_agent(&flags[p]) != epoch) {
            __builtin_amdgcn_s_sleep(4);
            if (wall_clock64() - t0 > kSpinLimitTicks) {
                seen = false;
                break;
            }
        }
    }
    const int wave_seen = __all(seen) ? 1 : 0;
    if (lane == 0) s_seen[w] = wave_seen;
    lds_barrier();
    bool all_seen = true;
#pragma unroll
    for (int k = 0; k < W; ++k) all_seen = all_seen && s_seen[k] != 0;
    float sum = 0.f;
    if (h < H && all_seen) {
        for (int p0 = w * NS + lane / HW; p0 < n; p0 += 8 * STEP) {
            float x[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int p = p0 + STEP * u;
                x[u] = p < n && !skip(p) ? load_agent(&parts[(size_t)p * H + h]) : 0.f;
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) sum += x[u];
        }
    }
    s_sum[w * 64 + lane] = sum;
    lds_barrier();
    float tot = 0.f;
    if (w == 0 && lane < HW) {
        for (int k = 0; k < W; ++k)
#pragma unroll
            for (int g = 0; g < NS; ++g) tot += s_sum[k * 64 + g * HW + lane];
        if (!all_seen) tot = __builtin_nanf("");            // make the failure visible
    }
    for (int p = threadIdx.x; p < n; p += THREADS) store_agent(&flags[p], 0ull);
    return tot;
}

}  // namespace echo
