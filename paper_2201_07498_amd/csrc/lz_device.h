// Device-side building blocks shared by the kernel sources: precision
// traits, conversions, the SplitMix64 generator, workgroup reductions and
// the fence-free "last workgroup reduces" protocol.
#pragma once

#include "lz_internal.h"

namespace lz {

// Storage type V, SpMV accumulation type A and working-vector type W.
template <int P> struct Tr;
template <> struct Tr<0> { using V = double;   using A = double; using W = double; };
template <> struct Tr<1> { using V = float;    using A = float;  using W = float; };
template <> struct Tr<2> { using V = uint16_t; using A = float;  using W = float; };

__device__ __forceinline__ double to_d(double x) { return x; }
__device__ __forceinline__ double to_d(float x) { return (double)x; }
__device__ __forceinline__ double to_d(uint16_t b) { return (double)__uint_as_float((uint32_t)b << 16); }

__device__ __forceinline__ double to_a(double x, double) { return x; }
__device__ __forceinline__ double to_a(float x, double) { return (double)x; }
__device__ __forceinline__ double to_a(uint16_t b, double) { return (double)__uint_as_float((uint32_t)b << 16); }
__device__ __forceinline__ float to_a(float x, float) { return x; }
__device__ __forceinline__ float to_a(uint16_t b, float) { return __uint_as_float((uint32_t)b << 16); }

// Round-to-nearest-even float -> bfloat16 bits (NaN stays NaN).
__device__ __forceinline__ uint16_t f32_to_bf16(float f) {
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40u);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}
template <class V> __device__ __forceinline__ V from_d(double x);
template <> __device__ __forceinline__ double from_d<double>(double x) { return x; }
template <> __device__ __forceinline__ float from_d<float>(double x) { return (float)x; }
template <> __device__ __forceinline__ uint16_t from_d<uint16_t>(double x) { return f32_to_bf16((float)x); }

// SplitMix64 (Steele, Lea, Flood 2014): output r (0-based) of the stream
// started at `seed`, and the uniform double in [0,1) from its top 53 bits.
__device__ __forceinline__ uint64_t splitmix64(uint64_t seed, uint64_t r) {
    uint64_t z = seed + (r + 1ull) * 0x9e3779b97f4a7c15ull;
    z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
    z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
    return z ^ (z >> 31);
}
__device__ __forceinline__ double u01(uint64_t seed, uint64_t r) {
    return (double)(splitmix64(seed, r) >> 11) * (1.0 / 9007199254740992.0);
}

// ------------------------------------------------------------ reductions
// Lane exchanges without LDS.  __shfl_xor moves every 32-bit word through the
// LDS crossbar (ds_bpermute); the 16 wavefronts of an orthogonalisation
// workgroup summing 8 FP64 columns that way queue for 4.1-5.3 us per launch
// (stamps of the device clock, n = 3000 to 500 000), against 0.5 us here.
// Exchanges inside a row of 16 lanes are DPP moves; those between rows are
// the row and half swaps of gfx950.
template <int CTRL> __device__ __forceinline__ uint32_t dpp_word(uint32_t x) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, 0xf, 0xf, true);
}
template <int CTRL> __device__ __forceinline__ float dpp_move(float x) {
    return __uint_as_float(dpp_word<CTRL>(__float_as_uint(x)));
}
template <int CTRL> __device__ __forceinline__ double dpp_move(double x) {
    const uint64_t u = (uint64_t)__double_as_longlong(x);
    const uint64_t lo = dpp_word<CTRL>((uint32_t)u), hi = dpp_word<CTRL>((uint32_t)(u >> 32));
    return __longlong_as_double((long long)(lo | (hi << 32)));
}
constexpr int DPP_XOR1 = 0xb1, DPP_XOR2 = 0x4e;          // quad_perm [1,0,3,2], [2,3,0,1]
constexpr int DPP_SHL4 = 0x104;                          // lane i takes lane i + 4 of its row
constexpr int DPP_ROR4 = 0x124, DPP_ROR8 = 0x128;        // lane i takes lane i - 4, i - 8 of its row, cyclic
constexpr int DPP_HALF_MIRROR = 0x141;                   // lane i takes lane 7 - i of its half row

// v of lane i plus v of lane i ^ D (D = 16 or 32), in every lane: swapping x
// with itself leaves the even rows (lower half) in one result and the odd
// rows (upper half) in the other.
template <int D> __device__ __forceinline__ void swap_word(uint32_t x, uint32_t& even, uint32_t& odd) {
    static_assert(D == 16 || D == 32, "row or half exchange");
    if constexpr (D == 16) {
        const auto r = __builtin_amdgcn_permlane16_swap(x, x, false, false);
        even = r[0];
        odd = r[1];
    } else {
        const auto r = __builtin_amdgcn_permlane32_swap(x, x, false, false);
        even = r[0];
        odd = r[1];
    }
}
template <int D> __device__ __forceinline__ float add_xor_rows(float x) {
    uint32_t a, b;
    swap_word<D>(__float_as_uint(x), a, b);
    return __uint_as_float(a) + __uint_as_float(b);
}
template <int D> __device__ __forceinline__ double add_xor_rows(double x) {
    const uint64_t u = (uint64_t)__double_as_longlong(x);
    uint32_t al, bl, ah, bh;
    swap_word<D>((uint32_t)u, al, bl);
    swap_word<D>((uint32_t)(u >> 32), ah, bh);
    return __longlong_as_double((long long)((uint64_t)al | ((uint64_t)ah << 32))) +
           __longlong_as_double((long long)((uint64_t)bl | ((uint64_t)bh << 32)));
}

// Sum over the wavefront, in every lane: pairs at distance 32, 16, 8, 4, 2, 1.
// After the first three steps a value depends on the lane mod 8 only, so the
// rotation by four lanes of a row pairs lane i with i ^ 4.
template <class T> __device__ __forceinline__ T wave_sum(T v) {
    v = add_xor_rows<32>(v);
    v = add_xor_rows<16>(v);
    v += dpp_move<DPP_ROR8>(v);
    v += dpp_move<DPP_ROR4>(v);
    v += dpp_move<DPP_XOR2>(v);
    v += dpp_move<DPP_XOR1>(v);
    return v;
}

// Largest value of the wavefront, in every lane (NaN if only NaN).
__device__ __forceinline__ double wave_max(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
    return v;
}

// Sum over the lanes i, i + CS, i + 2 CS, ... of the wavefront (pairs at
// distance CS, 2 CS, ... 32), valid in lanes i < CS.
template <int CS, class T> __device__ __forceinline__ T strided_wave_sum(T v) {
    static_assert(CS == 1 || CS == 2 || CS == 4 || CS == 8, "lanes per row group");
    if constexpr (CS <= 1) v += dpp_move<DPP_XOR1>(v);
    if constexpr (CS <= 2) v += dpp_move<DPP_XOR2>(v);
    if constexpr (CS <= 4) v += dpp_move<DPP_SHL4>(v);
    v += dpp_move<DPP_ROR8>(v);
    v = add_xor_rows<16>(v);
    return add_xor_rows<32>(v);
}

// Sum over the CS adjacent lanes of a row group (pairs at distance 1, 2, 4),
// in each of them.  After two steps a value is the same in the four lanes of a
// quad, so the half-row mirror pairs lane i with a lane holding i ^ 4's value.
template <int CS, class T> __device__ __forceinline__ T group_lane_sum(T v) {
    static_assert(CS == 1 || CS == 2 || CS == 4 || CS == 8, "lanes per row group");
    if constexpr (CS >= 2) v += dpp_move<DPP_XOR1>(v);
    if constexpr (CS >= 4) v += dpp_move<DPP_XOR2>(v);
    if constexpr (CS >= 8) v += dpp_move<DPP_HALF_MIRROR>(v);
    return v;
}

// The value of lane l (the same l in every lane).
__device__ __forceinline__ int lane_value(int x, int l) { return __builtin_amdgcn_readlane(x, l); }

// Sum over the threads of a workgroup of `nw` waves; every thread gets it.
template <class T> __device__ __forceinline__ T block_sum(T v, T* sh, int nw = BLOCK / 64) {
    v = wave_sum(v);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    T r = sh[0];
    for (int i = 1; i < nw; ++i) r += sh[i];
    return r;
}

// Cross-workgroup data inside one kernel goes through device-coherent
// accesses (they bypass the per-XCD L2 copies), so no device-wide cache
// write-back is needed to publish it.
__device__ __forceinline__ void st_dev(double* p, double v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ double ld_dev(const double* p) {
    return __hip_atomic_load(const_cast<double*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// True in exactly one workgroup: the last of `count` to arrive.  Every value
// the last workgroup reads from the others must have been written with
// st_dev and is read with ld_dev: each thread waits for its own stores to
// complete before the workgroup takes its ticket.  The ticket is reset for
// the next use.
__device__ __forceinline__ bool last_block(uint32_t* ticket, uint32_t count, int* s_flag) {
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (threadIdx.x == 0) {
        const uint32_t t = __hip_atomic_fetch_add(ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        *s_flag = (t == count - 1u);
    }
    __syncthreads();
    const bool last = *s_flag != 0;
    if (last && threadIdx.x == 0) __hip_atomic_store(ticket, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return last;
}

// Sum of x[0..cnt) (device-coherent loads) in a fixed order.
__device__ __forceinline__ double ordered_sum_dev(const double* x, int64_t cnt, double* sh) {
    double s = 0.0;
    int64_t i = threadIdx.x;
    for (; i + 3 * (int64_t)blockDim.x < cnt; i += 4 * (int64_t)blockDim.x) {
        const double a = ld_dev(x + i), b = ld_dev(x + i + blockDim.x), c = ld_dev(x + i + 2 * blockDim.x),
                     d = ld_dev(x + i + 3 * blockDim.x);
        s += ((a + b) + (c + d));
    }
    for (; i < cnt; i += blockDim.x) s += ld_dev(x + i);
    return block_sum(s, sh, blockDim.x / 64);
}

}  // namespace lz
