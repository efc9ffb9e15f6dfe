// Device helpers shared by the kernel files: address-space pointers, coherent
// accesses, the fixed-order workgroup reduction and the XCD-aware item split.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace jac {

namespace {

// Pointer into global (device) memory: lets the compiler emit global_* loads.
template <typename V>
using gptr = __attribute__((address_space(1))) V*;
// Pointer into memory no workgroup writes during the launch (the tile and
// slice layout): wave-uniform reads through it become scalar loads.
template <typename V>
using cptr = __attribute__((address_space(4))) V*;

// Coherent (device-wide) relaxed accesses for the few words workgroups of one
// persistent launch exchange; no cache-wide maintenance is implied.
__device__ __forceinline__ int32_t ld_dev(const int32_t* p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ double ld_dev(const double* p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_dev(int32_t* p, int32_t v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_dev(double* p, double v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Plain or coherent access, chosen at compile time.
template <bool DEV, typename V>
__device__ __forceinline__ V ldv(const V* p)
{
    if constexpr (DEV) return ld_dev(p);
    else return *p;
}
template <bool DEV, typename V>
__device__ __forceinline__ void stv(V* p, V v)
{
    if constexpr (DEV) st_dev(p, v);
    else *p = v;
}

__device__ __forceinline__ double maxnan(double a, double b)
{
    return (b > a || b != b) ? b : a;
}

// The value of lane i ^ OFF, for values already equal across the lanes that
// the offsets above OFF combine (a butterfly from 32 down): halves and rows
// swap by permlane, inside a row of 16 a rotation by OFF reaches the same
// value.  Vector instructions only: a butterfly step through LDS (ds_bpermute)
// waits some 130 cycles, these about 10.
template <int OFF>
__device__ __forceinline__ uint32_t lane_xor32(uint32_t x)
{
    if constexpr (OFF == 32) {
        const auto r = __builtin_amdgcn_permlane32_swap(x, x, false, false);
        return (__lane_id() & 32) ? r[0] : r[1];
    } else if constexpr (OFF == 16) {
        const auto r = __builtin_amdgcn_permlane16_swap(x, x, false, false);
        return (__lane_id() & 16) ? r[0] : r[1];
    } else {
        return (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0x120 + OFF, 0xf, 0xf, false);   // row_ror:OFF
    }
}
template <int OFF>
__device__ __forceinline__ double lane_xor(double v)
{
    const uint64_t u = (uint64_t)__double_as_longlong(v);
    const uint32_t lo = lane_xor32<OFF>((uint32_t)u), hi = lane_xor32<OFF>((uint32_t)(u >> 32));
    return __longlong_as_double((long long)((uint64_t)hi << 32 | lo));
}
template <bool MAX, int OFF, int NRHS>
__device__ __forceinline__ void wave_step(double (&v)[NRHS])
{
#pragma unroll
    for (int c = 0; c < NRHS; ++c) {
        const double o = lane_xor<OFF>(v[c]);
        v[c] = MAX ? maxnan(v[c], o) : v[c] + o;
    }
}
template <bool MAX, int NRHS>
__device__ __forceinline__ void wave_reduce(double (&v)[NRHS])
{
    wave_step<MAX, 32>(v);
    wave_step<MAX, 16>(v);
    wave_step<MAX, 8>(v);
    wave_step<MAX, 4>(v);
    wave_step<MAX, 2>(v);
    wave_step<MAX, 1>(v);
}
// Reduce NRHS values over the wavefront, in every lane, in a fixed order.
template <int NRHS>
__device__ __forceinline__ void wave_reduce(double (&v)[NRHS], bool is_max)
{
    if (is_max) wave_reduce<true>(v);
    else wave_reduce<false>(v);
}

// Reduce NRHS values over the workgroup in a fixed order; result in thread 0.
template <int NRHS>
__device__ __forceinline__ void block_reduce(double (&v)[NRHS], bool is_max, double* red)
{
    wave_reduce(v, is_max);
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, nw = blockDim.x >> 6;
    if (lane == 0) {
#pragma unroll
        for (int c = 0; c < NRHS; ++c) red[wave * NRHS + c] = v[c];
    }
    __syncthreads();
    if (threadIdx.x == 0) {
#pragma unroll
        for (int c = 0; c < NRHS; ++c) {
            double a = red[c];
            for (int w = 1; w < nw; ++w) a = is_max ? maxnan(a, red[w * NRHS + c]) : a + red[w * NRHS + c];
            v[c] = a;
        }
    }
    __syncthreads();
}

// Items [0,T) shared by G workgroups, XCD-aware.  Workgroup ids are dealt to
// the 8 XCDs round-robin, so XCD x holds workgroups x, x+8, ...; each XCD gets
// one contiguous block of items (sizes differing by at most one, the same
// split as its workgroup count when G == T, so then every workgroup gets
// exactly one item) and neighbouring tiles, which share x halos, meet in the
// same L2.
__device__ __forceinline__ void xcd_items(int32_t T, int32_t G, int32_t wg, int32_t& first, int32_t& end,
                                          int32_t& stride)
{
    if (G < 8) {
        first = wg; end = T; stride = G;
        return;
    }
    const int32_t x = wg & 7, l = wg >> 3;
    const int32_t gx = (G - x + 7) >> 3;                  // workgroups on this XCD
    const int32_t q = T >> 3, r = T & 7;
    const int32_t s0 = x * q + min(x, r);
    first = s0 + l;
    end = s0 + q + (x < r ? 1 : 0);
    stride = gx;
}

}  // namespace

}  // namespace jac
