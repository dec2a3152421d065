// Building blocks of the streaming walks (stream_step.h, stream_pair.h, stream_spinor.h,
// dp_walk.h): ring slots, the right-hand side of one cell, raw buffer loads and stores.
#pragma once

#include "step_body.h"

namespace phx {

// ring slot of the value that belongs to loop position t - back, ring length K
// (t and back are compile-time constants after unrolling)
template <int K>
__device__ __forceinline__ constexpr int slot(int t, int back)
{
    return ((t - back) % K + K) % K;
}

// Right-hand side of one cell from its stage argument p, the neighbour sums lr
// (x) and ud (y), the reservoir value nn and the per-cell constant kv (see
// step_stages for the formula).  Returns f and fn; IMAG (imaginary time, t -> -i tau)
// returns -i f.
template <typename R, bool RES, bool IMAG = false>
__device__ __forceinline__ void cell_rhs(const Coef<R>& c, typename cvec<R>::type p, R lrx, R lry, R udx, R udy,
                                         R nn, R pv, R kv, R& fx, R& fy, R& fn)
{
    const R rho = fma(p.x, p.x, p.y * p.y);
    R om = kv;
    if (RES) om = fma(c.grh, nn, om);
    om = fma(c.gh, rho, om);
    const R u = RES ? fma(c.half_R, nn, -c.half_gamma) : -c.half_gamma;
    const R tx = fma(c.ax, lrx, c.ay * udx);
    const R ty = fma(c.ax, lry, c.ay * udy);
    fx = fma(u, p.x, fma(om, p.y, -ty));
    fy = fma(u, p.y, fma(-om, p.x, tx));
    fn = RES ? fma(-fma(c.R_, rho, c.gamma_r), nn, pv) : R(0);
    if constexpr (IMAG) {
        const R t = fx;
        fx = fy;
        fy = -t;
    }
}

// Raw buffer stores (hardware range check: a store at an offset past the buffer's
// size is dropped), so lanes and rows that must not store take an out-of-range
// offset instead of a branch.  Offsets are in bytes; the output buffers are smaller
// than 2 GiB (enforced when the shape is chosen).
constexpr unsigned int kBufferWord3 = 0x00020000u;  // raw 32-bit data, gfx9 family
constexpr int kOutOfRange = 0x7fffffff;
constexpr int kNonTemporal = 2;  // cache-policy bit of the store

__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_of(const void* p, size_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)bytes, (int)kBufferWord3);
}

__device__ __forceinline__ void buf_store_nt(float v, __amdgpu_buffer_rsrc_t r, int off)
{
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned int, v), r, off, 0, kNonTemporal);
}
__device__ __forceinline__ void buf_store_nt(double v, __amdgpu_buffer_rsrc_t r, int off)
{
    typedef unsigned int u2 __attribute__((ext_vector_type(2)));
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u2, v), r, off, 0, kNonTemporal);
}
__device__ __forceinline__ void buf_store_nt(float2 v, __amdgpu_buffer_rsrc_t r, int off)
{
    typedef unsigned int u2 __attribute__((ext_vector_type(2)));
    __builtin_amdgcn_raw_buffer_store_b64(u2{__builtin_bit_cast(unsigned int, v.x), __builtin_bit_cast(unsigned int, v.y)},
                                          r, off, 0, kNonTemporal);
}
__device__ __forceinline__ void buf_store_nt(double2 v, __amdgpu_buffer_rsrc_t r, int off)
{
    typedef unsigned int u4 __attribute__((ext_vector_type(4)));
    const unsigned long long x = __builtin_bit_cast(unsigned long long, v.x);
    const unsigned long long y = __builtin_bit_cast(unsigned long long, v.y);
    __builtin_amdgcn_raw_buffer_store_b128(u4{(unsigned int)x, (unsigned int)(x >> 32), (unsigned int)y,
                                              (unsigned int)(y >> 32)},
                                           r, off, 0, kNonTemporal);
}

// Raw buffer loads of one element (an offset past the buffer's size reads 0).
template <typename T>
__device__ __forceinline__ T buf_load(__amdgpu_buffer_rsrc_t r, int voff, int soff);
template <>
__device__ __forceinline__ float buf_load<float>(__amdgpu_buffer_rsrc_t r, int voff, int soff)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, voff, soff, 0));
}
template <>
__device__ __forceinline__ double buf_load<double>(__amdgpu_buffer_rsrc_t r, int voff, int soff)
{
    return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, 0));
}
template <>
__device__ __forceinline__ float2 buf_load<float2>(__amdgpu_buffer_rsrc_t r, int voff, int soff)
{
    // reinterpret the loaded bits as the whole vector (a bit cast of one element of an
    // extended vector has been compiled into a copy of its first element)
    return __builtin_bit_cast(float2, __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, 0));
}
template <>
__device__ __forceinline__ double2 buf_load<double2>(__amdgpu_buffer_rsrc_t r, int voff, int soff)
{
    return __builtin_bit_cast(double2, __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, 0));
}

}  // namespace phx
