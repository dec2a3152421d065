// Building blocks of the walks with two columns per lane: 16- and 8-byte buffer accesses,
// and the pin that keeps a value where it is formed.
#pragma once

#include "stream_body.h"

namespace phx {

typedef float wf4 __attribute__((ext_vector_type(4)));
typedef float wf2 __attribute__((ext_vector_type(2)));
typedef unsigned int wu4 __attribute__((ext_vector_type(4)));
typedef unsigned int wu2 __attribute__((ext_vector_type(2)));

// Forms the value here: without this the compiler moves sums that only a later position
// reads to that position, where their operands then stay live as well.
__device__ __forceinline__ void keep_here(float& v) { asm volatile("" : "+v"(v)); }
__device__ __forceinline__ void keep_here(double& v) { asm volatile("" : "+v"(v)); }
__device__ __forceinline__ void keep_here(float2& v) { asm volatile("" : "+v"(v.x), "+v"(v.y)); }
__device__ __forceinline__ void keep_here(double2& v) { asm volatile("" : "+v"(v.x), "+v"(v.y)); }

// Moves a value that is constant over the walk to accumulation registers, where it stays to
// its next use.  The walks with one wave per SIMD have room there; left to itself the
// compiler keeps two or three such values in scratch memory and reads them at every position
// (driven complex128 pairs with zero boundaries, 2048^2: 86 us per step, parked 54).
__device__ __forceinline__ void park(double& v)
{
    const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
    int lo = (int)b, hi = (int)(b >> 32);
    asm volatile("" : "+a"(lo), "+a"(hi));
    v = __builtin_bit_cast(double, ((unsigned long long)(unsigned)hi << 32) | (unsigned)lo);
}

__device__ __forceinline__ wf4 wload4(__amdgpu_buffer_rsrc_t r, int voff, int soff)
{
    return __builtin_bit_cast(wf4, __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, 0));
}
__device__ __forceinline__ wf2 wload2(__amdgpu_buffer_rsrc_t r, int voff, int soff)
{
    return __builtin_bit_cast(wf2, __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, 0));
}
// The pair of complex values a lane stores per row: one 128-bit store whose whole
// offset (column and row) is in the VGPR operand.  With the row offset in the scalar
// operand instead, the compiler puts no wait state between the store and a following
// VALU write to its data registers, and on gfx950 such a write can reach the data
// while the store still reads it (the stored row then holds wrong values in the last
// four lanes of some 16-lane rows); with a constant scalar offset it keeps the wait
// state.  The sum is formed unsigned: a masked lane's offset (kOutOfRange) plus a row
// offset below 2 GiB stays out of range and never wraps.
__device__ __forceinline__ void wstore4(wf4 v, __amdgpu_buffer_rsrc_t r, int voff, int soff)
{
    const int off = (int)((unsigned)voff + (unsigned)soff);
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(wu4, v), r, off, 0, kNonTemporal);
}
__device__ __forceinline__ void wstore2(wf2 v, __amdgpu_buffer_rsrc_t r, int voff, int soff)
{
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(wu2, v), r, voff, soff, kNonTemporal);
}

}  // namespace phx
