// Buffer loads and stores of the streamed sweeps.  An access is at a byte offset
// from a base, within a range: loads beyond it read 0, stores are dropped, so
// rows and lanes outside the grid need no branches.  AUX: cache policy (2:
// non-temporal).
#pragma once

#include <hip/hip_runtime.h>

namespace tdp {

typedef __amdgpu_buffer_rsrc_t Rsrc;

__device__ __forceinline__ Rsrc rsrc_of(const void *p, unsigned bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, bytes, 0x00027000);
}
__device__ __forceinline__ double f64_of(unsigned lo, unsigned hi)
{
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
template <int AUX>
__device__ __forceinline__ void bload(double &v, Rsrc r, unsigned off)
{
    typedef unsigned u2 __attribute__((ext_vector_type(2)));
    const u2 w = __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, AUX);
    v = f64_of(w.x, w.y);
}
template <int AUX>
__device__ __forceinline__ void bload(float &v, Rsrc r, unsigned off)
{
    v = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, off, 0, AUX));
}
template <int AUX>
__device__ __forceinline__ void bload(double2 &v, Rsrc r, unsigned off)
{
    typedef unsigned u4 __attribute__((ext_vector_type(4)));
    const u4 w = __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, AUX);
    v.x = f64_of(w.x, w.y);
    v.y = f64_of(w.z, w.w);
}
template <int AUX>
__device__ __forceinline__ void bload(float2 &v, Rsrc r, unsigned off)
{
    typedef unsigned u2 __attribute__((ext_vector_type(2)));
    const u2 w = __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, AUX);
    v.x = __uint_as_float(w.x);
    v.y = __uint_as_float(w.y);
}
template <int AUX>
__device__ __forceinline__ void bstore(double v, Rsrc r, unsigned off)
{
    typedef unsigned u2 __attribute__((ext_vector_type(2)));
    const unsigned long long b = (unsigned long long)__double_as_longlong(v);
    const u2 w = {(unsigned)b, (unsigned)(b >> 32)};
    __builtin_amdgcn_raw_buffer_store_b64(w, r, off, 0, AUX);
}
template <int AUX>
__device__ __forceinline__ void bstore(float v, Rsrc r, unsigned off)
{
    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), r, off, 0, AUX);
}

}  // namespace tdp
