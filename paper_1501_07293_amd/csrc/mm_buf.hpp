// mm_buf.hpp -- loads and stores through buffer descriptors.
#pragma once
#include "mm_common.hpp"
#include "mm_kernels.hpp"

namespace mm {

// Global memory through buffer descriptors: an offset past the end reads zero and writes
// nothing, which is what the padding half of a line and the rows and columns beyond a
// ragged edge need, without a branch (the compiler turns a conditional load into one, and
// a branch inside a radix case costs the registers of every other case).  The base has to
// be the same for the whole work-group, offsets stay below 2 GiB (kBufEnd); the launchers
// see to both.  soff is added to the offset, the same for the whole work-group: a scalar
// register, so that it costs no vector instruction.
typedef unsigned uint2v __attribute__((ext_vector_type(2)));
typedef unsigned uint4v __attribute__((ext_vector_type(4)));
constexpr unsigned kBufEnd = (unsigned)kRLineBytes, kBufNone = 0x80000000u;
constexpr int kBufRaw = 0x00020000;  // descriptor word 3: raw 32-bit data, no swizzle
using Buf = __amdgpu_buffer_rsrc_t;
__device__ inline Buf buf_of(const void* p)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)kBufEnd, kBufRaw);
}
template <typename V>
__device__ inline V buf_ld(Buf b, unsigned off, unsigned soff = 0)
{
    if constexpr (sizeof(V) == 4)
        return __builtin_bit_cast(V, __builtin_amdgcn_raw_buffer_load_b32(b, (int)off, (int)soff, 0));
    else if constexpr (sizeof(V) == 8)
        return __builtin_bit_cast(V, __builtin_amdgcn_raw_buffer_load_b64(b, (int)off, (int)soff, 0));
    else
        return __builtin_bit_cast(V, __builtin_amdgcn_raw_buffer_load_b128(b, (int)off, (int)soff, 0));
}
template <typename V>
__device__ inline void buf_st(Buf b, unsigned off, V v, unsigned soff = 0)
{
    if constexpr (sizeof(V) == 4)
        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), b, (int)off, (int)soff, 0);
    else if constexpr (sizeof(V) == 8)
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(uint2v, v), b, (int)off, (int)soff, 0);
    else
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(uint4v, v), b, (int)off, (int)soff, 0);
}

}  // namespace mm
