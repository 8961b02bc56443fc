// Stores past the caches, and from what size of a result they pay.
#pragma once
#include <hip/hip_runtime.h>

namespace c2i8 {

// A result larger than the last-level cache (256 MB) leaves it anyway, one that fits the L2s (8 x 4 MB) beside the operands is written
// back when the kernel ends if it was not before; between the two a smaller one that is written again is still in the last-level cache.
constexpr double END_FLUSH_BYTES = 28e6;
inline bool past_caches(double bytes) { return bytes > 256e6 || bytes <= END_FLUSH_BYTES; }

// 16 bytes per lane past the caches, to `row` + `off` bytes (any dword) behind a wave-uniform base.  As buffer stores: of two global stores
// to one address in two branches, one of them __builtin_nontemporal_store, the compiler makes a single plain one, and of a store written
// out in assembly it does not know that it is one, so that it keeps neither the wait states in front of it (five behind a vector instruction
// that wrote the base) nor those behind it (two before a vector instruction writes the registers stored).  off + row + 16 stays below 2^32.
typedef unsigned past_v4u __attribute__((ext_vector_type(4)));
typedef int past_v4i __attribute__((ext_vector_type(4)));
__device__ __forceinline__ __amdgpu_buffer_rsrc_t past_base(void *base)
{
    return __builtin_amdgcn_make_buffer_rsrc(base, 0, -1, 0x00027000);   // (bytes, none of them out of range)
}
__device__ __forceinline__ void store_past16(__amdgpu_buffer_rsrc_t base, unsigned off, unsigned row, past_v4i x)
{
    constexpr int NT = 2;
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(past_v4u, x), base, off, row, NT);
}

}  // namespace c2i8
