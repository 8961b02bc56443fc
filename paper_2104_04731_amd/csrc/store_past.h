// Stores past the caches, and from what size of a result they pay.
#pragma once
#include <hip/hip_runtime.h>

namespace c2i8 {

// A result larger than the last-level cache (256 MB) leaves it anyway, one that fits the L2s (8 x 4 MB) beside the operands is written
// back when the kernel ends if it was not before; between the two a smaller one that is written again is still in the last-level cache.
constexpr double END_FLUSH_BYTES = 28e6;
inline bool past_caches(double bytes) { return bytes > 256e6 || bytes <= END_FLUSH_BYTES; }

// 16 bytes per lane to base + off (at any dword) past the caches.  Written out: of two stores to one address in two branches, one
// of them __builtin_nontemporal_store, the compiler makes a single plain one.  The two wait states behind it are those that a vector
// instruction has to keep before it writes the registers of a store of more than eight bytes (the compiler puts as many behind its own
// 16-byte stores): the compiler does not know that this is one.
typedef int past_v4i __attribute__((ext_vector_type(4)));
__device__ __forceinline__ void store_past16(char *base, unsigned off, past_v4i x)
{
    asm volatile("global_store_dwordx4 %0, %1, %2 nt\n\ts_nop 1" : : "v"(off), "v"(x), "s"(base) : "memory");
}

}  // namespace c2i8
