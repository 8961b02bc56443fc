// Stores past the caches, and from what size of a result they pay.
#pragma once
#include <hip/hip_runtime.h>

namespace c2i8 {

// A result larger than the last-level cache (256 MB) leaves it anyway: PAST_STREAM, non-temporal.  One that fits the L2s (8 x 4 MB) beside the
// operands is written back when the kernel ends if it was not before: PAST_THROUGH, written through to the last-level cache as it comes, where
// its reader finds it.  (Non-temporal it left that cache too, and the reader paid for what the call gained.  21 layers with results of 6 to
// 26 MB on four sets of buffers in turn, plain stores | non-temporal | through, us in the mean: the call alone 12.4 | 11.5 | 11.3; with a
// pass that reads the result behind it, requantisation 16.9 | 16.5 | 16.0, blocking 19.3 | 19.1 | 18.3, NHWC unpacking 18.1 | 19.2 | 17.2,
// int32 to float16 20.7 | 21.6 | 19.9.  On one set, which the L2s still hold a part of, unpacking is level, 17.6 | 18.0 | 17.8, up to 1.1 in
// single layers, the others as above.)  Between the two a smaller result that is written again is still in the last-level cache.  Above
// 28 MB through is up to 1.3 times non-temporal (2048 images 256 x 14 x 14 -> 512: 516 -> 625 us).
enum Past : int { PAST_NONE = 0, PAST_STREAM = 1, PAST_THROUGH = 2 };
constexpr double END_FLUSH_BYTES = 28e6;
inline Past past_caches(double bytes) { return bytes > 256e6 ? PAST_STREAM : bytes <= END_FLUSH_BYTES ? PAST_THROUGH : PAST_NONE; }

// 16 or 4 bytes per lane past the caches, to `row` + `off` bytes (any dword) behind a wave-uniform base.  As buffer stores: of two global stores
// to one address in two branches, one of them __builtin_nontemporal_store, the compiler makes a single plain one, and of a store written
// out in assembly it does not know that it is one, so that it keeps neither the wait states in front of it (five behind a vector instruction
// that wrote the base) nor those behind it (two before a vector instruction writes the registers stored).  off + row + 16 stays
// below 2^32.
typedef unsigned past_v4u __attribute__((ext_vector_type(4)));
typedef int past_v4i __attribute__((ext_vector_type(4)));
__device__ __forceinline__ __amdgpu_buffer_rsrc_t past_base(void *base)
{
    return __builtin_amdgcn_make_buffer_rsrc(base, 0, -1, 0x00027000);   // (bytes, none of them out of range)
}
template <Past HOW>
struct PastHow {   // HOW as an argument
    static constexpr Past value = HOW;
};
constexpr int past_bits(Past how) { return how == PAST_THROUGH ? 16 : 2; }   // sc1 (written through the XCD's L2), nt
template <Past HOW>
__device__ __forceinline__ void store_past16(__amdgpu_buffer_rsrc_t base, unsigned off, unsigned row, past_v4i x)
{
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(past_v4u, x), base, off, row, past_bits(HOW));
}
// The same with plain stores among the kinds.
template <Past HOW>
__device__ __forceinline__ void store_row16(__amdgpu_buffer_rsrc_t base, unsigned off, unsigned row, past_v4i x)
{
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(past_v4u, x), base, off, row, HOW == PAST_NONE ? 0 : past_bits(HOW));
}
template <Past HOW>
__device__ __forceinline__ void store_past4(__amdgpu_buffer_rsrc_t base, unsigned off, unsigned row, int x)
{
    __builtin_amdgcn_raw_buffer_store_b32((unsigned)x, base, off, row, past_bits(HOW));
}

}  // namespace c2i8
