// Kernels that write a 16-byte store's registers right behind it, and its base right in front of it: by the store past the caches, and by one
// that the compiler makes by itself.
#include "../../paper_2104_04731_amd/csrc/store_past.h"

using c2i8::past_v4i;

template <c2i8::Past HOW>
__device__ __forceinline__ void store(char *base, unsigned off, past_v4i t)
{
    if constexpr (HOW != c2i8::PAST_NONE) c2i8::store_past16<HOW>(c2i8::past_base(base), off, 0, t);
    else __builtin_nontemporal_store(t, reinterpret_cast<past_v4i *>(base + off));
}

template <c2i8::Past HOW>
__device__ __forceinline__ void rewrite_behind_the_store(past_v4i *out, int a)
{
    past_v4i t{a, a + 1, a + 2, a + 3};
    asm volatile("" : "+v"(t));
    store<HOW>(reinterpret_cast<char *>(out), threadIdx.x * 16, t);
    asm volatile("v_mov_b32 %0, 0" : "+v"(t[3]));
    asm volatile("" : "+v"(t));
    __builtin_nontemporal_store(t, out + 64 + threadIdx.x);
}

template <c2i8::Past HOW>
__device__ __forceinline__ void write_the_base(past_v4i *out, int a)
{
    past_v4i t{a, a + 1, a + 2, a + 3};
    asm volatile("" : "+v"(t));
    unsigned long long at = reinterpret_cast<unsigned long long>(out + (threadIdx.x & ~63u));
    const unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)(at >> 32)), lo = __builtin_amdgcn_readfirstlane((unsigned)at);
    at = (unsigned long long)hi << 32 | lo;
    store<HOW>(reinterpret_cast<char *>(at), (threadIdx.x & 63) * 16, t);
}

extern "C" __global__ void rewritten_behind_past(past_v4i *out, int a) { rewrite_behind_the_store<c2i8::PAST_STREAM>(out, a); }
extern "C" __global__ void rewritten_behind_compiled(past_v4i *out, int a) { rewrite_behind_the_store<c2i8::PAST_NONE>(out, a); }
extern "C" __global__ void base_written_past(past_v4i *out, int a) { write_the_base<c2i8::PAST_STREAM>(out, a); }

// One address in three branches: the stores stay what they are.
extern "C" __global__ void three_branches(past_v4i *out, int a, int past)
{
    const past_v4i t{a, a + 1, a + 2, a + 3};
    if (past == 1) store<c2i8::PAST_STREAM>(reinterpret_cast<char *>(out), threadIdx.x * 16, t);
    else if (past == 2) store<c2i8::PAST_THROUGH>(reinterpret_cast<char *>(out), threadIdx.x * 16, t);
    else out[threadIdx.x] = t;
}
