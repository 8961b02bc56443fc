// Two kernels that write a 16-byte store's registers right behind it: the store written out, and one that the compiler knows.
#include "../../paper_2104_04731_amd/csrc/store_past.h"

using c2i8::past_v4i;

template <bool PAST>
__device__ __forceinline__ void rewrite_behind_the_store(past_v4i *out, int a)
{
    past_v4i t{a, a + 1, a + 2, a + 3};
    asm volatile("" : "+v"(t));
    if (PAST) c2i8::store_past16(reinterpret_cast<char *>(out), threadIdx.x * 16, t);
    else __builtin_nontemporal_store(t, out + threadIdx.x);
    asm volatile("v_mov_b32 %0, 0" : "+v"(t[3]));  
    asm volatile("" : "+v"(t));
    __builtin_nontemporal_store(t, out + 64 + threadIdx.x);
}

extern "C" __global__ void store_written_out(past_v4i *out, int a) { rewrite_behind_the_store<true>(out, a); }
extern "C" __global__ void store_compiled(past_v4i *out, int a) { rewrite_behind_the_store<false>(out, a); }
