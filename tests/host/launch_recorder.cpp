// Stands in for the HIP runtime's launch call: nothing runs, the grid, block and LDS of the last launch and its kernel's name are kept.
#include <hip/hip_runtime.h>

#include <map>
#include <string.h>

static std::map<const void *, const char *> &names()
{
    static std::map<const void *, const char *> of;
    return of;
}

extern "C" {
int recorded[4];   // launches so far; workgroups, threads and LDS bytes of the last one
char recorded_name[512];

// what a library's kernels are called (they are registered when it is loaded, after this)
void __hipRegisterFunction(void **, const void *host, char *, const char *device, unsigned, void *, void *, void *, void *, int *) { names()[host] = device; }

hipError_t hipLaunchKernel(const void *kernel, dim3 grid, dim3 block, void **, size_t lds, hipStream_t)
{
    ++recorded[0];
    recorded[1] = (int)(grid.x * grid.y * grid.z);
    recorded[2] = (int)(block.x * block.y * block.z);
    recorded[3] = (int)lds;
    strncpy(recorded_name, names()[kernel], sizeof recorded_name - 1);
    return hipSuccess;
}
hipError_t hipFuncSetAttribute(const void *, hipFuncAttribute, int) { return hipSuccess; }
}
