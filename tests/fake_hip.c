/* HIP runtime calls on host memory, preloaded into a child process so that the
 * library's host code (argument checks, tables, choice and shape of a launch)
 * runs on a machine without a GPU.  Kernels do not run: a launch is recorded
 * and succeeds.  fake_malloc_limit: a larger hipMalloc fails with out of
 * memory. */
#define __HIP_PLATFORM_AMD__
#include <hip/hip_runtime_api.h>
#include <stdint.h>
#include <stdlib.h>
#include <string.h>

size_t fake_malloc_limit = SIZE_MAX;
int64_t fake_mallocs, fake_copies, fake_launches;
int64_t fake_last_grid, fake_last_block, fake_last_lds;

static hipError_t last_error = hipSuccess;

static hipError_t allocate(void** p, size_t n)
{
    ++fake_mallocs;
    *p = n > fake_malloc_limit ? NULL : aligned_alloc(256, (n + 255) / 256 * 256 + 256);
    return *p ? hipSuccess : (last_error = hipErrorOutOfMemory);
}

hipError_t hipGetLastError(void)
{
    hipError_t e = last_error;
    last_error = hipSuccess;
    return e;
}

const char* hipGetErrorString(hipError_t e) { return e ? "fake error" : "no error"; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int d) { return d ? hipErrorInvalidDevice : hipSuccess; }

hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t a, int d)
{
    *v = a == hipDeviceAttributeMultiprocessorCount ? 256
                                                    : (a == hipDeviceAttributeMaxSharedMemoryPerBlock
                                                           ? 160 * 1024 : 0);
    return *v ? hipSuccess : hipErrorInvalidValue;
}

hipError_t hipMalloc(void** p, size_t n) { return allocate(p, n); }
hipError_t hipMallocAsync(void** p, size_t n, hipStream_t s) { return allocate(p, n); }
hipError_t hipFree(void* p) { free(p); return hipSuccess; }
hipError_t hipFreeAsync(void* p, hipStream_t s) { free(p); return hipSuccess; }

hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind k)
{
    ++fake_copies;
    memcpy(d, s, n);
    return hipSuccess;
}

hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind k, hipStream_t q)
{
    return hipMemcpy(d, s, n, k);
}

hipError_t hipStreamSynchronize(hipStream_t s) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned f) { *s = NULL; return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t s) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned f) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) { *e = NULL; return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned f) { *e = NULL; return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t e) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t a, hipEvent_t b) { *ms = 0; return hipSuccess; }

hipError_t hipGetSymbolAddress(void** p, const void* symbol)
{
    static char array[(4 << 20) + 256];
    *p = (void*)(((uintptr_t)array + 255) & ~(uintptr_t)255);
    return hipSuccess;
}

hipError_t hipFuncSetAttribute(const void* f, hipFuncAttribute a, int v) { return hipSuccess; }

hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void* f, int b, size_t lds)
{
    *n = 1;
    return hipSuccess;
}

static dim3 push_grid, push_block;
static size_t push_lds;
static hipStream_t push_stream;

hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t lds, hipStream_t s)
{
    push_grid = g;
    push_block = b;
    push_lds = lds;
    push_stream = s;
    return hipSuccess;
}

hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* lds, hipStream_t* s)
{
    *g = push_grid;
    *b = push_block;
    *lds = push_lds;
    *s = push_stream;
    return hipSuccess;
}

hipError_t hipLaunchKernel(const void* f, dim3 g, dim3 b, void** args, size_t lds, hipStream_t s)
{
    ++fake_launches;
    fake_last_grid = g.x;
    fake_last_block = b.x;
    fake_last_lds = (int64_t)lds;
    return hipSuccess;
}
