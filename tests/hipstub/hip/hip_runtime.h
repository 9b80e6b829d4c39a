// A device of a few megabytes on the host, for the CPU test of host_memory.h:
// the calls that file makes, and nothing else.
#pragma once
#include <cstddef>
#include <cstdlib>
#include <cstring>
#include <map>

enum hipError_t { hipSuccess, hipErrorOutOfMemory, hipErrorInvalidValue };
enum hipMemoryType { hipMemoryTypeHost, hipMemoryTypeDevice, hipMemoryTypeUnregistered };
enum hipMemcpyKind { hipMemcpyHostToDevice, hipMemcpyDeviceToHost };
enum { hipHostMallocDefault, hipEventDisableTiming };
typedef void *hipStream_t;
typedef void *hipEvent_t;
struct hipPointerAttribute_t {
    hipMemoryType type;
};

struct StubDevice {
    size_t limit = size_t(4) << 20, used = 0;
    std::map<void *, size_t> blocks;
};
inline StubDevice &stub()
{
    static StubDevice d;
    return d;
}
inline hipError_t hipMalloc(void **p, size_t n)
{
    StubDevice &d = stub();
    if (d.used + n > d.limit) return hipErrorOutOfMemory;
    *p = std::malloc(n);
    d.blocks[*p] = n;
    d.used += n;
    return hipSuccess;
}
inline hipError_t hipFree(void *p)
{
    StubDevice &d = stub();
    if (!d.blocks.count(p)) return hipErrorInvalidValue;
    d.used -= d.blocks[p];
    d.blocks.erase(p);
    std::free(p);
    return hipSuccess;
}
inline hipError_t hipHostMalloc(void **p, size_t n, unsigned) { return (*p = std::malloc(n)) ? hipSuccess : hipErrorOutOfMemory; }
inline hipError_t hipHostFree(void *p) { return std::free(p), hipSuccess; }
inline hipError_t hipSetDevice(int) { return hipSuccess; }
inline hipError_t hipGetLastError() { return hipSuccess; }
inline hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { return *e = (hipEvent_t)1, hipSuccess; }
inline hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
inline hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
inline hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
inline hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
inline hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t) { return std::memcpy(d, s, n), hipSuccess; }
inline hipError_t hipPointerGetAttributes(hipPointerAttribute_t *a, const void *) { return a->type = hipMemoryTypeUnregistered, hipSuccess; }
