// A stand-in for the HIP runtime on the CPU, loaded in front of the real one: device memory is
// host address space, kernels do nothing, and a test decides how much memory there is and
// whether waits and frees are refused (as they are while a stream is captured).  Fresh
// memory reads as floats of 1.
#include <stdint.h>
#include <string.h>
#include <sys/mman.h>

#include <map>

static std::map<void *, size_t> live;
static size_t bytes_live, bytes_limit = ~(size_t)0;
static int refuse_wait, refuse_free, mallocs, frees, last_error;
static size_t big;  // allocations of at least this many bytes are counted
static const int kOutOfMemory = 2, kCaptureUnsupported = 900;

static int result(int e)
{
    if (e)
        last_error = e;
    return e;
}

extern "C" {
void fake_limit(size_t n) { bytes_limit = n; }
size_t fake_live_bytes() { return bytes_live; }
void fake_refuse(int wait, int free_) { refuse_wait = wait, refuse_free = free_; }
void fake_count(size_t at_least) { big = at_least, mallocs = frees = 0; }
int fake_mallocs() { return mallocs; }
int fake_frees() { return frees; }

int hipMalloc(void **p, size_t n)
{
    const size_t size = (n + 4095) / 4096 * 4096;
    if (bytes_live + size > bytes_limit)
        return result(kOutOfMemory);
    void *q = mmap(nullptr, size, PROT_READ | PROT_WRITE,
                   MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
    if (q == MAP_FAILED)
        return result(kOutOfMemory);
    for (size_t i = 0; i < (size < 65536 ? size : 65536) / 4; ++i)
        static_cast<uint32_t *>(q)[i] = 0x3f800000u;
    live[q] = size;
    bytes_live += size;
    mallocs += n >= big;
    *p = q;
    return 0;
}
int hipFree(void *p)
{
    if (!p)
        return 0;
    if (refuse_free)
        return result(kCaptureUnsupported);
    auto it = live.find(p);
    if (it == live.end())
        return result(1);
    bytes_live -= it->second;
    frees += it->second >= big;
    munmap(p, it->second);
    live.erase(it);
    return 0;
}
int hipMemcpy(void *d, const void *s, size_t n, int) { return memcpy(d, s, n), 0; }
int hipMemcpyAsync(void *d, const void *s, size_t n, int, void *) { return memcpy(d, s, n), 0; }
int hipMemset(void *, int, size_t) { return 0; }
int hipMemsetAsync(void *, int, size_t, void *) { return 0; }
int hipDeviceSynchronize() { return result(refuse_wait ? kCaptureUnsupported : 0); }
int hipStreamSynchronize(void *) { return result(refuse_wait ? kCaptureUnsupported : 0); }
int hipSetDevice(int) { return 0; }
int hipGetDevice(int *d) { return *d = 0, 0; }
int hipGetDeviceCount(int *n) { return *n = 1, 0; }
int hipGetSymbolAddress(void **p, const void *)
{
    static char here[256];
    return *p = here, 0;
}
int hipLaunchKernel(const void *, uint64_t, uint32_t, uint64_t, uint32_t, void **, size_t, void *)
{
    return 0;
}
int hipGetLastError()
{
    const int e = last_error;
    last_error = 0;
    return e;
}
}
