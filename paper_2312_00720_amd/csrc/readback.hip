// Counts back to the host. A call that sizes its outputs waits for a few words
// of device memory; a copy of each into pageable memory costs a blit kernel and a
// staging step of its own (four of them took 60-80 us of a 175 us join). Here
// one small kernel writes all of them into pinned host memory, and the stream is
// waited for once.
//
// The pinned block belongs to the calling thread: 64 KB, allocated on its first
// read, given back when the thread ends. Every use ends with the wait, so the
// thread's next call, on whatever stream, finds it free.
#include <string.h>

#include "internal.hpp"

namespace gj {
namespace {

constexpr size_t kPinnedBytes = 65536;

struct Pinned {
    void *p = nullptr;
    ~Pinned() {
        if (p) (void)hipHostFree(p);
    }
    void *get() {
        if (!p) {
            hipError_t e = hipHostMalloc(&p, kPinnedBytes, hipHostMallocPortable | hipHostMallocMapped);
            if (e != hipSuccess) {
                p = nullptr;
                throw Error(GJ_EHIP, std::string("pinned host memory: ") + hipGetErrorString(e));
            }
        }
        return p;
    }
};
thread_local Pinned t_pinned;

constexpr int kParts = 4;
struct ExportArgs {
    const uint32_t *src[kParts];
    uint32_t words[kParts];
    uint32_t *dst;  // host memory, the parts back to back
};

__global__ __launch_bounds__(256) void k_export(ExportArgs a) {
    uint32_t at = 0;
#pragma unroll
    for (int i = 0; i < kParts; ++i) {
        for (uint32_t w = threadIdx.x; w < a.words[i]; w += 256) a.dst[at + w] = a.src[i][w];
        at += a.words[i];
    }
}

}  // namespace

void read_back_parts(hipStream_t s, std::initializer_list<ReadPart> parts) {
    size_t total = 0;
    for (const ReadPart &p : parts) total += p.bytes;
    if (parts.size() > kParts || total > kPinnedBytes) {
        for (const ReadPart &p : parts) GJ_HIP(hipMemcpyAsync(p.host, p.dev, p.bytes, hipMemcpyDeviceToHost, s));
        GJ_HIP(hipStreamSynchronize(s));
        return;
    }
    char *host = static_cast<char *>(t_pinned.get());
    ExportArgs a{};
    int k = 0;
    for (const ReadPart &p : parts) {
        require(p.bytes % 4 == 0, "read back whole words", GJ_EHIP);
        a.src[k] = static_cast<const uint32_t *>(p.dev);
        a.words[k++] = (uint32_t)(p.bytes / 4);
    }
    void *dev = nullptr;
    GJ_HIP(hipHostGetDevicePointer(&dev, host, 0));
    a.dst = static_cast<uint32_t *>(dev);
    hipLaunchKernelGGL(k_export, dim3(1), dim3(256), 0, s, a);
    GJ_LAUNCHED("k_export");
    GJ_HIP(hipStreamSynchronize(s));
    for (const ReadPart &p : parts) {
        memcpy(p.host, host, p.bytes);
        host += p.bytes;
    }
}

}  // namespace gj
