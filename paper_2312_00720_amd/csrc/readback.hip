// Counts back to the host. A call that sizes its outputs waits for a few words
// of device memory; a copy of each into pageable memory costs a blit kernel and a
// staging step of its own (four of them took 60-80 us of a 175 us join). Here
// one small kernel writes all of them into pinned host memory, and the stream is
// waited for once.
//
// A read takes one of the process's pinned blocks and gives it back after the wait, so
// blocks are only ever shared by reads that follow each other. At most kKeep idle
// ones are held, until the process ends; no thread frees one at its end, where that
// would wait for all work on the device.
#include <string.h>

#include <mutex>

#include "internal.hpp"

namespace gj {
namespace {

constexpr size_t kPinnedBytes = 65536;
constexpr size_t kKeep = 16;

class PinnedBlocks {
  public:
    ~PinnedBlocks() {
        for (void *p : idle_) (void)hipHostFree(p);
    }
    void *take() {  // nullptr: none to be had
        {
            std::lock_guard<std::mutex> lock(mu_);
            if (!idle_.empty()) {
                void *p = idle_.back();
                idle_.pop_back();
                return p;
            }
        }
        void *p = nullptr;
        if (hipHostMalloc(&p, kPinnedBytes, hipHostMallocPortable | hipHostMallocMapped) == hipSuccess) return p;
        (void)hipGetLastError();
        return nullptr;
    }
    void give(void *p) {
        {
            std::lock_guard<std::mutex> lock(mu_);
            if (idle_.size() < kKeep) {
                idle_.push_back(p);
                return;
            }
        }
        (void)hipHostFree(p);
    }

  private:
    std::mutex mu_;
    std::vector<void *> idle_;
};

PinnedBlocks &pinned_blocks() {
    static PinnedBlocks b;
    return b;
}

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
    for (const ReadPart &p : parts) {
        require(p.bytes % 4 == 0, "read back whole words", GJ_EHIP);
        total += p.bytes;
    }
    void *host = parts.size() <= (size_t)kParts && total <= kPinnedBytes ? pinned_blocks().take() : nullptr;
    if (!host) {
        for (const ReadPart &p : parts) GJ_HIP(hipMemcpyAsync(p.host, p.dev, p.bytes, hipMemcpyDeviceToHost, s));
        GJ_HIP(hipStreamSynchronize(s));
        return;
    }
    ExportArgs a{};
    int k = 0;
    for (const ReadPart &p : parts) {
        a.src[k] = static_cast<const uint32_t *>(p.dev);
        a.words[k++] = (uint32_t)(p.bytes / 4);
    }
    void *dev = nullptr;
    // on an error from here on the block is not given back: the kernel may still write to it
    GJ_HIP(hipHostGetDevicePointer(&dev, host, 0));
    a.dst = static_cast<uint32_t *>(dev);
    hipLaunchKernelGGL(k_export, dim3(1), dim3(256), 0, s, a);
    GJ_LAUNCHED("k_export");
    GJ_HIP(hipStreamSynchronize(s));
    const char *from = static_cast<const char *>(host);
    for (const ReadPart &p : parts) {
        if (p.bytes) memcpy(p.host, from, p.bytes);
        from += p.bytes;
    }
    pinned_blocks().give(host);
}

}  // namespace gj
