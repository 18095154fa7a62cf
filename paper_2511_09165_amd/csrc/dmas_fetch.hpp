// Copies of device results into a caller's memory.
//
// Memory that HIP knows (pinned, registered, managed) takes one hipMemcpy: for
// pinned memory one DMA, 56.6 GB/s for a result of 53 MB (41 in the chunks
// below).
//
// Pageable memory: chunks go by DMA into pinned buffers and from there to the
// destination, on several host threads, so that the DMA, the copies and the
// destination's page faults overlap. A result of 53 MB into mapped and into
// fresh pages: hipMemcpy 18 and 10 GB/s, four threads with 1 MiB chunks and a
// stream each 40-46 and 35-37 (six or eight threads, 512 KiB or 2 MiB chunks and
// one stream for all measured the same or slower). Each thread maps its chunk's
// pages while the chunk's DMA is under way, since a fresh array's page faults
// cost more than the copies.
#pragma once

#include <hip/hip_runtime.h>
#include <sys/mman.h>
#include <unistd.h>

#include <algorithm>
#include <atomic>
#include <condition_variable>
#include <cstddef>
#include <cstdint>
#include <cstring>
#include <mutex>
#include <thread>
#include <vector>

namespace dmas {

class HostFetch {
public:
    static constexpr int kThreads = 4;                       // helpers and the caller
    static constexpr size_t kChunk = (size_t)1024 << 10;

    // Allocates the buffers and starts the helpers; on an error nothing is kept
    // and copy() falls back to hipMemcpy.
    hipError_t start(int device)
    {
        device_ = device;
        hipError_t e = hipHostMalloc(reinterpret_cast<void **>(&pinned_), kThreads * kChunk, hipHostMallocDefault);
        for (int i = 0; i < kThreads && e == hipSuccess; ++i)
            e = hipStreamCreateWithFlags(&streams_[i], hipStreamNonBlocking);
        if (e == hipSuccess) {
            try {
                for (int i = 1; i < kThreads; ++i) helpers_.emplace_back([this, i] { help(i); });
            } catch (...) {
                e = hipErrorOutOfMemory;
            }
        }
        ready_ = e == hipSuccess;
        if (!ready_) {
            shut();
            (void)hipGetLastError();   // not the caller's
        }
        return e;
    }

    ~HostFetch() { shut(); }

    // dst[0, bytes) = src[0, bytes), src on the device; returns when done.
    // Calls that overlap on one server take turns at the helpers: the later
    // ones copy by hipMemcpy.
    hipError_t copy(void *dst, const void *src, size_t bytes)
    {
        std::unique_lock<std::mutex> turn(turn_, std::try_to_lock);
        if (!ready_ || bytes < 2 * kChunk || !turn.owns_lock() || !pageable(dst))
            return hipMemcpy(dst, src, bytes, hipMemcpyDeviceToHost);
        {
            std::lock_guard<std::mutex> lk(mu_);
            dst_ = static_cast<char *>(dst);
            src_ = static_cast<const char *>(src);
            bytes_ = bytes;
            next_.store(0);
            error_.store((int)hipSuccess);
            open_ = true;
            ++job_;
        }
        wake_.notify_all();
        work(0);
        std::unique_lock<std::mutex> lk(mu_);
        open_ = false;                                       // no helper joins from here on
        idle_.wait(lk, [this] { return active_ == 0; });
        return (hipError_t)error_.load();
    }

private:
    // Whether HIP knows nothing of the memory at p.
    static bool pageable(const void *p)
    {
        hipPointerAttribute_t a{};
        if (hipPointerGetAttributes(&a, p) == hipSuccess) return a.type == hipMemoryTypeUnregistered;
        (void)hipGetLastError();   // some versions report such memory as an error
        return true;
    }

    // Moves chunks of the open job until none is left, through buffer i.
    void work(int i)
    {
        char *buf = pinned_ + i * kChunk;
        for (;;) {
            const size_t at = next_.fetch_add(1) * kChunk;
            if (at >= bytes_) return;
            const size_t n = std::min(kChunk, bytes_ - at);
            hipError_t e = hipMemcpyAsync(buf, src_ + at, n, hipMemcpyDeviceToHost, streams_[i]);
            if (e == hipSuccess) map_pages(dst_ + at, n);
            if (e == hipSuccess) e = hipStreamSynchronize(streams_[i]);
            if (e != hipSuccess) {
                error_.store((int)e);
                return;
            }
            std::memcpy(dst_ + at, buf, n);
        }
    }

    // Maps the pages of [p, p + n) for writing in one call, as the copy that
    // follows would one fault at a time; where the kernel or the mapping does not
    // support it the copy still does.
    static void map_pages(char *p, size_t n)
    {
#ifdef MADV_POPULATE_WRITE
        const uintptr_t at = reinterpret_cast<uintptr_t>(p), lo = at & ~((uintptr_t)sysconf(_SC_PAGESIZE) - 1);
        (void)madvise(reinterpret_cast<void *>(lo), at + n - lo, MADV_POPULATE_WRITE);
#else
        (void)p, (void)n;
#endif
    }

    void help(int i)
    {
        (void)hipSetDevice(device_);   // a failure shows in the first copy
        unsigned long long seen = 0;
        std::unique_lock<std::mutex> lk(mu_);
        for (;;) {
            wake_.wait(lk, [&] { return stop_ || (open_ && job_ != seen); });
            if (stop_) return;
            seen = job_;
            ++active_;
            lk.unlock();
            work(i);
            lk.lock();
            if (--active_ == 0) idle_.notify_all();
        }
    }

    void shut()
    {
        {
            std::lock_guard<std::mutex> lk(mu_);
            stop_ = true;
        }
        wake_.notify_all();
        for (auto &t : helpers_) t.join();
        helpers_.clear();
        for (auto &st : streams_) {
            if (st) (void)hipStreamDestroy(st);   // (each copy was waited for)
            st = nullptr;
        }
        if (pinned_) (void)hipHostFree(pinned_);
        pinned_ = nullptr;
        ready_ = false;
    }

    int device_ = 0;
    bool ready_ = false;
    char *pinned_ = nullptr;                                 // kThreads buffers of kChunk
    hipStream_t streams_[kThreads] = {};
    std::vector<std::thread> helpers_;

    std::mutex turn_;                                        // one job at a time
    std::mutex mu_;                                          // open_, job_, active_, stop_
    std::condition_variable wake_, idle_;
    bool open_ = false, stop_ = false;
    int active_ = 0;                                         // helpers at work on the job
    unsigned long long job_ = 0;
    char *dst_ = nullptr;                                    // the job; constant while open or active
    const char *src_ = nullptr;
    size_t bytes_ = 0;
    std::atomic<size_t> next_{0};
    std::atomic<int> error_{0};
};

}  // namespace dmas
