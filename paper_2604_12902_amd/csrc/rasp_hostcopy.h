// Copies between ordinary (pageable) host memory and the device, through a
// context's own pinned memory.
//
// hipMemcpyAsync on pageable memory moves it through a staging buffer of the
// stream, on the calling thread, and waits.  The first 16 MiB over a stream go
// at 2.6 GB/s (1 MiB 390 us, 51 later: the buffer's pages are touched for the
// first time), and copies down into memory the caller has just allocated, whose
// pages are touched too, at 4 GB/s.  Here copies of up to 1 MiB go through one
// pinned area, several of a call without a wait for each (1 MiB 51 us up, 60
// down).  Larger ones go in chunks: kWorkers threads (the caller and its
// helpers) claim them in turn; each keeps two pinned chunks, so its own copy in
// host memory overlaps the device's, and pages are touched by all of them (1 MiB
// 94-120 us, 4 MiB 216 up, 240 down and 460 into new pages, where one thread
// takes 130, 240 and 980 once its buffer has been touched).
#ifndef RASP_HOSTCOPY_H
#define RASP_HOSTCOPY_H

#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <condition_variable>
#include <cstdint>
#include <cstring>
#include <mutex>
#include <thread>
#include <vector>

namespace rasp {

class HostCopy {
public:
    static constexpr uint32_t kWorkers = 4, kSlots = 2;
    static constexpr uint64_t kChunk = 1ull << 20, kChunkMin = 256ull << 10;
    // the pinned area, and so the largest copy that does not go in chunks
    static constexpr uint64_t kArea = 1ull << 20;
    // Chunks and helpers take some 0.5 ms to make and 0.1 to end: they are made
    // at the first copy that goes in them, or before it once this much has been
    // copied, which a context for a small batch or two does not come to.
    static constexpr uint64_t kOpenAfter = 512ull << 10;

    ~HostCopy() { close(); }

    // Start of a call that uses put() or get().  The area starts anew, so a call
    // that ended without settled() or flush() (an error between its copies) is
    // waited for here: its copies may still read or write the area.
    hipError_t begin()
    {
        const hipError_t e = used_ != 0 ? hipStreamSynchronize(on_) : hipSuccess;
        settled();
        return e;
    }

    // The stream has been waited for since the last copy.
    void settled()
    {
        used_ = 0;
        got_.clear();
    }

    // A copy to the device whose source may be reused on return.
    hipError_t put(int device, void *dst, const void *src, uint64_t bytes, hipStream_t st)
    {
        hipError_t e = hipSuccess;
        char *p = take(device, bytes, st, &e);
        if (e) return e;
        if (!p) return copy(device, dst, src, bytes, hipMemcpyHostToDevice, st);
        std::memcpy(p, src, bytes);
        return hipMemcpyAsync(dst, p, bytes, hipMemcpyHostToDevice, st);
    }

    // A copy from the device whose data is there after flush().
    hipError_t get(int device, void *dst, const void *src, uint64_t bytes, hipStream_t st)
    {
        hipError_t e = hipSuccess;
        char *p = take(device, bytes, st, &e);
        if (e) return e;
        if (!p) return copy(device, dst, src, bytes, hipMemcpyDeviceToHost, st);
        e = hipMemcpyAsync(p, src, bytes, hipMemcpyDeviceToHost, st);
        if (!e) got_.push_back({dst, p, bytes});
        return e;
    }

    // Waits for the stream.
    hipError_t flush(hipStream_t st)
    {
        const hipError_t e = hipStreamSynchronize(st);
        if (!e)
            for (const Got &g : got_) std::memcpy(g.dst, g.p, g.bytes);
        settled();
        return e;
    }

    // As hipMemcpyAsync between pageable host and device memory on `st`: on
    // return the host memory of a copy to the device may be reused, and that
    // of a copy from the device holds the data.
    hipError_t copy(int device, void *dst, const void *src, uint64_t bytes, hipMemcpyKind kind, hipStream_t st)
    {
        if (bytes == 0) return hipSuccess;
        const bool up = kind == hipMemcpyHostToDevice;
        if (bytes <= kArea || !(up || kind == hipMemcpyDeviceToHost) || pinned(up ? src : dst) || !open(device))
            return hipMemcpyAsync(dst, src, bytes, kind, st);
        const uint64_t chunk = std::min<uint64_t>(kChunk, std::max<uint64_t>(kChunkMin, (bytes / (kWorkers * kSlots) + 4095) & ~4095ull));
        {
            std::lock_guard<std::mutex> g(mu_);
            dst_ = static_cast<char *>(dst);
            src_ = static_cast<const char *>(src);
            bytes_ = bytes;
            chunk_ = chunk;
            up_ = up;
            st_ = st;
            next_ = 0;
            error_ = hipSuccess;
            running_ = static_cast<uint32_t>(helpers_.size());
            ++job_;
        }
        wake_.notify_all();
        work(0);
        std::unique_lock<std::mutex> g(mu_);
        done_.wait(g, [&] { return running_ == 0; });
        return error_;
    }

    void close()
    {
        {
            std::lock_guard<std::mutex> g(mu_);
            stop_ = true;
        }
        wake_.notify_all();
        for (auto &t : helpers_) t.join();
        helpers_.clear();
        close_chunks();
        if (area_) (void)hipHostFree(area_);
        area_ = nullptr;
    }

private:
    struct Got {
        void *dst;
        const char *p;
        uint64_t bytes;
    };
    struct Slot {
        char *p = nullptr;
        hipEvent_t ev = nullptr;
        bool busy = false;               // a copy to the device still reads it
    };

    void close_chunks()
    {
        if (!chunks_) return;
        for (auto &w : slots_)
            for (auto &s : w) {
                if (s.busy) (void)hipEventSynchronize(s.ev);
                if (s.ev) (void)hipEventDestroy(s.ev);
                s = Slot{};
            }
        (void)hipHostFree(chunks_);
        chunks_ = nullptr;
    }

    // `bytes` of the area, or null; the area is made at the first such copy, and
    // the stream waited for when it is used up
    char *take(int device, uint64_t bytes, hipStream_t st, hipError_t *e)
    {
        const uint64_t n = (bytes + 255) & ~255ull;
        if (bytes == 0 || bytes > kArea || (!area_ && !open_area())) return nullptr;
        moved_ += bytes;
        if (moved_ > kOpenAfter) (void)open(device);
        if ((used_ + n > kArea || got_.size() == got_.capacity()) && (*e = flush(st))) return nullptr;
        char *p = area_ + used_;
        used_ += n;
        on_ = st;
        return p;
    }

    bool open_area()
    {
        if (no_area_) return false;
        no_area_ = true;
        try {
            got_.reserve(16);
        } catch (...) {
            return false;
        }
        area_ = host_malloc(kArea);
        return area_ != nullptr;
    }

    static char *host_malloc(uint64_t bytes)
    {
        void *p = nullptr;
        if (hipHostMalloc(&p, bytes, hipHostMallocDefault) == hipSuccess) return static_cast<char *>(p);
        (void)hipGetLastError();
        return nullptr;
    }

    static bool pinned(const void *p)
    {
        hipPointerAttribute_t a{};
        const hipError_t e = hipPointerGetAttributes(&a, p);
        if (e != hipSuccess) {
            (void)hipGetLastError();
            return false;
        }
        return a.type != hipMemoryTypeUnregistered;
    }

    // the chunks and the helpers
    bool open(int device)
    {
        if (chunks_) return true;
        if (failed_) return false;
        failed_ = true;
        device_ = device;
        if (!(chunks_ = host_malloc(kWorkers * kSlots * kChunk))) return false;
        for (uint32_t w = 0; w < kWorkers; ++w)
            for (uint32_t s = 0; s < kSlots; ++s) {
                slots_[w][s].p = chunks_ + (w * kSlots + s) * kChunk;
                if (hipEventCreateWithFlags(&slots_[w][s].ev, hipEventDisableTiming) != hipSuccess) {
                    (void)hipGetLastError();
                    slots_[w][s].ev = nullptr;
                    close_chunks();
                    return false;
                }
            }
        try {
            helpers_.reserve(kWorkers);
            for (uint32_t w = 1; w < kWorkers; ++w) helpers_.emplace_back([this, w] { help(w); });
        } catch (...) {
            // fewer helpers, or the caller alone
        }
        return true;
    }

    void help(uint32_t w)
    {
        (void)hipSetDevice(device_);
        uint64_t seen = 0;
        for (;;) {
            {
                std::unique_lock<std::mutex> g(mu_);
                wake_.wait(g, [&] { return stop_ || job_ != seen; });
                if (stop_) return;
                seen = job_;
            }
            work(w);
            std::lock_guard<std::mutex> g(mu_);
            if (--running_ == 0) done_.notify_one();
        }
    }

    void note(hipError_t e)
    {
        std::lock_guard<std::mutex> g(mu_);
        if (error_ == hipSuccess) error_ = e;
    }

    void work(uint32_t w)
    {
        uint64_t off[kSlots], len[kSlots] = {};          // a chunk on its way from the device
        hipError_t e = hipSuccess;
        for (uint32_t s = 0; !e; s = (s + 1) % kSlots) {
            Slot &t = slots_[w][s];
            if (t.busy) {
                e = hipEventSynchronize(t.ev);
                t.busy = false;
            }
            if (!e && len[s]) {
                e = hipEventSynchronize(t.ev);
                if (!e) std::memcpy(dst_ + off[s], t.p, len[s]);
                len[s] = 0;
            }
            if (e) break;
            const uint64_t at = next_.fetch_add(1) * chunk_;
            if (at >= bytes_) {
                bool left = false;
                for (uint64_t l : len) left |= l != 0;
                if (!left) break;
                continue;
            }
            const uint64_t n = std::min(chunk_, bytes_ - at);
            if (up_) {
                std::memcpy(t.p, src_ + at, n);
                e = hipMemcpyAsync(dst_ + at, t.p, n, hipMemcpyHostToDevice, st_);
                t.busy = true;
            } else {
                e = hipMemcpyAsync(t.p, src_ + at, n, hipMemcpyDeviceToHost, st_);
                off[s] = at;
                len[s] = n;
            }
            if (!e) e = hipEventRecord(t.ev, st_);
        }
        if (e) {
            // nothing may read or write the chunks or the caller's memory any more
            (void)hipStreamSynchronize(st_);
            for (auto &t : slots_[w]) t.busy = false;
            note(e);
        }
    }

    int device_ = 0;
    char *chunks_ = nullptr, *area_ = nullptr;
    bool failed_ = false, no_area_ = false;      // tried already (null: without success)
    uint64_t moved_ = 0;                 // bytes copied by way of the area
    Slot slots_[kWorkers][kSlots];
    uint64_t used_ = 0;                  // of the area, by copies on the stream
    hipStream_t on_ = nullptr;
    std::vector<Got> got_;
    std::vector<std::thread> helpers_;
    std::mutex mu_;
    std::condition_variable wake_, done_;
    bool stop_ = false;
    uint64_t job_ = 0;
    uint32_t running_ = 0;
    // the copy at hand
    char *dst_ = nullptr;
    const char *src_ = nullptr;
    uint64_t bytes_ = 0, chunk_ = 1;
    bool up_ = false;
    hipStream_t st_ = nullptr;
    std::atomic<uint64_t> next_{0};
    hipError_t error_ = hipSuccess;
};

}  // namespace rasp

#endif
