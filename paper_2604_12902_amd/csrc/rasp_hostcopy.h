// Copies between ordinary (pageable) host memory and the device, through a
// context's own pinned memory.
//
// hipMemcpyAsync on pageable memory moves it through the runtime's staging
// buffer on the calling thread, and waits.  That is 30 GB/s up and 17 down, but
// 4 down into memory the caller has just allocated, whose pages the copy
// touches first.  Large copies down go in chunks: kWorkers threads (the caller
// and its helpers) claim them in turn; each keeps two pinned chunks, so its own
// copy in host memory overlaps the device's, and the pages are touched by all
// of them.  Small copies (at most 256 KiB) of one call go through one pinned
// area, without a wait for each.
#ifndef RASP_HOSTCOPY_H
#define RASP_HOSTCOPY_H

#include <hip/hip_runtime.h>
#include <sys/mman.h>
#include <unistd.h>

#include <algorithm>
#include <atomic>
#include <condition_variable>
#include <cstdint>
#include <cstring>
#include <initializer_list>
#include <mutex>
#include <thread>
#include <vector>

namespace rasp {

class HostCopy {
public:
    static constexpr uint32_t kWorkers = 4, kSlots = 2;
    static constexpr uint64_t kChunk = 1ull << 20, kChunkMin = 256ull << 10;
    // Smallest copies that go in chunks (a helper wakes in some 30 us), plain
    // against chunks: down into new pages 1 MiB 241 us against 207, 4 MiB 982
    // against 518; into pages that are there 3 MiB 183 against 224, 4 MiB 242
    // against 245, 8 MiB 476 against 340; up 16 MiB 459 against 575, 64 MiB 2258
    // against 2152.
    static constexpr uint64_t kMinNew = 1ull << 20, kMinDown = 4ull << 20, kMinUp = 64ull << 20;
    // Chunks and helpers take some 1 ms to make, which is what they gain over
    // 8 MiB: they are made once copies of that size have been.
    static constexpr uint64_t kOpenAfter = 8ull << 20;
    // the pinned area of small copies, and the largest of them
    static constexpr uint64_t kArea = 1ull << 20, kSmall = 256ull << 10;

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
        char *p = take(bytes, st);
        if (!p) return copy(device, dst, src, bytes, hipMemcpyHostToDevice, st);
        std::memcpy(p, src, bytes);
        return hipMemcpyAsync(dst, p, bytes, hipMemcpyHostToDevice, st);
    }

    // A copy from the device whose data is there after flush().
    hipError_t get(int device, void *dst, const void *src, uint64_t bytes, hipStream_t st)
    {
        char *p = take(bytes, st);
        if (!p) return copy(device, dst, src, bytes, hipMemcpyDeviceToHost, st);
        const hipError_t e = hipMemcpyAsync(p, src, bytes, hipMemcpyDeviceToHost, st);
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
        if (bytes < kMinNew || !(up || kind == hipMemcpyDeviceToHost) ||
            bytes < (up ? kMinUp : present(dst, bytes) ? kMinDown : kMinNew) || pinned(up ? src : dst) || !open(device, bytes))
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

    // `bytes` of the area, or null; the area is made at the first small copy
    char *take(uint64_t bytes, hipStream_t st)
    {
        const uint64_t n = (bytes + 255) & ~255ull;
        if (bytes == 0 || bytes > kSmall || used_ + n > kArea || (!area_ && !open_area()) || got_.size() == got_.capacity())
            return nullptr;
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

    // are the pages of this memory there already (by its first, middle and last)
    static bool present(const void *p, uint64_t bytes)
    {
        const uint64_t page = static_cast<uint64_t>(sysconf(_SC_PAGESIZE)), a = reinterpret_cast<uint64_t>(p);
        for (uint64_t at : {a, a + bytes / 2, a + bytes - 1}) {
            unsigned char in = 1;
            if (mincore(reinterpret_cast<void *>(at / page * page), 1, &in) == 0 && !(in & 1)) return false;
        }
        return true;
    }

    // the chunks and the helpers
    bool open(int device, uint64_t bytes)
    {
        if (chunks_) return true;
        if (failed_) return false;
        wanted_ += bytes;
        if (wanted_ < kOpenAfter) return false;
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
    uint64_t wanted_ = 0;                // bytes that would have gone in chunks so far
    bool failed_ = false, no_area_ = false;      // tried already (null: without success)
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
