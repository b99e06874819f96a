// A model of the part of the HIP runtime that librasp's host-side headers use,
// for tests of those headers on the CPU.  Device memory is ordinary memory.  A
// copy with a pinned host side is carried out when its stream (or an event
// behind it) is waited for, and not before: the latest that a device may be.
// One with a pageable source reads it in the call, one into pageable memory
// waits for the stream, as hipMemcpyAsync does.
#pragma once
#include <stdint.h>
#include <stdlib.h>
#include <string.h>

#include <map>
#include <mutex>
#include <string>
#include <vector>

enum hipError_t { hipSuccess = 0, hipErrorInvalidValue = 1, hipErrorOutOfMemory = 2 };
enum hipMemcpyKind { hipMemcpyHostToDevice = 1, hipMemcpyDeviceToHost = 2, hipMemcpyDeviceToDevice = 3 };
enum hipMemoryType { hipMemoryTypeUnregistered = 0, hipMemoryTypeHost = 1 };
struct hipPointerAttribute_t { hipMemoryType type; };

struct Copy {
    char *dst;
    const char *src;
    size_t n;
    std::string staged;                  // a pageable source's bytes
};
struct Stream { std::vector<Copy> queue; };
struct Event { Stream *on = nullptr; };
typedef Stream *hipStream_t;
typedef Event *hipEvent_t;
constexpr unsigned hipHostMallocDefault = 0, hipEventDisableTiming = 2;

struct Model {
    std::mutex mu;
    std::map<char *, size_t> pinned;
    size_t pinned_bytes = 0;
    int events = 0;
    bool refuse = false;                 // no pinned memory
    bool is_pinned(const void *p)
    {
        auto it = pinned.upper_bound(static_cast<char *>(const_cast<void *>(p)));
        if (it == pinned.begin()) return false;
        --it;
        return static_cast<const char *>(p) < it->first + it->second;
    }
    void drain(Stream *s)
    {
        for (Copy &c : s->queue) memcpy(c.dst, c.src ? c.src : c.staged.data(), c.n);
        s->queue.clear();
    }
};
inline Model &model() { static Model m; return m; }

inline hipError_t hipSetDevice(int) { return hipSuccess; }
inline hipError_t hipGetLastError() { return hipSuccess; }
inline hipError_t hipHostMalloc(void **p, size_t n, unsigned)
{
    std::lock_guard<std::mutex> g(model().mu);
    if (model().refuse) return hipErrorOutOfMemory;
    *p = malloc(n);
    model().pinned[static_cast<char *>(*p)] = n;
    model().pinned_bytes += n;
    return hipSuccess;
}
inline hipError_t hipHostFree(void *p)
{
    std::lock_guard<std::mutex> g(model().mu);
    model().pinned_bytes -= model().pinned[static_cast<char *>(p)];
    model().pinned.erase(static_cast<char *>(p));
    free(p);
    return hipSuccess;
}
inline hipError_t hipPointerGetAttributes(hipPointerAttribute_t *a, const void *p)
{
    std::lock_guard<std::mutex> g(model().mu);
    a->type = model().is_pinned(p) ? hipMemoryTypeHost : hipMemoryTypeUnregistered;
    return hipSuccess;
}
inline hipError_t hipMemcpyAsync(void *dst, const void *src, size_t n, hipMemcpyKind kind, hipStream_t s)
{
    std::lock_guard<std::mutex> g(model().mu);
    Copy c{static_cast<char *>(dst), static_cast<const char *>(src), n, {}};
    if (kind == hipMemcpyHostToDevice && !model().is_pinned(src)) {
        c.staged.assign(c.src, n);
        c.src = nullptr;
    }
    s->queue.push_back(c);
    if (kind == hipMemcpyDeviceToHost && !model().is_pinned(dst)) model().drain(s);
    return hipSuccess;
}
inline hipError_t hipStreamSynchronize(hipStream_t s)
{
    std::lock_guard<std::mutex> g(model().mu);
    if (s) model().drain(s);
    return hipSuccess;
}
inline hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned)
{
    std::lock_guard<std::mutex> g(model().mu);
    *e = new Event;
    ++model().events;
    return hipSuccess;
}
inline hipError_t hipEventDestroy(hipEvent_t e)
{
    std::lock_guard<std::mutex> g(model().mu);
    delete e;
    --model().events;
    return hipSuccess;
}
inline hipError_t hipEventRecord(hipEvent_t e, hipStream_t s)
{
    std::lock_guard<std::mutex> g(model().mu);
    e->on = s;
    return hipSuccess;
}
inline hipError_t hipEventSynchronize(hipEvent_t e)
{
    std::lock_guard<std::mutex> g(model().mu);
    if (e->on) model().drain(e->on);
    return hipSuccess;
}
