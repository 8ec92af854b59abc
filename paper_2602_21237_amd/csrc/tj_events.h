// Events that a call records on its stream and the host then waits for.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>
#include <utility>
#include <vector>

namespace tj {

// One event per device, kept by the thread that uses it. They carry no times,
// and a wait for one blocks: a thread that spins in hipEventSynchronize holds up
// the others' calls (400 small requests submitted to a server of two slots:
// 3.8 ms with waits for the stream, 5.1 with spinning waits, 2.8 with these; a
// single caller's calls take the same time either way).
class WaitEvents {
public:
    ~WaitEvents()
    {
        for (auto& pe : events_) (void)hipEventDestroy(pe.second);
    }

    // The event for waits on `st`, of that stream's device (not the thread's
    // current one: a caller may pass another device's stream); null if it
    // cannot be had. The current device stays what it was.
    hipEvent_t of(hipStream_t st)
    {
        int cur = 0;
        hipDevice_t dev = 0;
        if (hipGetDevice(&cur) != hipSuccess) return nullptr;
        // (the null stream, and the handles that name it or the thread's own, are the current device's)
        if ((uintptr_t)st <= 2) dev = cur;
        else if (hipStreamGetDevice(st, &dev) != hipSuccess) return nullptr;
        for (auto& pe : events_)
            if (pe.first == dev) return pe.second;
        if (dev != cur && hipSetDevice(dev) != hipSuccess) return nullptr;
        hipEvent_t e = nullptr;
        const hipError_t rc = hipEventCreateWithFlags(&e, hipEventDisableTiming | hipEventBlockingSync);
        if (dev != cur && hipSetDevice(cur) != hipSuccess) return nullptr;
        if (rc != hipSuccess) return nullptr;
        events_.push_back({dev, e});
        return e;
    }

private:
    std::vector<std::pair<int, hipEvent_t>> events_;
};

}  // namespace tj
