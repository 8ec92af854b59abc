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

    // The event for waits on `st`; null if it cannot be had.
    hipEvent_t of(hipStream_t)
    {
        int dev = 0;
        if (hipGetDevice(&dev) != hipSuccess) return nullptr;
        for (auto& pe : events_)
            if (pe.first == dev) return pe.second;
        hipEvent_t e = nullptr;
        if (hipEventCreateWithFlags(&e, hipEventDisableTiming | hipEventBlockingSync) != hipSuccess) return nullptr;
        events_.push_back({dev, e});
        return e;
    }

private:
    std::vector<std::pair<int, hipEvent_t>> events_;
};

}  // namespace tj
