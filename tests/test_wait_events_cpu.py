"""The host's wait events (csrc/tj_events.h), compiled against stand-ins for the
HIP calls they make: flags, reuse and release, without a GPU."""
import json
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include "tj_events.h"
#include <cstdio>

static int current = 0, made = 0, gone = 0, made_on[16];
static unsigned made_flags[16];

extern "C" {
hipError_t hipGetDevice(int* d) { *d = current; return hipSuccess; }
hipError_t hipSetDevice(int d) { current = d; return hipSuccess; }
// a stream's device is the value of its handle, less 100
hipError_t hipStreamGetDevice(hipStream_t s, hipDevice_t* d) { *d = (int)(uintptr_t)s - 100; return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned flags)
{
    made_on[made] = current;
    made_flags[made] = flags;
    *e = (hipEvent_t)(uintptr_t)(1000 + made++);
    return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t) { gone++; return hipSuccess; }
}

int main()
{
    auto stream = [](int dev) { return (hipStream_t)(uintptr_t)(100 + dev); };
    {
        tj::WaitEvents w;
        hipStream_t seq[] = {nullptr, stream(0), stream(3), stream(3), nullptr, stream(0)};
        std::printf("{\"got\": [");
        for (int i = 0; i < 6; i++) {
            current = i == 4 ? 3 : 0;
            const int was = current;
            std::printf("%s[%d, %d]", i ? ", " : "", (int)(uintptr_t)w.of(seq[i]) - 1000, current == was);
        }
        std::printf("], \"made_on\": [");
        for (int i = 0; i < made; i++) std::printf("%s%d", i ? ", " : "", made_on[i]);
        std::printf("], \"flags\": [");
        for (int i = 0; i < made; i++) std::printf("%s%u", i ? ", " : "", made_flags[i]);
        std::printf("], \"want\": %u", (unsigned)(hipEventDisableTiming | hipEventBlockingSync));
    }
    std::printf(", \"gone\": %d}\n", gone);
}
"""


@pytest.fixture(scope="module")
def seen(tmp_path_factory):
    cxx = shutil.which("g++")
    if not cxx:
        pytest.skip("no host compiler")
    d = tmp_path_factory.mktemp("events")
    (d / "main.cpp").write_text(PROGRAM)
    subprocess.check_call([cxx, "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                           "-I" + os.path.join(ROOT, "paper_2602_21237_amd", "csrc"), "-o", str(d / "main"),
                           str(d / "main.cpp")])
    return json.loads(subprocess.check_output([str(d / "main")]))


def test_waits_block(seen):
    assert seen["flags"] and all(f == seen["want"] for f in seen["flags"])


def test_events_are_released(seen):
    assert seen["gone"] == len(seen["made_on"])


def test_events_are_of_the_streams_device(seen):
    # null stream, streams of devices 0, 3, 3, null stream with device 3 current, stream of device 0
    assert [g[0] for g in seen["got"]] == [0, 0, 1, 1, 1, 0] and seen["made_on"] == [0, 3]
    assert all(g[1] for g in seen["got"])  # the current device stays
