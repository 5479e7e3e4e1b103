"""The pinned slots that reductions return their results in (host code against
stand-ins for the HIP calls): a slot whose kernel was not waited for is never
handed out again, and the page is not freed under a call that holds one."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <unistd.h>

#include <condition_variable>
#include <cstdio>
#include <cstring>
#include <set>
#include <thread>

#include "host_slot.h"

static hipError_t wait_result = hipSuccess;
static int copies = 0;

extern "C" {
hipError_t hipHostMalloc(void **p, size_t n, unsigned) {
    *p = std::malloc(n);
    return hipSuccess;
}
hipError_t hipHostFree(void *) {
    if (write(1, "freed\n", 6) != 6) std::abort();
    return hipSuccess;
}
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode *) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return wait_result; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t) {
    std::memcpy(d, s, n);
    ++copies;
    return hipSuccess;
}
}
namespace prx {
void set_error(const std::string &) {}
prx_status fail(prx_status st, const std::string &) { return st; }
prx_status hip_fail(hipError_t, const char *) { return PRX_ERR_HIP; }
}  // namespace prx

static double dev[2], h[2];

static double *call(double v, prx_status want, hipError_t launched = hipSuccess) {
    double *where = nullptr;
    const prx_status st = prx::read_back(
        [&](double *out) {
            where = out;
            out[0] = v;
            out[1] = -v;
            return launched;
        },
        dev, h, nullptr, "launch");
    if (st != want || (st == PRX_OK && (h[0] != v || h[1] != -v))) std::abort();
    return where;
}

int main(int, char **argv) {
    const std::string what = argv[1];
    double *first = call(1.0, PRX_OK);
    if (what == "reuse") {
        if (call(2.0, PRX_OK) != first || call(3.0, PRX_ERR_HIP, hipErrorUnknown) != first ||
            call(4.0, PRX_OK) != first)
            return 1;
    } else if (what == "failed_wait") {
        std::set<double *> lost;
        for (int i = 0; i < 64; ++i) {
            wait_result = hipErrorUnknown;
            double *p = call(5.0, PRX_ERR_HIP, i % 2 ? hipErrorUnknown : hipSuccess);
            if (!lost.insert(p).second || p == dev) return 2;
            wait_result = hipSuccess;
            if (lost.count(call(6.0, PRX_OK))) return 3;
        }
        if (call(7.0, PRX_OK) != dev || copies != 2) return 4;
    } else {  // a thread that is still inside a call when the process ends
        std::mutex m;
        std::condition_variable cv;
        bool inside = false;
        std::thread([&] {
            prx::read_back(
                [&](double *) {
                    {
                        std::lock_guard<std::mutex> l(m);
                        inside = true;
                    }
                    cv.notify_one();
                    for (;;) pause();
                    return hipSuccess;
                },
                dev, h, nullptr, "launch");
        }).detach();
        std::unique_lock<std::mutex> l(m);
        cv.wait(l, [&] { return inside; });
        std::exit(0);
    }
    return 0;
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("host_slot")
    (d / "slot.cpp").write_text(PROGRAM)
    exe = str(d / "slot")
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-w",
                        "-I/opt/rocm/include", "-I", os.path.join(ROOT, "include"),
                        "-I", os.path.join(ROOT, "paper_2504_17881_amd", "csrc"),
                        str(d / "slot.cpp"), "-o", exe, "-pthread"],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return exe


@pytest.mark.parametrize("what,freed", [("reuse", "freed\n"), ("failed_wait", ""),
                                        ("exit_inside", "")])
def test_slots(program, what, freed):
    r = subprocess.run([program, what], capture_output=True, text=True, timeout=60)
    assert (r.returncode, r.stdout) == (0, freed), r.stderr
