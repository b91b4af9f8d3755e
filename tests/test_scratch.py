"""The scratch memory of the squaring integrations under failing allocations, on the host: the
library's own header with the allocator replaced, built and run without a GPU."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "..", "paper_1804_03859_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

FAKE = r"""
#include <hip/hip_runtime.h>
#include <cstdio>
#include <cstdlib>
#include <map>
static std::map<char*, size_t> live;
static int allocs = 0, fail_at = -1;
static hipStreamCaptureStatus capturing = hipStreamCaptureStatusNone;
static hipError_t fake_malloc(void** p, size_t n) {
    if (allocs++ == fail_at) return hipErrorOutOfMemory;
    *p = std::malloc(n);
    live[static_cast<char*>(*p)] = n;
    return hipSuccess;
}
static hipError_t fake_free(void* p) {
    live.erase(static_cast<char*>(p));
    std::free(p);
    return hipSuccess;
}
static hipError_t fake_capturing(hipStream_t, hipStreamCaptureStatus* s) { *s = capturing; return hipSuccess; }
static hipError_t fake_mode(hipStreamCaptureMode*) { return hipSuccess; }
static hipError_t fake_sync() { return hipSuccess; }
#define hipMalloc(p, n) fake_malloc((void**)(p), n)
#define hipFree fake_free
#define hipStreamIsCapturing fake_capturing
#define hipThreadExchangeStreamCaptureMode fake_mode
#define hipDeviceSynchronize fake_sync
#include "cpower.hpp"
namespace tsk {
tsk_status fail(tsk_status st, const std::string&) { return st; }
}
using namespace tsk;
#define CHECK(c) do { if (!(c)) { std::printf("line %d: %s\n", __LINE__, #c); return 1; } } while (0)
// every array of the layout inside one live allocation
static bool inside(const void* p, size_t n) {
    for (auto& a : live)
        if (static_cast<const char*>(p) >= a.first && static_cast<const char*>(p) + n <= a.first + a.second) return true;
    return false;
}
template <typename real> static bool fits(const CpowWork& w) {
    for (int b = 0; b < w.nbuf; ++b)
        if (!inside(w.D<real>(b), cpow_stride(w.ld) * w.count * sizeof(real))) return false;
    for (int b = 0; b < 2; ++b)
        if (!inside(w.v<real>(b), size_t(4) * w.ld * w.count * sizeof(real))) return false;
    return inside(w.diag(), size_t(3) * w.ld * w.count * sizeof(double)) &&
           reinterpret_cast<uintptr_t>(w.diag()) % 8 == 0;
}
"""

FAILING = r"""
int main() {
    // one matrix, then a batch whose k-th allocation fails, then the batch again: what place() grants has
    // room for all of its arrays, whichever allocation failed before
    for (int k = 0; k < 4; ++k) {
        Scratch s;
        CpowWork w;
        fail_at = -1;
        CHECK(w.place(s, nullptr, 60, 1, 8, 2, 0) && fits<double>(w));
        fail_at = allocs + k;
        const bool first = w.place(s, nullptr, 60, 40, 8, 2, 0);
        CHECK(!first || fits<double>(w));
        CHECK(k > 0 || !first);
        const bool second = w.place(s, nullptr, 60, 40, 8, 2, 0);
        CHECK(!second || fits<double>(w));
        fail_at = -1;
        CHECK(w.place(s, nullptr, 60, 40, 8, 2, 0) && fits<double>(w));
        CHECK(w.place(s, nullptr, 127, 63, 4, 4, 2) && fits<float>(w));
        CHECK(w.place(s, nullptr, 60, 1, 8, 2, 0) && fits<double>(w));
        capturing = hipStreamCaptureStatusActive;
        CHECK(!w.place(s, nullptr, 60, 1, 8, 2, 0));
        capturing = hipStreamCaptureStatusNone;
    }
    CHECK(live.empty());
    return 0;
}
"""


def _run(tmp_path, body):
    src, exe = tmp_path / "t.hip", tmp_path / "t"
    src.write_text(FAKE + body)
    if not os.path.exists(HIPCC):
        pytest.skip("no hipcc")
    r = subprocess.run([HIPCC, "--offload-arch=gfx950", "-O1", "-std=c++17", "-w", "-Xclang", "-target-feature", "-Xclang",
                        "-packed-fp32-ops", "-I", CSRC, "-I", os.path.join(HERE, "..", "include"), str(src), "-o",
                        str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr


def test_layouts_have_room_after_failed_allocations(tmp_path):
    _run(tmp_path, FAILING)
