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
static hipError_t fake_device(int* d) { *d = 0; return hipSuccess; }
#define hipMalloc(p, n) fake_malloc((void**)(p), n)
#define hipFree fake_free
#define hipStreamIsCapturing fake_capturing
#define hipThreadExchangeStreamCaptureMode fake_mode
#define hipDeviceSynchronize fake_sync
#define hipGetDevice fake_device
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
        IdleMemory::get().trim();
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
    IdleMemory::get().trim();
    CHECK(live.empty());
    return 0;
}
"""

SHARED = r"""
int main() {
    auto s1 = reinterpret_cast<hipStream_t>(16), s2 = reinterpret_cast<hipStream_t>(32);
    {
        // the operators of one stream share, those of another do not; one call at a time
        auto a = Scratch::of(s1), b = Scratch::of(s1), c = Scratch::of(s2);
        CHECK(a == b && a != c);
        CpowWork w, x, y;
        CHECK(w.place(*a, s1, 60, 40, 8, 2, 0) && fits<double>(w));
        CHECK(!b->mu.try_lock());
        CHECK(y.place(*c, s2, 60, 40, 8, 2, 0) && fits<double>(y) && y.base != w.base);
        w.lock.unlock();
        const int before = allocs;
        CHECK(x.place(*b, s1, 33, 7, 4, 4, 2) && fits<float>(x) && x.base == w.base && allocs == before);
        CHECK(!Scratch::of(hipStreamPerThread)->get(64, hipStreamPerThread));
    }
    // handed back with the last operator, and taken by the next stream's without an allocation
    CHECK(live.size() == 2);
    int before = allocs;
    for (int i = 0; i < 20; ++i) {
        auto a = Scratch::of(reinterpret_cast<hipStream_t>(64 + 16 * i));
        CpowWork w;
        CHECK(w.place(*a, nullptr, 60, 40, 8, 2, 0) && fits<double>(w));
    }
    CHECK(allocs == before && live.size() == 2);
    // bounded: by size, by number
    {
        std::vector<std::shared_ptr<Scratch>> many;
        for (int i = 0; i < 20; ++i) {
            many.push_back(std::make_shared<Scratch>());
            CHECK(many.back()->get(1 << 20, s1));
        }
        many.push_back(std::make_shared<Scratch>());
        CHECK(many.back()->get(IdleMemory::kIdleBytes + 1, s1));
    }
    size_t held = 0;
    for (auto& a : live) held += a.second;
    CHECK(live.size() <= IdleMemory::kIdleBlocks && held <= IdleMemory::kIdleBytes);
    // an allocation that fails gets the idle memory first
    DevBuf d;
    fail_at = allocs;
    CHECK(d.ensure(1 << 21) == TSK_OK && live.size() == 1);
    // a block that was never idle is not handed out: growth frees the old one
    Scratch g;
    CHECK(g.get(1000, s1) && g.get(5000, s1) && live.size() == 2);
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


def test_operators_of_a_stream_share_and_idle_memory_is_bounded(tmp_path):
    _run(tmp_path, SHARED)
