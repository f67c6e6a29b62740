"""The library's memory on a device that has none left, and under work that has
not ended: csrc/workspace.cpp, compiled for the host against a model of the
runtime that counts its waits, holds so many bytes and no more, and ends a
stream's work when it is told to."""

import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2107_05537_amd", "csrc")

RUNTIME = r"""
#pragma once
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <iterator>
#include <map>
#include <string>
struct float2 { float x, y; };
typedef int hipError_t;
enum { hipSuccess = 0, hipErrorOutOfMemory = 2, hipErrorNotReady = 600, hipHostMallocDefault = 0,
       hipEventDisableTiming = 2 };
struct ihipStream_t { bool busy = false; };
typedef ihipStream_t* hipStream_t;
struct ihipEvent_t { hipStream_t on = nullptr; };
typedef ihipEvent_t* hipEvent_t;
struct Model {
    size_t room = 0;                  // bytes left on the device
    std::map<void*, size_t> device, host;
    int waits = 0, mallocs = 0;
};
inline Model& model() { static Model m; return m; }
inline hipError_t hipGetLastError() { return hipSuccess; }
inline const char* hipGetErrorString(hipError_t) { return "error"; }
inline hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
// the address space is used up as it is handed out, never touched
template <class T> hipError_t hipMalloc(T** p, size_t bytes) {
    static uintptr_t next = 1 << 20;
    if (bytes > model().room) return hipErrorOutOfMemory;
    model().room -= bytes;
    ++model().mallocs;
    model().device[(void*)next] = bytes;
    *p = (T*)next;
    next += (bytes + 4095) / 4096 * 4096;
    return hipSuccess;
}
inline hipError_t hipFree(void* p) {
    model().room += model().device.at(p);
    model().device.erase(p);
    return hipSuccess;
}
template <class T> hipError_t hipHostMalloc(T** p, size_t bytes, unsigned) {
    *p = (T*)malloc(bytes);
    model().host[(void*)*p] = bytes;
    return hipSuccess;
}
inline hipError_t hipHostFree(void* p) { model().host.erase(p); free(p); return hipSuccess; }
inline hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { *e = new ihipEvent_t; return hipSuccess; }
inline hipError_t hipEventDestroy(hipEvent_t e) { delete e; return hipSuccess; }
inline hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) { e->on = s; return hipSuccess; }
inline hipError_t hipEventQuery(hipEvent_t e) { return e->on && e->on->busy ? hipErrorNotReady : hipSuccess; }
inline hipError_t hipEventSynchronize(hipEvent_t) { ++model().waits; return hipSuccess; }
inline hipError_t hipStreamSynchronize(hipStream_t) { ++model().waits; return hipSuccess; }
"""

HEAD = r"""
#include "internal.hpp"
namespace pmlsh {
void fail(int code, const std::string& msg) { throw Error{code, msg}; }
void set_error(const std::string&) {}
}
using namespace pmlsh;
#define CHECK(x) do { if (!(x)) { printf("line %d: %s\n", __LINE__, #x); exit(1); } } while (0)
template <class F> int code_of(F f) { try { f(); } catch (const Error& e) { return e.code; } return 0; }
int main() {
"""


def _run(tmp_path, body):
    (tmp_path / "hip").mkdir()
    (tmp_path / "hip" / "hip_runtime.h").write_text(RUNTIME)
    (tmp_path / "main.cpp").write_text(HEAD + body + "\nreturn 0;\n}\n")
    exe = str(tmp_path / "main")
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", f"-I{tmp_path}", f"-I{CSRC}",
                        f"-I{os.path.join(ROOT, 'include')}", str(tmp_path / "main.cpp"),
                        os.path.join(CSRC, "workspace.cpp"), "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr


def test_build_gives_its_scratch_up_for_the_index(tmp_path):
    """An array that fits beside everything but the build's scratch is allocated
    when no temporary is in use, and refused while one is."""
    _run(tmp_path, r"""
    model().room = (200 << 20);
    {
        BuildScratch s(1 << 20);                       // 97 MB
        const size_t left = model().room;
        CHECK(left < (110 << 20));
        void* t = BuildScratch::take_piece(1 << 20);
        CHECK(t && model().room == left);
        CHECK(code_of([&] { device_malloc(150 << 20); }) == PMLSH_ENOMEM);
        CHECK(BuildScratch::give_back(t));
        void* big = device_malloc(150 << 20);          // the scratch goes
        CHECK(model().room == (50 << 20));
        // what comes after it is allocated on its own
        CHECK(!BuildScratch::take_piece(256));
        CHECK(!BuildScratch::give_back(big));
        (void)hipFree(big);
    }
    CHECK(model().room == (200 << 20) && model().device.empty());
    """)


def test_scratch_pieces(tmp_path):
    _run(tmp_path, r"""
    model().room = (200 << 20);
    {
        BuildScratch s(1000);
        char* a = (char*)BuildScratch::take_piece(1000);
        char* b = (char*)BuildScratch::take_piece(5000);
        char* c = (char*)BuildScratch::take_piece(1);
        CHECK(a && b >= a + 1000 && c >= b + 5000 && (uintptr_t)b % 256 == 0);
        CHECK(BuildScratch::give_back(a) && BuildScratch::give_back(c) && BuildScratch::give_back(b));
        CHECK(!BuildScratch::give_back(b));
        CHECK(BuildScratch::take_piece(1 << 20) == a);   // one free run again
        {
            BuildScratch inner(10);
            CHECK(!BuildScratch::give_back(a));
        }
        CHECK(BuildScratch::give_back(a));
        CHECK(!BuildScratch::take_piece(size_t(1) << 40));
    }
    CHECK(!BuildScratch::take_piece(1) && model().device.empty());
    {
        model().room = 1000;                             // no scratch to be had
        BuildScratch s(1000);
        CHECK(!BuildScratch::take_piece(1));
    }
    """)


def test_idle_workspace_is_given_back(tmp_path):
    _run(tmp_path, r"""
    ihipStream_t st, other;
    model().room = (100 << 20);
    void* a = ws_alloc(40 << 20, &st);
    void* b = ws_alloc(40 << 20, &other);
    other.busy = true;
    ws_free(a, &st);
    ws_free(b, &other);
    CHECK(model().room == (20 << 20));
    CHECK(code_of([&] { device_malloc(70 << 20); }) == PMLSH_ENOMEM);   // b's work goes on
    CHECK(model().room == (60 << 20) && model().waits == 0);
    other.busy = false;
    (void)device_malloc(70 << 20);
    CHECK(model().room == (30 << 20) && model().waits == 0);
    """)


def test_workspace_shrinks_to_the_memory_there_is(tmp_path):
    _run(tmp_path, r"""
    ihipStream_t st;
    model().room = (100 << 20);
    int asked = 0;
    auto halves = [&](int64_t* b) { ++asked; *b /= 2; return *b >= (16 << 20); };
    void* a = ws_alloc_least(int64_t(1) << 30, &st, halves);
    CHECK(a && asked == 4 && model().device.at(a) == (64 << 20));
    CHECK(code_of([&] { ws_alloc_least(int64_t(1) << 30, &st, [](int64_t* b) {
        *b /= 2; return *b >= (40 << 20); }); }) == PMLSH_ENOMEM);
    CHECK(ws_alloc_least(30 << 20, &st, halves) && asked == 4);
    """)


def test_pinned_blocks(tmp_path):
    """Blocks given back under work that has not ended: no wait until 64 small ones
    are out, no block handed out twice, a bounded number kept afterwards."""
    _run(tmp_path, r"""
    ihipStream_t st, other;
    st.busy = true;
    std::map<void*, int> seen;
    for (int i = 0; i < 60; ++i) {
        const size_t bytes = i % 8 ? 1000 + i : 8 << 20;
        char* p = (char*)pinned_alloc(bytes);
        CHECK(++seen[p] == 1);
        p[0] = p[bytes - 1] = 1;
        pinned_free(p, &st);
    }
    CHECK(model().waits == 0);
    // another stream's block is free at once
    void* q = pinned_alloc(1000);
    CHECK(!seen.count(q));
    pinned_free(q, &other);
    for (int i = 0; i < 11; ++i) {
        void* p = pinned_alloc(1000);
        CHECK(model().waits == 0);
        if (p != q) CHECK(++seen[p] == 1);
        pinned_free(p, p == q ? &other : &st);
    }
    while (pinned_alloc(65536) && model().waits == 0) {}   // all 64 are out
    CHECK(model().waits == 1);
    st.busy = false;
    void* r = pinned_alloc(9 << 20);                       // the large ones go, but one
    CHECK(r && model().waits == 1);
    size_t large = 0;
    for (auto& h : model().host) large += h.second > (4u << 20);
    CHECK(large == 2);
    pinned_free(r, &st);
    CHECK(pinned_alloc(9 << 20) == r);
    """)
