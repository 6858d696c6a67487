"""What the library keeps of destroyed graphs' device memory (CPU: csrc/fw_pool.h compiled against a
stub of the HIP allocator).
"""
from __future__ import annotations

import os
import shutil
import subprocess

import pytest

from tests.conftest import ROOT

CXX = shutil.which("g++")
pytestmark = pytest.mark.skipif(CXX is None, reason="needs g++")

STUB = r"""
#pragma once
#include <stddef.h>
#include <stdint.h>
#include <map>
#include <mutex>
typedef int hipError_t;
constexpr hipError_t hipSuccess = 0, hipErrorOutOfMemory = 2;
// addresses only, no memory; `room` bytes per device
struct Stub {
    std::mutex mu;
    std::map<uintptr_t, std::pair<size_t, int>> live;
    size_t used[2] = {0, 0}, room = (size_t)288 << 30;
    uintptr_t next = 4096;
    int mallocs = 0;
    bool bad_free = false;
};
inline Stub &stub() { static Stub s; return s; }
inline int &device() { static thread_local int d = 0; return d; }
inline hipError_t hipGetDevice(int *d) { *d = device(); return hipSuccess; }
inline hipError_t hipGetLastError() { return hipSuccess; }
inline hipError_t hipMalloc(void **p, size_t n)
{
    std::lock_guard<std::mutex> lk(stub().mu);
    ++stub().mallocs;
    if (stub().used[device()] + n > stub().room) return hipErrorOutOfMemory;
    stub().used[device()] += n;
    stub().live[stub().next] = {n, device()};
    *p = (void *)stub().next;
    stub().next += n + 4096;
    return hipSuccess;
}
inline hipError_t hipFree(void *p)
{
    std::lock_guard<std::mutex> lk(stub().mu);
    if (!p) return hipSuccess;
    auto it = stub().live.find((uintptr_t)p);
    if (it == stub().live.end()) { stub().bad_free = true; return hipSuccess; }
    stub().used[it->second.second] -= it->second.first;
    stub().live.erase(it);
    return hipSuccess;
}
"""

MAIN = r"""
#include "fw_pool.h"
#include <stdio.h>
#include <string.h>
#include <thread>
#include <vector>
using namespace fw;
static const size_t MB = (size_t)1 << 20, GB = (size_t)1 << 30;
#define CHECK(x) do { if (!(x)) { printf("%s:%d: %s\n", CASE, __LINE__, #x); return 1; } } while (0)
static const char *CASE;
static size_t used(int d = 0) { std::lock_guard<std::mutex> lk(stub().mu); return stub().used[d]; }
struct G { std::vector<void *> p; };
static G make(std::vector<size_t> sizes)
{
    G g;
    dev_pool().made();
    for (size_t n : sizes) { void *p; if (dev_pool().alloc(&p, n) == hipSuccess) g.p.push_back(p); }
    return g;
}
static void destroy(G &g, bool unused = true) { for (void *p : g.p) dev_pool().free(p, unused); g.p.clear(); dev_pool().turn(); }
static void go() { G a = make({MB}); destroy(a); G b = make({MB}); destroy(b); dev_pool(); }  // (from here on memory is kept)
int main(int, char **argv)
{
    CASE = argv[1];
    auto is = [&](const char *s) { return strcmp(CASE, s) == 0; };
    if (is("first_graphs")) {  // nothing is kept until a graph is made after one was destroyed
        G a = make({5 * MB, GB}), b = make({7 * MB});
        void *scratch; CHECK(dev_pool().alloc(&scratch, GB) == hipSuccess);
        dev_pool().free(scratch, true);
        CHECK(used() == 12 * MB + GB);
        destroy(a); CHECK(used() == 7 * MB);
        destroy(b); CHECK(used() == 0);
        G c = make({5 * MB, GB}); destroy(c); CHECK(used() == 5 * MB + GB);
        const int before = stub().mallocs;
        G d = make({5 * MB, GB}); CHECK(stub().mallocs == before);
        destroy(d); CHECK(used() == 5 * MB + GB);
    } else if (is("release")) {
        go(); G a = make({GB, 3 * MB}), live = make({2 * MB}); destroy(a); CHECK(used() > 2 * MB);
        dev_pool().release(); CHECK(used() == 2 * MB);
        destroy(live); CHECK(used() == 0);  // none made since
        G b = make({GB}); destroy(b); CHECK(used() == GB);
        dev_pool().release(); CHECK(used() == 0);
        dev_pool().release(); CHECK(used() == 0);
    } else if (is("most")) {  // 8 GiB at most, the oldest make room; larger blocks are not kept
        go(); G a = make({3 * GB, 3 * GB, 3 * GB, 9 * GB, 3 * GB}); destroy(a);
        CHECK(used() <= 8 * GB && used() >= 6 * GB);
        G b = make({3 * GB, 3 * GB}); CHECK(used() <= 8 * GB); destroy(b);
        CHECK(used() <= 8 * GB);
    } else if (is("blocks")) {  // 64 blocks at most
        go(); G a = make(std::vector<size_t>(200, 2 * MB)); destroy(a); CHECK(used() == 64 * 2 * MB);
    } else if (is("turns")) {  // eight graphs in a row without a use
        go(); G a = make({GB}); destroy(a);
        for (int i = 0; i < 8; ++i) { CHECK(used() >= GB); G b = make({2 * MB}); destroy(b); }
        G b = make({2 * MB}); destroy(b); CHECK(used() < GB);
    } else if (is("malloc_fails")) {  // the idle blocks of this device make room, those of others stay
        go(); device() = 1; G o = make({GB}); destroy(o); device() = 0;
        G a = make({4 * GB, 3 * GB}); destroy(a);
        stub().room = 8 * GB;
        void *p; CHECK(dev_pool().fresh(&p, 6 * GB) == hipSuccess); CHECK(used() == 6 * GB); CHECK(used(1) == GB);
        void *q; CHECK(dev_pool().alloc(&q, 6 * GB) != hipSuccess && q == nullptr);
    } else if (is("in_use")) {  // work may still use it: to the driver, whose free waits
        go(); G a = make({GB}); destroy(a, false); CHECK(used() < GB);
    } else if (is("fit")) {  // only blocks of nearly the size are taken
        go(); G a = make({16 * MB}); destroy(a);
        G b = make({13 * MB}); CHECK(used() >= 29 * MB); destroy(b); dev_pool().release();
        G c = make({MB}); destroy(c); G d = make({16 * MB}); destroy(d);
        const int before = stub().mallocs;
        G e = make({15 * MB - 5}); CHECK(stub().mallocs == before); destroy(e);
    } else if (is("many_live")) {  // blocks beyond the table of live ones are freed, not kept
        go(); G a = make(std::vector<size_t>(1500, MB)); destroy(a); CHECK(used() <= 64 * MB);
    } else if (is("threads")) {
        go();
        std::vector<std::thread> t;
        for (int k = 0; k < 6; ++k) t.emplace_back([k] {
            for (int i = 0; i < 400; ++i) {
                G g = make({(size_t)(1 + (i * 7 + k) % 40) * MB, (size_t)(1 + i % 3) * 100 * MB, 100});
                if (i % 50 == 49) dev_pool().release();
                destroy(g, i % 5 != 0);
            }
        });
        for (auto &x : t) x.join();
        CHECK(used() <= 8 * GB);
        dev_pool().release(); CHECK(used() == 0);
    } else return 2;
    CHECK(!stub().bad_free);
    return 0;
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("pool")
    (d / "hip").mkdir()
    (d / "hip" / "hip_runtime.h").write_text(STUB)
    (d / "main.cpp").write_text(MAIN)
    subprocess.run([CXX, "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-pthread", f"-I{d}",
                    f"-I{os.path.join(ROOT, 'paper_2512_00705_amd', 'csrc')}", str(d / "main.cpp"), "-o",
                    str(d / "pool")], check=True)
    return str(d / "pool")


@pytest.mark.parametrize("case", ["first_graphs", "release", "most", "blocks", "turns", "malloc_fails", "in_use", "fit",
                                  "many_live", "threads"])
def test_pool(program, case):
    r = subprocess.run([program, case], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr
