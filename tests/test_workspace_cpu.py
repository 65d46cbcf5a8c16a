"""Lifetime of the buffers a weight handle keeps between calls (csrc/psb_workspace.h), with an allocator that counts."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1904_02205_amd", "csrc")

PROGRAM = r"""
#include "psb_workspace.h"
#include <cstdio>
#include <cstdlib>
#include <set>
#define CHECK(x) do { if (!(x)) { std::printf("line %d: %s\n", __LINE__, #x); return 1; } } while (0)
struct Device {
    std::set<void*> live;
    int waits = 0;
    bool can_wait = true, can_allocate = true;
    bool allocate(void** p, size_t n) { if (!can_allocate) return false; *p = std::malloc(n); live.insert(*p); return true; }
    void release(void* p) { if (live.erase(p) != 1) std::abort(); std::free(p); }
    bool wait() { ++waits; return can_wait; }
};
using psb::Grow;
int main() {
    Device d;
    psb::WorkspaceMemory m;
    psb::GrownBuffer a, b;
    // eager calls only: the old buffer is waited for and freed
    CHECK(m.reserve(a, 100, false, d) == Grow::ok && a.bytes == 100 && d.waits == 0);
    void* p = a.ptr;
    CHECK(m.reserve(a, 50, false, d) == Grow::ok && a.ptr == p && a.bytes == 100);
    CHECK(m.reserve(a, 200, false, d) == Grow::ok && d.waits == 1 && d.live.size() == 1);
    // captured, then larger eager calls: what the graph uses stays
    CHECK(m.reserve(a, 200, true, d) == Grow::ok);
    p = a.ptr;
    CHECK(m.reserve(a, 300, false, d) == Grow::ok && a.ptr != p && d.live.count(p) && d.live.size() == 2 && d.waits == 1);
    // the next buffer is in no graph: freed as usual; captured again, kept again
    CHECK(m.reserve(a, 400, false, d) == Grow::ok && d.live.size() == 2 && d.waits == 2);
    CHECK(m.reserve(a, 10, true, d) == Grow::ok && m.reserve(a, 500, false, d) == Grow::ok && d.live.size() == 3);
    // other buffers of the handle are not concerned
    CHECK(m.reserve(b, 10, false, d) == Grow::ok && m.reserve(b, 20, false, d) == Grow::ok && d.live.size() == 4 && d.waits == 3);
    // failures leave a buffer that is either whole or empty
    d.can_wait = false;
    p = b.ptr;
    CHECK(m.reserve(b, 30, false, d) == Grow::wait_failed && b.ptr == p && b.bytes == 20);
    d.can_wait = true; d.can_allocate = false;
    CHECK(m.reserve(b, 30, false, d) == Grow::no_memory && !b.ptr && b.bytes == 0);
    CHECK(m.reserve(a, 10, true, d) == Grow::ok);
    p = a.ptr;
    CHECK(m.reserve(a, 600, false, d) == Grow::no_memory && !a.ptr && a.bytes == 0 && d.live.count(p));
    d.can_allocate = true;
    CHECK(m.reserve(a, 600, false, d) == Grow::ok && !a.recorded);
    m.release(a, d); m.release(b, d); m.release_retired(d); m.release_retired(d);
    CHECK(d.live.empty());
    return 0;
}
"""


def test_a_buffer_in_a_graph_outlives_growth(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("no host compiler")
    src, exe = tmp_path / "workspace.cpp", tmp_path / "workspace"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Wextra", "-Werror", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
