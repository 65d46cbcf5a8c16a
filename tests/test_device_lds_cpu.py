"""Large LDS is asked for once per kernel and device, and a refusal leaves no error behind (csrc/psb_device_lds.h), with a runtime that counts."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1904_02205_amd", "csrc")

PROGRAM = r"""
#include "psb_device_lds.h"
#include <cstdio>
#define CHECK(x) do { if (!(x)) { std::printf("line %d: %s\n", __LINE__, #x); return 1; } } while (0)
struct Runtime {
    int current = 0, asked[100] = {}, error = 0;
    bool grants[100], knows_device = true;
    size_t last = 0;
    Runtime() { for (bool& g : grants) g = true; }
    bool device(int* d) { if (!knows_device) { error = 1; return false; } *d = current; return true; }
    bool request(size_t bytes) { ++asked[current]; last = bytes; if (!grants[current]) error = 2; return grants[current]; }
    void clear_error() { error = 0; }
};
int main() {
    Runtime r;
    static psb::LdsGrant a, b;
    CHECK(a(65536, r) && r.asked[0] == 0);                           // nothing to ask for
    CHECK(a(65537, r) && a(65537, r) && r.asked[0] == 1 && r.last == 65537);
    r.current = 1;                                                   // a second GPU of the process
    CHECK(a(65537, r) && a(65537, r) && r.asked[1] == 1 && r.asked[0] == 1);
    CHECK(b(159744, r) && r.asked[1] == 2);                          // another kernel
    r.current = 2; r.grants[2] = false;
    CHECK(!a(65537, r) && r.error == 0 && !a(65537, r) && r.asked[2] == 1);
    r.current = 0;
    CHECK(a(65537, r) && r.asked[0] == 1);                           // the other devices keep theirs
    r.current = 70;
    CHECK(a(65537, r) && a(65537, r) && r.asked[70] == 2);
    r.knows_device = false;
    CHECK(!a(65537, r) && r.error == 0);
    return 0;
}
"""


def test_once_per_kernel_and_device(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("no host compiler")
    src, exe = tmp_path / "lds.cpp", tmp_path / "lds"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Wextra", "-Werror", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout


def test_no_launcher_asks_once_per_process():
    """Only the runtime handed to LdsGrant makes the request."""
    for name in sorted(os.listdir(CSRC)):
        with open(os.path.join(CSRC, name)) as f:
            lines = [line for line in f if "hipFuncSetAttribute(" in line]
        assert len(lines) == (1 if name == "psb_kernels_shared.hip.h" else 0) and all("bool request(" in line for line in lines), name
