"""Per-device set-up of the kernels (csrc/once_per_device.h), on the host: a second device, and a set-up that fails at first."""
import os
import re
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2506_19505_amd", "csrc")

PROGRAM = r"""
#include "once_per_device.h"
#include <cstdio>
int main()
{
    antkv::OncePerDevice once;
    int calls = 0, status = 0;
    auto on = [&](int device) { return once(device, [&] { ++calls; return status; }); };
    if (on(0) != 0 || on(0) != 0 || calls != 1) return std::printf("device 0: %d calls\n", calls), 1;
    if (on(1) != 0 || calls != 2) return std::printf("device 1: %d calls\n", calls), 2;
    status = 7;
    if (on(63) != 7 || on(63) != 7 || calls != 4) return std::printf("failing: %d calls\n", calls), 3;
    if (on(0) != 0 || calls != 4) return 4;
    status = 0;
    if (on(63) != 0 || on(63) != 0 || calls != 5) return std::printf("after a failure: %d calls\n", calls), 5;
    if (on(64) != 0 || on(64) != 0 || on(-1) != 0 || calls != 8) return std::printf("beyond the mask: %d calls\n", calls), 6;
    return 0;
}
"""


def test_set_up_once_per_device(tmp_path):
    src, exe = tmp_path / "once.cpp", tmp_path / "once"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    done = subprocess.run([str(exe)], capture_output=True, text=True)
    assert done.returncode == 0, done.stdout


def test_no_kernel_attribute_is_set_once_per_process():
    for name in sorted(os.listdir(CSRC)):
        text = open(os.path.join(CSRC, name)).read()
        assert not re.search(r"static\s+const\s+hipError_t", text), f"{name}: a status kept for the whole process"
