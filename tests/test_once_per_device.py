"""The host helper that sets a kernel's LDS limit: once on every device, not once per process.  CPU only."""
import os
import re
import subprocess
import tempfile

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include <thread>
#include <vector>
#include "once_per_device.h"
int main() {
    moe::OncePerDevice once;
    int calls[80] = {};
    for (int device : {0, 1, 0, 1, 63, 0, 63, 70, 70}) once.run(device, [&] { ++calls[device]; });
    if (calls[0] != 1 || calls[1] != 1 || calls[63] != 1 || calls[70] != 2) return 1;
    moe::OncePerDevice shared;                       // nobody goes on before it has been done on its device
    std::atomic<int> set[4] = {{0}, {0}, {0}, {0}}, early{0};
    std::vector<std::thread> threads;
    for (int i = 0; i < 16; ++i)
        threads.emplace_back([&, device = i % 4] {
            for (int n = 0; n < 1000; ++n) {
                shared.run(device, [&] { set[device] = 1; });
                if (!set[device]) ++early;
            }
        });
    for (auto& t : threads) t.join();
    return early ? 2 : 0;
}
"""


def test_once_on_every_device():
    with tempfile.TemporaryDirectory() as tmp:
        src, exe = os.path.join(tmp, "t.cpp"), os.path.join(tmp, "t")
        with open(src, "w") as f:
            f.write(PROGRAM)
        subprocess.run(["g++", "-std=c++17", "-O1", "-pthread", "-I", os.path.join(ROOT, "paper_2504_14960_amd", "csrc"),
                        "-o", exe, src], check=True)
        assert subprocess.run([exe], timeout=60).returncode == 0


def test_no_launch_keeps_a_process_wide_flag():
    """A kernel with more than 64 KiB of LDS needs its limit set on whatever device is current: every launch goes through the
    helper, with a once-per-device flag of its own for each kernel that it chooses from."""
    csrc = os.path.join(ROOT, "paper_2504_14960_amd", "csrc")
    calls = []
    for name in sorted(os.listdir(csrc)):
        text = open(os.path.join(csrc, name)).read()
        assert "static bool" not in re.sub(r"static bool \w+\(", "", text), name     # functions apart
        calls += [name] * text.count("hipFuncSetAttribute(")
    assert calls == ["common.h"], calls


def test_streaming_kernels_keep_no_process_wide_flag():
    """fp32 and odd-size layers run on these kernels on whatever device is current."""
    text = open(os.path.join(ROOT, "paper_2504_14960_amd", "csrc", "gemm_stream.hip")).read()
    assert "static bool" not in text
