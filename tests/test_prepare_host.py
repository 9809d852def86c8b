"""What a kernel needs before its first launch is done once per kernel and
device, from any thread: prepare_kernel against a stand-in runtime on the CPU,
and no launcher that keeps such a fact in a flag for all devices."""
import glob
import os
import re
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1805_08166_amd", "csrc")

FAKE = r"""
#include <cstdio>
#include <thread>
#include <vector>
#include "at_internal.h"

static thread_local int device = 0;
static std::atomic<int> limits[128], queries;
static size_t shared = 0;
static bool fail_next = false;
extern "C" hipError_t hipGetDevice(int* d) { *d = device; return hipSuccess; }
extern "C" hipError_t hipFuncGetAttributes(hipFuncAttributes* a, const void*) {
    ++queries;
    a->sharedSizeBytes = shared;
    return hipSuccess;
}
extern "C" hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int bytes) {
    if (fail_next) { fail_next = false; return hipErrorInvalidValue; }
    limits[device] += bytes == 4096 ? 1 : 1000;
    return hipSuccess;
}
#define CHECK(c) do { if (!(c)) { std::printf("line %d: %s\n", __LINE__, #c); return 1; } } while (0)
int main() {
    int fn = 0;
    std::atomic<uint64_t> done{0}, other{0}, shy{0};
    for (int round = 0; round < 3; ++round)
        for (int d : {0, 1, 63, 64, 100}) {
            device = d;
            CHECK(at::prepare_kernel(&fn, -1, 4096, done) == hipSuccess);
        }
    // once on each of the devices that have a bit, every time beyond
    CHECK(limits[0] == 1 && limits[1] == 1 && limits[63] == 1 && limits[64] == 3 && limits[100] == 3);
    CHECK(queries == 0);
    // another kernel's word is another matter
    device = 1;
    CHECK(at::prepare_kernel(&fn, -1, 4096, other) == hipSuccess && limits[1] == 2);
    // a failure is not remembered as done
    device = 5;
    fail_next = true;
    CHECK(at::prepare_kernel(&fn, -1, 4096, done) == hipErrorInvalidValue && limits[5] == 0);
    CHECK(at::prepare_kernel(&fn, -1, 4096, done) == hipSuccess && limits[5] == 1);
    // static LDS: checked, on each device, and no limit raised when none is asked for
    shared = 16;
    CHECK(at::prepare_kernel(&fn, 0, 4096, shy) == hipErrorInvalidKernelFile && limits[5] == 1);
    CHECK(at::prepare_kernel(&fn, 16, 0, shy) == hipSuccess && limits[5] == 1 && queries == 2);
    CHECK(at::prepare_kernel(&fn, 16, 0, shy) == hipSuccess && queries == 2);
    // threads on two devices at once
    std::atomic<uint64_t> both{0};
    std::vector<std::thread> ts;
    for (int t = 0; t < 8; ++t)
        ts.emplace_back([&, t] {
            device = 10 + t % 2;
            for (int i = 0; i < 1000; ++i) (void)at::prepare_kernel(&fn, -1, 4096, both);
        });
    for (auto& t : ts) t.join();
    CHECK(limits[10] >= 1 && limits[10] <= 4 && limits[11] >= 1 && limits[11] <= 4 && both == (3ull << 10));
    std::printf("ok\n");
    return 0;
}
"""


def test_once_per_kernel_and_device(tmp_path):
    src, exe = tmp_path / "fake.cpp", tmp_path / "fake"
    src.write_text(FAKE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-pthread", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I", CSRC,
                    str(src), os.path.join(CSRC, "at_prepare.cpp"), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert out.returncode == 0 and out.stdout == "ok\n", out.stdout + out.stderr


def test_no_launcher_keeps_a_flag_for_all_devices():
    for path in sorted(glob.glob(os.path.join(CSRC, "*.hip")) + glob.glob(os.path.join(CSRC, "*.cpp"))):
        with open(path) as f:
            assert not re.search(r"\bstatic\s+bool\b", f.read()), os.path.basename(path)
