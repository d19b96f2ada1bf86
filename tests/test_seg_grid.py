"""Grid of the short segments' launch: every segment count that a batch may have gets at least the workgroups it
needs, up to 2^32 - 2 segments, where rounding up in 32 bits would wrap to an empty launch."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = """
#include "segmented.hpp"
using evosort::seg_wave_groups;
static_assert(seg_wave_groups(0) == 0 && seg_wave_groups(1) == 1 && seg_wave_groups(4) == 1, "");
static_assert(seg_wave_groups(5) == 2 && seg_wave_groups(8) == 2 && seg_wave_groups(100001) == 25001, "");
static_assert(seg_wave_groups(0xfffffffcu) == 0x3fffffffu, "");
static_assert(seg_wave_groups(0xfffffffdu) == 0x40000000u, "");
static_assert(seg_wave_groups(0xfffffffeu) == 0x40000000u, "");
"""


def test_groups_of_a_batch():
    cmd = ["g++", "-std=c++17", "-fsyntax-only", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
           "-I" + os.path.join(ROOT, "paper_2505_18681_amd", "csrc"), "-x", "c++", "-"]
    r = subprocess.run(cmd, input=SOURCE, text=True, capture_output=True, timeout=120)
    assert r.returncode == 0, r.stderr
