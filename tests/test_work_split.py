"""How launches divide their work, checked on the CPU over sizes that no GPU test allocates: the program below is compiled
against the header the kernels and their launchers use."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _run(tmp_path, body):
    src, exe = tmp_path / "check.cpp", tmp_path / "check"
    src.write_text('#include "qadam_work.h"\n#include <cstdio>\n#include <cstdlib>\nusing namespace qadam;\n'
                   '#define CHECK(c, ...) do { if (!(c)) { std::printf(#c ": " __VA_ARGS__); std::exit(1); } } while (0)\n'
                   "int main() {\n" + body + "\nreturn 0; }\n")
    inc = os.path.join(ROOT, "paper_2004_14180_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I", inc, "-o", str(exe), str(src)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout


def test_every_layer_has_a_workgroup_in_a_launch_that_fits(tmp_path):
    """One dimension of a launch holds fewer than 2^32 work-items; with 2^24 tiles at most, a list has up to 2^24 layers
    that are not empty."""
    _run(tmp_path, """
    const long long sizes[] = {1, 15, 16, 17, 1023, 1024, 1025, 65537, (1 << 22) - 1, 1 << 22, (1 << 22) + 1,
                               kMaxTiles - 1, kMaxTiles};
    for (long long L : sizes)
        for (int num = 1; num <= 32; ++num) {
            const unsigned long long blocks = reduce_blocks((int)L, num);
            const int per = reduce_by_list((int)L, num) ? kListLayers : 1;
            CHECK(blocks * per >= (unsigned long long)L && (blocks - 1) * per < (unsigned long long)L, "L %lld num %d", L, num);
            CHECK(blocks * kReduceThreads < (1ull << 32), "L %lld num %d", L, num);
        }""")
