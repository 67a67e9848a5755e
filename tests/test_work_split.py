"""How launches divide their work, checked on the CPU over sizes that no GPU test allocates: the program below is compiled
against the header the kernels and their launchers use."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _run(tmp_path, body):
    src, exe = tmp_path / "check.cpp", tmp_path / "check"
    src.write_text('#include "qadam_work.h"\n#include <cstdio>\n#include <cstdlib>\n#include <initializer_list>\nusing namespace qadam;\n'
                   '#define CHECK(c, ...) do { if (!(c)) { std::puts(#c); std::printf(__VA_ARGS__); std::exit(1); } } while (0)\n'
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


def test_pieces_cover_every_tile_and_every_workgroup_has_its_own(tmp_path):
    """Both sides of every size at which tiles are cut into fewer pieces, for the two piece lengths in use (256: the main
    pass and the server; 512: the worker quantizer, whose turns the kernel repeats over a longer piece)."""
    _run(tmp_path, """
    for (int turn : {256, 512}) {
        uint32_t most = kTileElems / turn, before = most;
        bool fewer = false;
        for (long long n = 1; n < kMaxTiles; n = n < 70000 ? n + 1 + n / 50 : n + 997) {
            const Items I = wave_items((int)n, turn);
            CHECK(I.parts >= 1 && (long long)I.parts * I.part_len >= kTileElems, "%lld", n);
            CHECK((long long)(I.parts - 1) * I.part_len < kTileElems && I.part_len % turn == 0, "%lld", n);
            CHECK(I.count == (unsigned long long)n * I.parts && I.parts <= before, "%lld", n);
            const unsigned long long blocks = wave_blocks(I);
            CHECK(blocks >= I.count && blocks * 64 < (1ull << 32), "%lld", n);
            fewer = fewer || I.parts < most;
            before = I.parts;
        }
        const Items last = wave_items((int)kMaxTiles - 1, turn);
        CHECK(fewer && last.parts < most && last.parts * last.part_len >= kTileElems, "the sizes do not reach fewer pieces");
    }
    // every item is some workgroup's, and no two workgroups have the same one
    for (int n : {1, 3, 7, 8, 9, 63, 64, 127, 129, 1000, 4095, 4096, 4097, 70001, 300007}) {
        const Items I = wave_items(n, 256);
        const uint32_t blocks = wave_blocks(I);
        unsigned char* seen = (unsigned char*)std::calloc(blocks, 1);
        for (uint32_t b = 0; b < blocks; ++b) {
            const uint32_t item = item_of(I, b);
            CHECK(item < blocks && !seen[item], "%d", n);
            seen[item] = 1;
        }
        std::free(seen);
    }""")
