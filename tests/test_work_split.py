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
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-Wno-unused", "-I", inc, "-o", str(exe), str(src)], check=True)
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


SHAPES = """
    // n tiles of `len` elements, and the same behind n / 100 whole ones
    const int lens[] = {1, 10, 255, 256, 257, 600, 1000, 1024, 1025, 2048, 2049, 4095, 4096};
    auto shape = [](long long n, int len, bool mixed) {
        ListShape s{};
        const long long whole = mixed ? n / 100 : 0;
        add_tiles(s, whole, kTileElems);
        add_tiles(s, n - whole, len);
        return s;
    };
    auto next = [](long long n) { return n < 70000 ? n + 1 + n / 20 : n + 9973; };
"""


def test_pieces_cover_every_tile_in_a_launch_that_fits(tmp_path):
    """For the piece lengths in use (256: the main pass and the server; 512: the worker quantizer, whose turns the kernel
    repeats over a longer piece; 1024: variant W's first pass), over both sides of every size at which pieces change."""
    _run(tmp_path, SHAPES + """
    int fewest = 16, most = 0;
    for (int len : lens) for (int mixed = 0; mixed < 2; ++mixed)
        for (long long n = 1; n < kMaxTiles; n = next(n)) {
            const ListShape s = shape(n, len, mixed);
            CHECK(s.num_tiles == n && (n < 100 || !mixed || s.longest == kTileElems), "%lld x %d", n, len);
            for (int turn : {256, 512, 1024}) {
                const Items I = wave_items(s, turn);
                const Cut c = turn == 1024 ? moment_cut(s) : I.cut;
                CHECK(c.parts >= 1 && (long long)c.parts * c.part_len >= s.longest, "%lld x %d, turn %d", n, len, turn);
                CHECK(((long long)c.parts - 1) * c.part_len < s.longest && c.part_len % turn == 0 && c.part_len <= kTileElems,
                      "%lld x %d, turn %d", n, len, turn);
                if (turn == 1024) {
                    CHECK((unsigned long long)n * c.parts * 256 < (1ull << 32), "%lld x %d", n, len);
                    continue;
                }
                const unsigned long long blocks = wave_blocks(I);
                CHECK(I.count == (unsigned long long)n * c.parts && blocks >= I.count && blocks * 64 < (1ull << 32),
                      "%lld x %d, turn %d", n, len, turn);
                if (len == kTileElems && turn == 256) {
                    fewest = c.parts < (uint32_t)fewest ? (int)c.parts : fewest;
                    most = (int)c.parts > most ? (int)c.parts : most;
                }
            }
        }
    CHECK(most == 16 && fewest < 8, "the sizes do not reach fewer pieces");""")


def test_no_launch_is_mostly_empty(tmp_path):
    """Beyond what fills the chip, at most every second wavefront finds nothing to do."""
    _run(tmp_path, SHAPES + """
    for (int len : lens) for (int mixed = 0; mixed < 2; ++mixed)
        for (long long n = 1; n < kMaxTiles; n = next(n))
            for (int turn : {256, 512}) {
                const ListShape s = shape(n, len, mixed);
                const Items I = wave_items(s, turn);
                int k = 0;
                while ((256 << k) < I.cut.part_len) ++k;
                CHECK(I.count <= 2 * s.pieces[k] || s.pieces[k + 1] < kFullChip, "%lld x %d, turn %d", n, len, turn);
            }""")


def test_every_workgroup_has_an_item_of_its_own(tmp_path):
    _run(tmp_path, SHAPES + """
    for (int n : {1, 3, 7, 8, 9, 63, 64, 127, 129, 1000, 4095, 4096, 4097, 70001, 300007}) {
        const Items I = wave_items(shape(n, kTileElems, false), 256);
        const uint32_t blocks = wave_blocks(I);
        unsigned char* seen = (unsigned char*)std::calloc(blocks, 1);
        for (uint32_t b = 0; b < blocks; ++b) {
            const uint32_t item = item_of(I, b);
            CHECK(item < blocks && !seen[item], "%d", n);
            seen[item] = 1;
        }
        std::free(seen);
    }""")


def test_scale_pass_has_a_workgroup_for_every_tile(tmp_path):
    """And the tile's workgroup is on the XCD of the wavefronts that quantize it, where those of one tile are on one."""
    _run(tmp_path, SHAPES + """
    for (int n : {1, 7, 8, 16, 17, 127, 128, 129, 512, 1000, 4095, 4097, 70001}) {
        const ListShape s = shape(n, kTileElems, false);
        const Items I = scan_items(s), q = wave_items(s, 512), f = wave_items(s, 256);
        const uint32_t blocks = wave_blocks(I);
        CHECK(scan_fits(I) && I.count == (uint32_t)n, "%d", n);
        unsigned char* seen = (unsigned char*)std::calloc(blocks, 1);
        int* xcd = (int*)std::calloc(n, sizeof(int));
        for (uint32_t b = 0; b < blocks; ++b) {
            const uint32_t tile = item_of(I, b);
            CHECK(tile < blocks && !seen[tile], "%d", n);
            seen[tile] = 1;
            if (tile < I.count) xcd[tile] = (int)(b & 7);
        }
        for (const Items& w : {q, f})
            for (uint32_t b = 0; b < wave_blocks(w); ++b) {
                const uint32_t item = item_of(w, b);
                if (item < w.count && n >= 128 && n <= 2048)
                    CHECK(xcd[item / w.cut.parts] == (int)(b & 7), "%d tiles, item %u", n, item);
            }
        std::free(seen);
        std::free(xcd);
    }
    CHECK(!scan_fits(scan_items(shape(kMaxTiles - 1, 1, false))), "the largest list");""")


def test_short_layers_have_a_workgroup_that_holds_them(tmp_path):
    _run(tmp_path, """
    const int counts[] = {0, 1, 255, 256, 319, 320, 2047, 2048, 1 << 20, (1 << 24) - 4097, (1 << 24) - 1};
    const int holds[kShortSizes] = {256, 1024, 4096}, threads[kShortSizes] = {64, 256, 256};
    int taken = 0;
    for (int a : counts) for (int b : counts) for (int c : counts) for (int longer : {0, 5}) for (int N : {1, 8, 9, 32}) {
        const long long n = (long long)a + b + c;
        if (n + longer >= kMaxTiles) continue;
        ShortLayers have{};
        have.num[0] = a; have.num[1] = b; have.num[2] = c;
        const ShortLayers s = short_layers_apart(have, n + longer, N);
        CHECK((long long)s.num[0] + s.num[1] + s.num[2] == (s.any() ? n : 0), "%d %d %d", a, b, c);
        if (!s.any()) continue;
        ++taken;
        int left[kShortSizes] = {s.num[0], s.num[1], s.num[2]};
        for (int k = 0; k < kShortSizes; ++k) {
            CHECK(s.as[k] >= k && holds[s.as[k]] >= holds[k], "%d %d %d", a, b, c);
            left[s.as[k]] -= have.num[k];
            const Items I = layer_items(s.num[k]);
            CHECK((unsigned long long)wave_blocks(I) * threads[k] < (1ull << 32) && wave_blocks(I) >= (unsigned)s.num[k], "%d", s.num[k]);
        }
        CHECK(!left[0] && !left[1] && !left[2], "%d %d %d", a, b, c);
    }
    CHECK(taken > 100, "%d", taken);
    for (int len = 1; len <= kTileElems; ++len) CHECK(len <= holds[short_size(len)], "%d", len);""")


def test_flat_launches_cover_the_longest_vector(tmp_path):
    """Vectors have up to 2^36 elements (tiles of 4096 below 2^24); x counts work-items below 2^32, y stays below 2^16."""
    _run(tmp_path, """
    for (int threads : {64, 256}) for (int per : {256, 512, 2048, 4096, 8192})
        for (long long n : {1ll, 255ll, 256ll, 257ll, (1ll << 31) - 1, (1ll << 33) - 1, 1ll << 33, (1ll << 33) + 1, (1ll << 36) - 1}) {
            const FlatGrid g = flat_blocks(n, threads, per);
            const unsigned long long blocks = (unsigned long long)g.x * g.y;
            CHECK(g.x >= 1 && (unsigned long long)g.x * threads < (1ull << 32) && g.y < (1u << 16), "%lld", n);
            CHECK(blocks * per >= (unsigned long long)n && blocks * per < n + (unsigned long long)g.x * per, "%lld", n);
        }""")


def test_server_by_section_where_one_launch_would_be_sparse(tmp_path):
    _run(tmp_path, """
    const auto list = [](int whole, int rest, int tiny, int len) {
        ListShape s{}; add_tiles(s, whole, kTileElems); if (rest) add_tiles(s, whole / 2, rest); add_tiles(s, tiny, len); return s; };
    CHECK(server_by_section(list(500, 0, 8000, 64), true) && !server_by_section(list(500, 0, 8000, 64), false), "tiles alone");
    CHECK(server_by_section(list(800, 809, 8400, 64), true), "beside longer layers");
    CHECK(!server_by_section(list(20000, 0, 0, 1), true) && !server_by_section(list(0, 0, 20000, 1000), true), "uniform");
    CHECK(!server_by_section(list(30, 0, 330, 64), true), "too few to fill the chip");""")


def test_units_cover_a_parked_layer(tmp_path):
    """Chunk c of a layer is in unit c mod n, and no unit has more chunks than a unit holds; the workgroups that are there, with
    the two units or three that each holds, can hold the longest layer, its units fit the counts of arrivals and departures, and it has
    no more polled copies of the scale than one wavefront writes."""
    _run(tmp_path, """
    const int unit = kParkedChunk * kParkedChunks;
    for (int64_t len : {(int64_t)1, (int64_t)kParkedChunk, (int64_t)kParkedChunk + 1, (int64_t)unit, (int64_t)unit + 1, (int64_t)9 * unit - 1,
                        kParkedLongest - 1, kParkedLongest, kParkedLongest + 1, (int64_t)512 * unit, (int64_t)512 * unit + 1,
                        kParkedLongestOfThree - 1, kParkedLongestOfThree}) {
        const int n = parked_units(len), held = len > kParkedLongest ? 3 : 2;
        const int64_t chunks = (len + kParkedChunk - 1) / kParkedChunk;
        for (int u = 0; u < n; ++u) CHECK((chunks - u + n - 1) / n >= 1 && (chunks - u + n - 1) / n <= kParkedChunks, "%lld", (long long)len);
        CHECK(n < held * kParkedGroups && (held == 3 || n < kParkedGroups) && (unsigned)n <= kArrivals && (uint64_t)n * kDeparture < (1ull << 32), "%lld", (long long)len);
        CHECK(meeting_copies(n) >= 1 && meeting_copies(n) <= 64, "%lld", (long long)len);
        CHECK(meeting_words(n) == (n > 1 ? (1 + meeting_copies(n)) * kMeetingLine : 0), "%lld", (long long)len);
    }
    const int64_t M = 1 << 20;
    CHECK(worth_parking(8 * M, 512, 8 * M, 1, false) && !worth_parking(8 * M - 1, 512, 8 * M, 1, false), "one worker");
    CHECK(worth_parking(12 * M, 768, 12 * M, 1, false, false, kParkedLongest + 1) && !worth_parking(12 * M - 1, 768, 12 * M, 1, false, false, kParkedLongest + 1) &&
          worth_parking(8 * M, 512, 8 * M, 1, false, false, kParkedLongest), "one worker, three units");
    CHECK(worth_parking(6 * M, 384, 12 * M, 4, false) && !worth_parking(6 * M - 1, 384, 6 * M, 4, false), "four workers");
    CHECK(worth_parking(12 * M, 768, 48 * M, 4, false) && !worth_parking(12 * M - 1, 768, 24 * M, 4, false), "beside a longer layer");
    CHECK(!worth_parking(12 * M, 768, 48 * M + 1, 4, false), "beside a much longer layer");
    CHECK(worth_parking(12 * M, 768, 12 * M, 4, true) && !worth_parking(12 * M - 1, 768, 12 * M, 4, true), "stochastic");
    CHECK(worth_parking(18 * M, 4000, 18 * M, 4, false) && !worth_parking(18 * M - 1, 4000, 18 * M, 4, false), "mostly empty units");""")


def test_a_parked_launch_has_a_unit_for_every_workgroup(tmp_path):
    """A workgroup's first unit is the one of its own number."""
    _run(tmp_path, """
    const int64_t unit = kParkedChunk * kParkedChunks;
    for (int num = 1; num <= 32; ++num) for (int stochastic = 0; stochastic < 2; ++stochastic)
        for (int64_t units = 1; units <= 2 * kParkedGroups; ++units) for (int64_t elems : {units, units * unit / 2, units * unit})
            CHECK(!(worth_parking(elems, units, elems, num, stochastic) || worth_parking(elems, units, elems, num, stochastic, true)) || units * num >= kParkedGroups, "%lld", (long long)units);""")


def test_buffers_dealt_to_two_groups_are_recognized(tmp_path):
    """The distance of the groups is found from the addresses of the buffers that a call has; a buffer that lies elsewhere is
    noticed, whichever it is."""
    _run(tmp_path, """
    auto bytes = [](Buffer b) { return arena_round(b == Buffer::codes ? 300 << 20 : b == Buffer::wcodes ? 700 << 20 : b == Buffer::scales ? 100 : (uint64_t)3 << 30); };
    for (int N : {1, 2, 3, 8, 32}) for (int w = 0; w < 2; ++w) for (uint64_t apart : {(uint64_t)200 << 30, (uint64_t)500 << 30}) {
        uint64_t place[11][32] = {}, fill[2] = {0, 0};
        int dealt = 0;
        deal_buffers(N, w, [&](Buffer b, int i, int group) {
            place[(int)b][i] = (1ull << 44) + group * apart + fill[group];
            fill[group] += bytes(b);
            ++dealt;
        });
        CHECK(dealt == 5 + (w ? 6 : 4) * N, "%d of %d", dealt, N);
        for (int moved = -1; moved < 8; ++moved) {
            const bool used = moved < 0 || w || (moved != (int)Buffer::mw && moved != (int)Buffer::vw);
            if (!used) continue;
            auto at = [&](Buffer b, int i) -> uint64_t {
                if (b >= Buffer::codes || (w && (b == Buffer::m || b == Buffer::v))) return 0;
                return place[(int)b][i] + ((int)b == moved && i == (b >= Buffer::err ? N - 1 : 0) ? kArenaAlign : 0);
            };
            const bool counts = moved >= 0 && !(w && (moved == (int)Buffer::m || moved == (int)Buffer::v));
            CHECK(groups_apart(N, w, bytes, at) == (counts ? 0 : (int64_t)apart), "%d workers, moved %d", N, moved);
        }
    }""")


def test_where_the_whole_step_goes_by_worker(tmp_path):
    """Both sides of the lines, which lie further out off the 16-byte grid, for many workers and for variant W."""
    _run(tmp_path, """
    const int64_t M = 1 << 20;
    auto grid = [&](int64_t n, int num) { return worth_by_worker(n, 0, num, false, false); };
    auto off = [&](int64_t n, int num) { return worth_by_worker(n, n, num, false, true); };
    auto w = [&](int64_t n, int num) { return worth_by_worker(n, 0, num, true, false); };
    auto w_off = [&](int64_t n, int num) { return worth_by_worker(n, n, num, true, false); };
    CHECK(grid(24 * M + 1, 1) && !grid(24 * M, 1) && grid(24 * M + 1, 4) && !grid(24 * M, 4), "one worker, four");
    CHECK(grid(12 * M + 1, 8) && !grid(12 * M, 8) && grid(14 * M, 16) && !grid(14 * M - 1, 16), "eight, sixteen");
    CHECK(off(128 * M, 1) && !off(128 * M - 1, 1) && off(48 * M + 1, 2) && !off(48 * M, 2), "one worker off the grid, two");
    CHECK(off(54 * M, 3) && !off(53 * M, 3) && off(48 * M, 4) && !off(48 * M - 1, 4), "off the grid");
    CHECK(off(40 * M, 8) && !off(40 * M - 1, 8) && !off(400 * M, 9) && !off(400 * M, 16), "off the grid, many workers");
    CHECK(!worth_by_worker(25 * M, 13 * M, 4, false, false) && worth_by_worker(25 * M, 12 * M, 4, false, false), "half of it off the grid");
    CHECK(w(128 * M + 1, 1) && !w(128 * M, 1) && w(32 * M + 1, 4) && !w(32 * M, 4), "variant W");
    CHECK(w(50 * M, 8) && !w(50 * M - 1, 8) && w(50 * M, 16) && !w(50 * M - 1, 16) && !w(400 * M, 5), "variant W, many workers");
    CHECK(w_off(128 * M + 1, 1) && w_off(64 * M + 1, 2) && !w_off(64 * M, 2) && !w_off(400 * M, 3), "variant W off the grid");
    CHECK(!worth_by_worker(400 * M, 0, 4, true, true), "variant W, stochastic rounding");""")


def test_lines_of_parking_for_a_separate_call_and_stochastic_rounding(tmp_path):
    _run(tmp_path, """
    const int64_t M = 1 << 20, unit = kParkedChunk * kParkedChunks;
    auto call = [&](int64_t elems, bool stochastic, int64_t longest = 1 << 20) {
        return worth_parking(elems, (elems + unit - 1) / unit, elems, 1, stochastic, true, longest);
    };
    CHECK(!call(8 * M, false) && !call(12 * M, false) && !call(20 * M, false) && !call(22 * M, false), "turns partly empty, or one");
    CHECK(call(15 * M, false) && call(16 * M, false) && !call(16 * M + 1, false) && call(24 * M, false) && call(25 * M, false), "full turns, many");
    CHECK(call(16 * M, false, kParkedLongest) && !call(16 * M, false, kParkedLongest + 1) && !call(24 * M - 1, false, 16 * M) &&
          call(24 * M, false, 16 * M), "a call whose layers need a third unit");
    CHECK(call(64 * M, true) && !call(64 * M - 1, true), "stochastic");
    CHECK(worth_parking(32 * M, 2048, 32 * M, 2, true) && !worth_parking(32 * M - 1, 2048, 32 * M, 2, true), "two workers");
    CHECK(worth_parking(12 * M, 768, 24 * M, 8, true) && !worth_parking(12 * M - 1, 768, 24 * M, 8, true), "beside longer layers");""")


def test_lines_of_parking_in_variant_w(tmp_path):
    _run(tmp_path, """
    const int64_t M = 1 << 20, unit = kParkedChunk * kParkedChunks;
    auto parks = [](int64_t elems, int64_t all, int num, bool stochastic, int64_t longest) {
        return worth_parking_w(elems, (elems + unit - 1) / unit, all, num, stochastic, longest);
    };
    CHECK(parks(48 * M, 48 * M, 1, false, M) && !parks(48 * M - 1, 48 * M, 1, false, M), "one worker");
    CHECK(parks(10 * M, 30 * M, 4, false, M) && !parks(10 * M - 1, 10 * M, 4, false, M) && !parks(10 * M, 30 * M + 1, 4, false, M), "four workers");
    CHECK(parks(18 * M, 18 * M, 4, true, M) && !parks(18 * M - 1, 18 * M, 4, true, M), "stochastic");
    CHECK(parks(20 * M, 20 * M, 4, false, kParkedLongest + 1) && !parks(20 * M - 1, 20 * M, 4, false, kParkedLongest + 1), "three units");
    CHECK(!worth_parking_w(20 * M, 4000, 20 * M, 4, false, 5000), "mostly empty units");
    for (int num = 1; num <= 32; ++num)
        for (int64_t units = 1; units <= 2 * kParkedGroups; ++units)
            CHECK(!worth_parking_w(units * unit, units, units * unit, num, false, M) || units * num >= kParkedGroups, "a unit for every workgroup");""")


def _c_list(sizes):
    return "{" + ", ".join("%d" % n for n in sizes) + "}"


def test_the_lists_of_the_gpu_tests_lie_on_both_sides_of_the_rules(tmp_path):
    """The lists with which the GPU tests of the step by worker and of parked layers compare the ways that a step can take."""
    import test_gpu_by_worker as by
    import test_gpu_parked as parked
    body = """
    struct Counts { int64_t all, elems, units, off, longest; };
    auto count = [](std::initializer_list<int64_t> sizes) {
        Counts c{};
        for (int64_t n : sizes) {
            if (c.all % 4 != 0) c.off += n;
            if (n <= kParkedLongestOfThree) { c.elems += n; c.units += parked_units(n); c.longest = n > c.longest ? n : c.longest; }
            c.all += n;
        }
        return c;
    };
    auto parks = [](const Counts& c, int num, bool stochastic, bool call = false) {
        return worth_parking(c.elems, c.units, c.all, num, stochastic, call, c.longest);
    };
    auto parks_w = [](const Counts& c, int num, bool stochastic) {
        return worth_parking_w(c.elems, c.units, c.all, num, stochastic, c.longest);
    };"""
    for kind in by.LAST:
        for more in (0, 1):
            body += """
    for (int stochastic = 0; stochastic < 2; ++stochastic) {
        const Counts c = count(%s);
        CHECK(%d || !parks(c, %d, stochastic), "%s");
        CHECK(worth_by_worker(c.all, c.off, %d, %d, stochastic) == (%d && !(%d && stochastic)), "%s %d");
    }""" % (_c_list(by.sizes_of(kind, more)), kind == "w", by.N, kind, by.N, kind == "w", more, kind == "w", kind, more)
    for stochastic in (0, 1):
        for less in (0, 1):
            body += """
    CHECK(parks(count(%s), %d, %d) == %d, "parked, %d");""" % (
                _c_list(parked._sizes((1 + stochastic) * parked.LEAST - less)), parked.N, stochastic, 1 - less, less)
    for sizes in (parked.SIZES, *parked.ON_FOUR_STREAMS):
        body += """
    CHECK(parks(count(%s), 1, false, true), "separate calls");""" % _c_list(sizes)
    for sizes, workers, _, scanned in parked.ORACLE:
        body += """
    { const Counts c = count(%s); CHECK((parks(c, %d, false) ? c.all - c.elems : c.all) == %d, "against the oracle"); }""" % (
            _c_list(sizes), workers, scanned)
    for sizes, stochastic in parked.W_CALLS:
        body += """
    CHECK(parks_w(count(%s), 1, %d) && !parks_w(count(%s), 1, %d), "one worker's call of variant W");""" % (
            _c_list(sizes), stochastic, _c_list(parked.beside_longer(sizes)), stochastic)
    _run(tmp_path, body)
