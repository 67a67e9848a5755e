// How the kernels' work is divided over their launches: arithmetic that the host and the kernels share.  Plain C++, so
// that it can be checked on the CPU at sizes no test allocates.
#pragma once

#include <stdint.h>

namespace qadam {

constexpr int64_t kMaxTiles = (int64_t)1 << 24;     // a handle has fewer: one 256-thread workgroup per tile must fit a launch
constexpr int kTileElems = 4096;                     // elements per tile (16 per lane of a 256-thread workgroup)

// ---- how a list of layers is cut into pieces -------------------------------------------------------------------------
// What the cut depends on.  Tiles are not all whole: the last one of a layer holds the rest, and a list of short layers
// has no other.
struct ListShape {
    int32_t num_tiles;
    int32_t longest;            // elements of the longest tile
    int64_t pieces[5];          // [k]: pieces of 256 << k elements, counted from the beginning of each tile, with an element
};

constexpr void add_tiles(ListShape& s, int64_t tiles, int len)
{
    s.num_tiles += (int32_t)tiles;
    if (tiles > 0 && len > s.longest) s.longest = len;
    for (int k = 0; k < 5; ++k) s.pieces[k] += tiles * ((len + (256 << k) - 1) / (256 << k));
}

// A launch gives every tile the same number of pieces of the same length.
struct Cut {
    uint32_t parts;             // pieces per tile
    int32_t  part_len;          // elements per piece; parts * part_len covers the longest tile
};

constexpr int64_t kFullChip = 8192;     // pieces that fill the chip: 256 CUs with 16 wavefronts, twice

// Pieces of `turn` elements (256 << k), as many as the longest tile has.  They are twice as long where the launch would
// have more than `most` of them, and where its empty ones, behind the end of shorter tiles, cost more than the rest while
// longer ones still fill the chip (`empty_cost`: of an empty piece against one with elements).  us per step of 4 workers,
// pieces of `turn` / this rule / whole tiles: GPT-2 small 2292 / 2292 / 2584; 5000 times layers of 4096 and 64 elements
// 435 / 434 / 597; 4000 times 4096 and four of 64 484 / 417 / 432; 3000 times 4096 and eight of 64 580 / 448 / 430; one of
// 40 M and 20000 of 100 1040 / 1000 / 967.  With sixteen pieces for every tile, however short the longest is:
// 100000 layers of 100 1565, with one 719.
constexpr Cut cut_tiles(const ListShape& s, int turn, int64_t most, double empty_cost)
{
    Cut c{1, turn};
    int k = 0;
    while ((256 << k) < turn) ++k;
    for (;; ++k, c.part_len *= 2) {
        c.parts = s.longest > c.part_len ? (uint32_t)((s.longest + c.part_len - 1) / c.part_len) : 1u;
        if (c.part_len >= kTileElems) return c;
        const int64_t items = (int64_t)s.num_tiles * c.parts;
        const bool sparse = (double)(items - s.pieces[k]) * empty_cost > (double)s.pieces[k] && s.pieces[k + 1] >= kFullChip;
        if (items <= most && !sparse) return c;
    }
}

// The pieces of the first pass of variant W: one 256-thread workgroup and one maximum each.  An empty one is four
// wavefronts and a barrier.  us per step of 4 workers, pieces of 1024 / 2048 elements: 5000 times layers of 4096 and 64
// (0.6 empty pieces of 1024 to one with elements) 728 / 770, 4000 of 5000 elements (0.6) 646 / 671; of 2048 / 4096: 4000
// times 4096 and four of 64 (0.67) 661 / 615, 3000 times 4096 and eight of 64 (0.8) 720 / 613.
constexpr Cut moment_cut(const ListShape& s) { return cut_tiles(s, 1024, kMaxTiles - 1, 1.6); }

// ---- work items of the kernels whose workgroups are single wavefronts ------------------------------------------------
// (the main pass, the worker quantizer, the server): every piece of a tile is one workgroup.  Wavefronts that share a
// workgroup start together and then load and store in step, and the next four start when the last of them has ended; on
// their own they drift apart, so reads and writes mix, and the workgroups in flight cover a narrower stretch of each of
// the 2N+4 read and N+5 written streams (whole step on the same buffers, workgroups of four wavefronts tile by tile -> of
// one, with the scale paths that came with them: 11.7 M parameters, 4 workers 264 -> 215 us; 124 M, 8 workers 4.12 ->
// 3.84 ms; 1.3 G, 4 workers 22.7 -> 21.3 ms).
//
// Workgroups go to the eight XCDs in turn.  item_of gives the workgroups of one XCD runs of consecutive items, so
// that the pieces of a line of packed codes, which neighbouring items write, meet in one L2.
struct Items {
    uint32_t count;             // tiles * cut.parts
    Cut      cut;
    uint32_t run_shift;         // log2 of the items in a row that go to one XCD
};

constexpr uint32_t item_of(const Items& I, uint32_t block)
{
    const uint32_t xcd = block & 7u, k = block >> 3;
    const uint32_t mask = (1u << I.run_shift) - 1u;
    return (((k & ~mask) << 3) | (xcd << I.run_shift)) + (k & mask);
}

// Runs are 256 items (of whole tiles: 256 KiB of every stream in the main pass and the server, 512 KiB in the worker
// quantizer) where that leaves each XCD eight or more of them, shorter on short vectors.  Runs of 16 / 64 / 256 items, ms per
// step on the same buffers (medians of 9 turns within 1 %): 124 M parameters, 8 workers 4.00 / 3.88 / 3.83, 3 workers off
// the grid 2.30 / 2.22 / 2.24; 1.3 G, 4 workers 22.3 / 21.6 / 21.9; 2^28, 16 workers 14.2 / 14.3 / 15.3 where its buffers
// lay in that run, and 14.3 with 256 where they lay in another.
constexpr Items wave_items(const ListShape& s, int turn)
{
    Items I{};
    I.cut = cut_tiles(s, turn, ((int64_t)1 << 26) - 4096, 1);
    I.count = (uint32_t)s.num_tiles * I.cut.parts;
    while (I.run_shift < 8 && (I.count >> I.run_shift) >= 128) ++I.run_shift;
    return I;
}

// workgroups of the launch: whole rounds of a run per XCD, of which the last may hold more than `count`
constexpr uint32_t wave_blocks(const Items& I)
{
    const uint32_t round = 8u << I.run_shift;
    return (I.count + round - 1) / round * round;
}

// Tiles of the scale pass, a workgroup each, on the XCD whose wavefronts quantize them (the worker quantizer's and the main
// pass's runs are the same elements where they are short enough to matter): what the pass leaves in an L2 is then found
// there.  us, tiles round the XCDs in turn / this way: one worker's call, 128 tiles 8.5 / 7.3, 512 12.4 / 10.5, 1024
// 20.1 / 15.2, 2048 33.5 / 32.2; step of 4 workers, 256 tiles 26.3 / 22.7, 512 47.7 / 45.0, 1024 85.5 / 84.0, 2048 158 / 157.
constexpr Items scan_items(const ListShape& s)
{
    const Items q = wave_items(s, 512);
    Items I{};
    I.cut = Cut{1, kTileElems};
    I.count = (uint32_t)s.num_tiles;
    while ((q.cut.parts << (I.run_shift + 1)) <= (1u << q.run_shift)) ++I.run_shift;
    return I;
}

// one dimension of a launch holds fewer than 2^32 work-items
constexpr bool scan_fits(const Items& I) { return (uint64_t)wave_blocks(I) * 256 < ((uint64_t)1 << 32); }

// ---- layers of one tile, done from the gradient to the codes by one workgroup each (k_layers) -----------------------
// Sizes of its workgroups: one wavefront for up to 256 elements, four for up to 1024 and for up to a tile.
constexpr int kShortSizes = 3;
constexpr int short_size(int len) { return len <= 256 ? 0 : len <= 1024 ? 1 : 2; }

struct ShortLayers {
    int32_t num[kShortSizes];   // layers of each size
    int32_t as[kShortSizes];    // [k]: the size whose workgroups do the layers of size k

    constexpr bool any() const { return num[0] + num[1] + num[2] > 0; }
    constexpr int size_of(int len) const { return as[short_size(len)]; }
};

// Which of a list's layers of one tile are done that way: all or none.  The general path reads g and e twice and launches
// its passes mostly for workgroups of a few hundred elements; a workgroup that does its layer alone is a chain of one load,
// one maximum and one store per worker, and beside longer layers a launch more.  us per step, general path / this way.
// Only layers of one tile: 20000 of 1000 elements, 4 workers 430 / 298; 100000 of 100 716 / 217; 64 of 100 14.4 / 12.2, one
// worker's call 7.1 / 4.4; 256 of 4096 26.1 / 27.4, 400 of 4096 42.4 / 34.2; variant W, 8 workers, 64 of 100 23.3 / 24.2, 16
// workers 34 / 43 and with 256 of them 40 / 42.  Beside longer ones: one of 20 M and 300 of 1000, 4 workers 387 / 397, and
// 20000 of 1000 1055 / 691; 500 times 10000 and 100 112 / 119, 3000 times 654 / 639 (one worker 307 / 309).
// Sizes with fewer layers than there are CUs go along with the next one, which saves a launch.
constexpr ShortLayers short_layers_apart(const ShortLayers& have, int64_t num_tiles, int num_workers)
{
    ShortLayers s = have;
    for (int k = 0; k < kShortSizes; ++k) s.as[k] = k;
    const int64_t n = (int64_t)have.num[0] + have.num[1] + have.num[2];
    const bool alone = n == num_tiles;
    const bool apart = alone ? n >= 320 || (have.num[2] == 0 && num_workers <= 8) : n >= 2048;
    if (!apart || n > kMaxTiles - 4096) return ShortLayers{};       // a launch in whole rounds (wave_blocks) must fit
    for (int k = 0; k + 1 < kShortSizes; ++k) {
        int next = k + 1;
        while (next < kShortSizes && s.num[next] == 0) ++next;
        if (s.num[k] == 0 || s.num[k] >= 256 || next == kShortSizes) continue;
        s.num[next] += s.num[k];
        s.num[k] = 0;
        for (int j = 0; j <= k; ++j) if (s.as[j] == k) s.as[j] = next;
    }
    return s;
}

// Their workgroups, in runs of up to 32 per XCD: long enough for the scales of neighbours to meet in a line of one L2, and no
// longer, since every layer of a run is as many bytes of every stream that the XCDs drift apart by.  us per step, runs of 1 /
// 8 / 32 / 256: 20000 layers of 1000 elements, 4 workers 300 / 288 / 290 / 303, one worker 164 / 158 / 158 / 166; 100000 of
// 100, one worker 139 / 127 / 127 / 126.
constexpr Items layer_items(int32_t num)
{
    Items I{};
    I.cut = Cut{1, kTileElems};
    I.count = (uint32_t)num;
    while (I.run_shift < 5 && (I.count >> I.run_shift) >= 128) ++I.run_shift;
    return I;
}

// Whether the server takes the section of longer layers and each size of short ones in launches of their own: where one
// launch would be cut into longer pieces because short tiles among whole ones leave most of them empty.  us, one launch /
// by section: one layer of 20 M and 20000 of 1000, 4 workers 230 / 165, one worker 215 / 168; 3000 times 4096 and eight of
// 64, 4 workers 82 / 71; 400 times 9000 and twenty of 64 37.4 / 26.7; 500 times 4096 and sixteen of 64 31.8 / 19.3.
constexpr bool server_by_section(const ListShape& all, bool split)
{
    return split && cut_tiles(all, 256, ((int64_t)1 << 26) - 4096, 1).part_len > 256;
}

// ---- which data a first pass leaves in the cache, and which vectors are large --------------------------------------------
// Whether the scale pass over n elements of num workers leaves g and e in the cache for the quantizing pass.  A hit
// costs the memory nothing, a line kept in vain pushes out another's.  us per step, non-temporal / ordinary loads:
// 4 workers of 2 M (2^20) elements 48.9 / 47.4, 8 M 165.3 / 158.3, 16 M 317.6 / 304.4, 24 M 470.5 / 457.4, 32 M 618 / 611;
// 8 workers of 12 M 407 / 401; the handle-free call on 24 M 83.4 / 82.4.  One worker's separate call has little else
// to push out, and gains less: four calls of 8 M in a row 188.4 / 185.5, one of 16 M 159.8 / 159.3, of 24 M 232.0 /
// 233.2, of 40 M 375.6 / 379.7; four of 119 M 2299 / 2342.
constexpr bool keep_scanned(int64_t n, int num)
{
    const int64_t bytes = 8 * n * num;
    return bytes <= (num > 1 ? (int64_t)768 << 20 : (int64_t)192 << 20);
}

// Whether the first pass of variant W leaves the parked p of num workers in the cache for the pass that quantizes it.
// us per step, non-temporal / ordinary stores: 4 workers of 4 M (2^20) elements 125.7 / 123.4, 16 M 480 / 458, 24 M
// 709 / 685, 30 M 874 / 866, 48 M 1374 / 1407; one worker of 64 M 601 / 577.
constexpr bool keep_parked(int64_t n, int num) { return 4 * n * num <= (int64_t)512 << 20; }

// Whether the whole step runs as one launch per worker and one for the server instead of as one main pass.  The main pass
// writes no code word that it has to read again, but it has 2N + 4 read and N + 5 written streams open at once; three or four
// at a time lie in fewer DRAM pages, and the memory gives 6.3 to 6.6 TB/s for 5.2 to 6.3 wherever the buffers lie.  Where the
// scale pass (variant W: the moments) leaves its data in the cache the streams cost less and the launches more.  us per
// step, main pass / by worker: one worker of 24 M (2^20) elements 241 / 241, 64 M 656 / 641; 4 of 16 M 323 / 338, 24 M 497 / 498,
// 32 M 673 / 638, 96 M 2035 / 1901; 8 of 12 M 436 / 444, 16 M 581 / 547, 96 M 3566 / 3238; 16 of 4 M 255 / 301, 8 M 550 / 543,
// 96 M 6798 / 6002; variant W, 4 of 24 M 726 / 723, 64 M 1964 / 1929, 8 of 12 M 705 / 708, 96 M 5769 / 5588.
// Near the lines it took longer in some forms, which begin later.  us per step, main pass / by worker, nearest rounding: 12 workers of
// 8 M 409 / 425, 12 M 594 / 604; 16 of 6 M 390 / 410, 8 M 523 / 518, 12 M 734 / 736, 16 M 999 / 963.  Variant W: 5 workers of 85 M
// 2781 / 2841, 200 M 6593 / 6691; 8 of 18 M 978 / 992, 37 M 1994 / 1997, 50 M 2650 / 2639; 16 of 28 M 2790 / 2877, 50 M 5379 / 5300; with
// stochastic rounding 1 of 129 M 1184 / 1232, 4 of 56 M 1595 / 1640, 8 of 16 M 925 / 959, 16 of 14 M 1535 / 1616.
// Layers off the 16-byte grid, where the main pass depends more on where the buffers lie; the least and the largest ratio main pass / by
// worker of two to three allocations each, one layer and GPT lists: one worker of 34 M 0.96 0.98, 100 M 0.98 1.00, 185 M 1.00 1.00, 500 M
// 1.01 1.02; 2 of 50 M 1.02 1.03, 72 M 1.03 1.06, 276 M 1.05 1.07; 3 of 34 M 0.95 1.01, 67 M 1.04 1.07, 257 M 1.06 1.08; 4 of 34 M 0.93
// 0.97, 50 M 1.02 1.04, 120 M 1.02 1.04, 351 M 1.05 1.08; 5 of 30 M 0.94 0.97, 50 M 0.99 1.02, 276 M 1.02 1.02; 8 of 21 M 0.91 0.91, 40 M
// 0.97 1.03, 120 M 1.04 1.07; 16 of 30 M 0.94 1.03, 80 M 0.99 1.05, 120 M 0.96 0.98, 130 M 0.96 0.96.  Variant W: one of 130 M 1.02
// 1.03, 1 G 1.03 1.04; 2 of 65 M 1.01 1.01, 600 M 1.01 1.01; 3 of 45 M 0.98 0.98, 120 M 0.97 1.02; 4 of 33 M 0.99 1.03, 330 M 1.05 1.05,
// 351 M 0.97 0.98; 5 of 82 M 0.97 1.03, 200 M 0.98 0.99; 8 of 51 M 0.99 0.99, 170 M 0.97 0.97.
constexpr bool worth_by_worker(int64_t n, int64_t off_grid, int num, bool variant_w, bool stochastic)
{
    const int64_t work = n * num, M = 1 << 20;
    const bool off = 2 * off_grid > n;
    if (variant_w) return !stochastic && !keep_parked(n, num) && (off ? num <= 2 : num <= 4 || (num >= 8 && n >= 50 * M));
    if (keep_scanned(n, num)) return false;
    if (off) return num == 1 ? n >= 128 * M : num == 2 || (num <= 8 && work >= (64 + 32 * num) * M);
    return num <= 8 || n >= 14 * M;
}

// ---- layers that the chip's registers hold (k_parked) -----------------------------------------------------------------
// Unit u of a layer's n is its chunks u, u + n, ..., kParkedChunks at most, so that the workgroups of a layer walk it side
// by side.  A workgroup holds two units or, where a list has layers that need it, three.
constexpr int kParkedThreads = 512;
constexpr int kParkedChunk = kParkedThreads * 4, kParkedChunks = 8;

constexpr int parked_units(int64_t len)
{
    const int64_t chunks = (len + kParkedChunk - 1) / kParkedChunk;
    return (int)((chunks + kParkedChunks - 1) / kParkedChunks);
}

// Layers of up to kParkedLongestOfThree: 1088 units, 17.8 M elements.  The 512 workgroups of a launch (kParkedGroups, two per CU) hold two or
// three units each, of which one is being replaced, and a layer of nearly as many units as they hold beside it leaves none for its
// neighbours.  The third unit costs loads in flight and a turn more that only loads, so it is there only for lists with a layer of
// more than kParkedLongest elements (256 units).  The line is one for all calls and lies where the step whose scale pass is the filtered
// one stops gaining; a call with the full pass would gain up to 10 % beyond it.  One worker's call of 85 M elements, us, two passes / two units / three: layers of 36 units 260 / 202 /
// 206, 144 260 / 194 / 202, 256 259 / 203, 300 259 / 209 / 202, 384 272 / 232 / 212, 512 257 / 262 / 209, 768 275 / 273 / 218, 1024 261 / 263 /
// 209, 1100 (90 M) 277 / - / 242, 1280 (105 M) 323 / - / 291; step of 4 workers whose scale pass is the filtered one, 768 (88 M) 1348 / - /
// 1257, 1024 (117 M) 1790 / - / 1650, 1100 (90 M) 1388 / - / 1383, 1280 (105 M) 1599 / - / 1623.
constexpr int kParkedGroups = 512;
// Polls for a scale, of about 0.7 us each, before a workgroup puts its unit aside: where the layer's units are all held, and
// between two looks whether they are.
constexpr int kParkedPolls = 250, kPollsUnheld = 8;
// Every wait ends, also where two calls for one worker overlap, which the boundary forbids, and their counts are wrong: this
// many polls (about a second) at most, and for a scale that has to come a NaN in its place then.
constexpr int kLastPolls = 1 << 20;
constexpr int64_t kParkedLongest = (int64_t)256 * kParkedChunk * kParkedChunks;
constexpr int64_t kParkedLongestOfThree = (int64_t)1088 * kParkedChunk * kParkedChunks;

// Whether a step of num workers, or one worker's separate call (`call`), does the layers of up to kParkedLongestOfThree elements this way:
// `elems` in `units`, of the `all` elements whose scales have a pass of their own.  The launch starts by loading only and ends by
// storing only, which costs it about 30 us with two units (layers of 144 units, 85 M elements in 193 us, 340 M in 682), 34 with three
// (1024 units, 84 M in 209, 336 M in 735).  The figures from here to "a third unit" are of turns with guarded stores, 5 % slower at 85 M.
// us, without / with, layers of 2^18 to 2^21 elements: step of one worker of 4 M (2^20) 37.0 / 47.0, 8 M 83.1 / 79.2, 16 M 156 / 147, 64 M 559 / 517; 4 workers of 4 M 80.8 /
// 82.6, 8 M 155 / 141, 32 M 599 / 482; 8 of 2 M 71.0 / 71.9, 4 M 137 / 121, 32 M 1020 / 755.  A unit costs about the same however few
// elements it has: 4000 layers of 5000, one worker's call 69.4 / 78.8, step of 4 workers 404 / 395; 500 of 10000 and 100, 4 workers
// 107 / 123, 3000 times 609 / 513; 1000 of 20000 375 / 338.  Beside a long layer the step goes worker by worker for its sake: one of
// 20 M and 300 of 1000, 4 workers 371 / 412; 1.3 G with 0.1 G of them 20.96 / 20.95 ms.  A list most of which is a longer layer: 5 M
// beside 12 M, 8 workers 558 / 568; 12 M beside 30 M, 4 workers 777 / 763.
// One worker's call has little to gain while its data is in the cache, and a last turn of few workgroups takes it as long as a full
// one: layers of 1 M, 8 M in all 29.8 / 30.7, 9 M 35.0 / 36.1 to 38.9, 12 M 43.6 / 45.5, 16 M 54.3 / 51.9, 24 M 79.9 / 73.1, 64 M 207 /
// 165; of 5 M, 10 M 37.7 / 40.5, 15 M 51.3 / 51.1, 20 M 67.5 / 71.5, 25 M 86 / 76.
// Stochastic rounding, whose random numbers keep the vector units busy: one worker's call of 16 M 58 / 65, 32 M 109 / 109, 50 M in
// layers of 5 M 165 / 166 and off the grid 191 / 196, 64 M 211 / 196; step of 2 workers of 24 M 286 / 293, 30 M 358 / 362, 4 of 8 M 159 /
// 162, off the grid 168 / 178, of 16 M 306 / 286 and 380 / 317.  Beside longer layers, 8 workers, 6 M beside 12 M 612 / 627, off the
// grid 684 / 737, 12 M beside 12 M 812 / 783 and 916 / 918, 4 workers 465 / 476 and 522 / 567.
// Layers that need a third unit, whose start takes longer (longest: elements of the longest): step of one worker, one layer of 8 M 82.0 /
// 83.8, two 160 / 150, one of 16 M 160 / 149; of 4, one of 8 M 158 / 151, 12 M 236 / 209, 16 M 308 / 268; stochastic, 5 of 8 M, its
// call 136 / 133, step of 4 workers 753 / 630, 3 of 16 M 899 / 798.  One worker's call, alone and then each of four at once on
// streams of their own, whose launches have few workgroups for many units: two layers of 8 M 57 / 59 and 55 / 69, one of 16 M 56 / 58 and
// 56 / 71; two of 12 M 82 / 76 and 82 / 88, two of 16 M 108 / 99 and 106 / 119, three 157 / 137 and 158 / 169, five 257 / 208 and 259 / 249.
constexpr bool worth_parking(int64_t elems, int64_t units, int64_t all, int num, bool stochastic, bool call = false,
                             int64_t longest = 0)
{
    const int64_t work = elems * num, M = 1 << 20, turns = (units + kParkedGroups - 1) / kParkedGroups;
    const bool filled = units * kParkedChunk * kParkedChunks <= 2 * elems;
    const bool full_turns = 16 * units >= 15 * turns * kParkedGroups;
    const int64_t least = stochastic && elems < all ? 96 : !filled ? 72 : stochastic ? (call || num == 2 ? 64 : 48)
                        : 2 * elems < all ? 48 : num > 1 ? 24 : !call ? (longest > kParkedLongest ? 12 : 8)
                        : full_turns && longest <= kParkedLongest ? 15 : 24;
    return work >= least * M && 4 * elems >= all;
}

// The same for variant W, a worker's separate call being a step of one.  It saves 8 of 36 bytes per element, so parking pays later.  us
// per step, two passes / parked.  Layers of 36 units: one worker of 16 M (2^20) elements 147 / 148, 24 M 213 / 219, 47 M 419 / 405, 94 M
// 853 / 812; 2 of 12 M 181 / 181; 4 of 8 M 223 / 225, 12 M 330 / 323, 24 M 654 / 602; 8 of 4 M 213 / 216, 8 M 421 / 399; 16 of 2 M 247 / 231;
// off the grid 4 of 12 M 373 / 360, 8 of 8 M 480 / 447; one worker's call of 24 M 148 / 156, 47 M 292 / 277.  Layers that need a third unit: 4
// workers, one of 8 M 228 / 235, 12 M 334 / 327, 16 M 428 / 432, two of 5 M 265 / 269, five 651 / 600, three of 8 M 668 / 625, of 16 M 1383 /
// 1205; 8, four of 16 M 3451 / 3000; 5 of 7.3 M 253 / 270.  Stochastic: 3 of 17 M 386 / 398, 4 of 12 M 341 / 342, 24 M 676 / 607.  Units mostly
// empty, 4000 layers of 5000 and 4 workers 629 / 660.  Beside a longer layer, 4 workers: 9 M beside 23 M 971 / 980, 20 M beside 31 M 1479 /
// 1449.
constexpr bool worth_parking_w(int64_t elems, int64_t units, int64_t all, int num, bool stochastic, int64_t longest)
{
    const int64_t work = elems * num, M = 1 << 20;
    const bool filled = units * kParkedChunk * kParkedChunks <= 2 * elems;
    const int64_t least = longest > kParkedLongest ? 80 : stochastic ? 72 : num >= 4 ? 40 : 48;
    return filled && work >= least * M && 3 * elems >= all;
}

// The meeting place of a layer's workgroups: a word that counts arrivals and departures, and copies of the published scale
// to poll, every one in a line of its own, for up to eight of them each in layers of up to 512 units and 17 in the longest: one
// wavefront writes all copies.  Words.
constexpr int kMeetingLine = 32;
constexpr uint32_t kArrivals = 0xffffu, kDeparture = 0x10000u;
// In front of a worker's meeting places: the counts of a launch, and the claims of the workgroups' first units.
constexpr int kClaims = kMeetingLine, kMeetingCounts = kClaims + kParkedGroups;
constexpr int meeting_copies(int units) { return units <= 8 ? 1 : units >= 512 ? 64 : (units + 7) / 8; }
constexpr int meeting_words(int units) { return units > 1 ? (1 + meeting_copies(units)) * kMeetingLine : 0; }

// ---- buffers in one block (qadam_arena_layout) -------------------------------------------------------------------------
enum class Buffer { x, m, v, werr, err, mw, vw, grad, codes, wcodes, scales };

// f(buffer, worker, group) in the order in which the layout deals them to its two groups: the read+write streams first, then the
// read-only gradients, then the small write-only ones.
template <typename F>
void deal_buffers(int workers, bool worker_moments, F&& f)
{
    int dealt = 0;
    auto deal = [&](Buffer b, int i) { f(b, i, dealt++ & 1); };
    for (Buffer b : {Buffer::x, Buffer::m, Buffer::v, Buffer::werr}) deal(b, 0);
    for (int i = 0; i < workers; ++i) deal(Buffer::err, i);
    if (worker_moments)
        for (int i = 0; i < workers; ++i) { deal(Buffer::mw, i); deal(Buffer::vw, i); }
    for (int i = 0; i < workers; ++i) deal(Buffer::grad, i);
    for (int i = 0; i < workers; ++i) deal(Buffer::codes, i);
    deal(Buffer::wcodes, 0);
    for (int i = 0; i < workers; ++i) deal(Buffer::scales, i);
}

// What a buffer of `elems` parameters takes in the block: buffers start on 2 MiB boundaries (the driver's large pages).
constexpr uint64_t kArenaAlign = 2u << 20;
constexpr uint64_t arena_round(uint64_t n) { return (n + kArenaAlign - 1) / kArenaAlign * kArenaAlign; }

// Bytes from the first group to the second where the buffers lie as the layout deals them, 0 where they do not.  bytes(b): of
// one buffer, rounded up; at(b, i): its address, 0: not in use.
template <typename Bytes, typename At>
int64_t groups_apart(int workers, bool worker_moments, Bytes&& bytes, At&& at)
{
    uint64_t begin[2] = {0, 0}, fill[2] = {0, 0};
    bool dealt = true;
    deal_buffers(workers, worker_moments, [&](Buffer b, int i, int group) {
        if (const uint64_t p = at(b, i)) {
            if (begin[group] == 0) begin[group] = p - fill[group];
            dealt = dealt && begin[group] == p - fill[group];
        }
        fill[group] += bytes(b);
    });
    return dealt && begin[0] != 0 && begin[1] > begin[0] ? (int64_t)(begin[1] - begin[0]) : 0;
}

// ---- flat launches (weight quantizer, decoder) -----------------------------------------------------------------------
// Workgroups of `per_block` consecutive elements each, in rows of 2^31 work-items.
struct FlatGrid {
    uint32_t x, y;
};

constexpr FlatGrid flat_blocks(int64_t n, int threads, int per_block)
{
    const int64_t row = ((int64_t)1 << 31) / threads, blocks = (n + per_block - 1) / per_block;
    return {(uint32_t)(blocks < row ? blocks : row), (uint32_t)((blocks + row - 1) / row)};
}

// ---- folding the maxima of the layers (k_reduce_scales, k_reduce_scales_list) ----------------------------------------
constexpr int kReduceThreads = 1024;
constexpr int kListLayers = kReduceThreads / 64;    // layers per workgroup of k_reduce_scales_list, one per wavefront
constexpr int kListMaxima = 64 * 8;                 // maxima one wavefront folds in one turn

// Whether k_reduce_scales_list folds the maxima of num workers.  Up to two fillings of the chip (1024 pairs of worker and
// layer) the workgroup per layer is level or faster, its long layers running beside each other: whole step of a GPT-2 small
// list, one worker (145 pairs), 1088 us / 1113 with the list form; 150 layers of 100 elements, 4 workers (600 pairs)
// 16.8 / 16.9.  Beyond that most of its 16 wavefronts have nothing to do: 300 layers of 100 elements, 4 workers 21.4 / 19.9;
// 2000 layers, 4 workers 53.8 / 39.6; 10000 layers, 16 workers 768 / 491; GPT-2 small, 8 workers (1160 pairs) 4104 / 4091;
// one layer of 40 M and 3000 of 100, 4 workers 801 / 786.  It also keeps the launch below 2^32 work-items where a
// workgroup per layer would not (2^22 layers).
constexpr bool reduce_by_list(int num_segments, int num) { return (int64_t)num_segments * num > 1024; }

constexpr unsigned reduce_blocks(int num_segments, int num)
{
    return reduce_by_list(num_segments, num) ? (unsigned)(((int64_t)num_segments + kListLayers - 1) / kListLayers)
                                             : (unsigned)num_segments;
}

// Whether the quantizing kernel folds the maxima itself: every wavefront those of its layer (`longest`: most maxima of one
// layer, `per_tile` to a tile) for each of its workers, one after the other, which saves the launch of k_reduce_scales.  A
// step this short is bound by what the host enqueues, and the launch is 2.7 us of it; on the GPU alone (a captured graph) the
// fold is level up to about four workers and the slower way beyond (sixteen of 16 tiles 24.1 / 29.2), so it goes as far as
// the host's time covers that.  us per step in a loop of calls, with the launch / folded, one layer.  One maximum per tile:
// one worker, 512 tiles 22.3 / 21.3; two, 256 20.1 / 17.4, 512 29.5 / 28.3; four, 128 22.6 / 20.1, 256 22.6 / 22.7; eight, 64
// 27.9 / 25.2, 128 27.7 / 25.1; sixteen, 64 37.8 / 35.1, 128 42.7 / 46.0.  Four maxima per tile (variant W): one worker, 256
// tiles 19.9 / 17.2, 512 25.4 / 26.8, 1024 46.5 / 52.7; two, 256 22.6 / 22.7, 512 40.6 / 44.4; four, 128 24.8 / 23.1, 256
// 36.7 / 38.6; eight, 64 32.7 / 30.2, 128 38.5 / 41.7; sixteen, 32 48.6 / 46.0, 64 49.6 / 51.1.  Lists: eight workers, 45
// tiles of 16 layers 27.9 / 25.1; variant W, 78 of 77 33.7 / 30.9.
// GPU time of one worker's call, one layer: 512 tiles 14.4 / 14.3, 1024 20.8 / 24.9.  One worker, layers with a maximum or none
// for each lane: 1500 tiles in layers of 15, its call 24.6 / 23.9, its step 60.0 / 56.8; 1488 in layers of 62, 24.6 / 23.5
// and 62.3 / 59.0; 4000 in layers of 25, call 53.2 / 57.5.
constexpr bool fold_in_quantizer(int num_tiles, int64_t num_elems, int longest, int num_workers, int per_tile)
{
    if (num_workers == 1 && longest <= 64) return num_tiles <= 2048;
    return (num_tiles <= 128 || (int64_t)num_tiles * num_workers <= 1024) && longest <= (per_tile == 1 ? 768 : 1024)
        && num_elems * num_workers <= (int64_t)1 << (per_tile == 1 ? 22 : 21);
}

}  // namespace qadam
