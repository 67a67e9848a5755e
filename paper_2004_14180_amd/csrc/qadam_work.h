// How the kernels' work is divided over their launches: arithmetic that the host and the kernels share.  Plain C++, so
// that it can be checked on the CPU at sizes no test allocates.
#pragma once

#include <stdint.h>

namespace qadam {

constexpr int64_t kMaxTiles = (int64_t)1 << 24;     // a handle has fewer: one 256-thread workgroup per tile must fit a launch
constexpr int kTileElems = 4096;                     // elements per tile (16 per lane of a 256-thread workgroup)

// ---- work items of the kernels whose workgroups are single wavefronts ------------------------------------------------
// (the main pass, the worker quantizer, the server): a tile is cut into `parts` pieces of `part_len` elements and each is
// one workgroup.  Wavefronts that share a workgroup start together and then load and store in step, and the next four
// start when the last of them has ended; on their own they drift apart, so reads and writes mix, and the workgroups in
// flight cover a narrower stretch of each of the 2N+4 read and N+5 written streams (main pass with four wavefronts per
// workgroup -> one: 11.7 M parameters, 4 workers 204 -> 172 us; 124 M, 8 workers 3.29 -> 3.04 ms; 1.3 G, 4 workers
// 19.5 -> 18.4 ms).
//
// Workgroups go to the eight XCDs in turn.  item_of gives the workgroups of one XCD runs of consecutive items, so
// that the pieces of a line of packed codes, which neighbouring items write, meet in one L2.
struct Items {
    uint32_t count;             // tiles * parts
    uint32_t parts;             // pieces per tile
    int32_t  part_len;          // elements per piece; parts * part_len covers a tile
    uint32_t run_shift;         // log2 of the items in a row that go to one XCD
};

constexpr uint32_t item_of(const Items& I, uint32_t block)
{
    const uint32_t xcd = block & 7u, k = block >> 3;
    const uint32_t mask = (1u << I.run_shift) - 1u;
    return (((k & ~mask) << 3) | (xcd << I.run_shift)) + (k & mask);
}

// Pieces of `part_len` elements, longer where the launch would reach 2^32 work-items.  Runs are 256 items (256 KiB of
// every stream) where that leaves each XCD eight or more of them (1.3 G parameters, 4 workers: 18.97 ms with runs
// of 16, 18.41 with 64, 18.8 with 256; 124 M, 3 workers: 1.765 / 1.728 / 1.702 ms), shorter on short vectors.
constexpr Items wave_items(int num_tiles, int part_len)
{
    Items I{};
    I.parts = (uint32_t)(kTileElems / part_len);
    while ((int64_t)num_tiles * I.parts > ((int64_t)1 << 26) - 4096) I.parts /= 2;
    I.part_len = kTileElems / (int)I.parts;
    I.count = (uint32_t)num_tiles * I.parts;
    while (I.run_shift < 8 && (I.count >> I.run_shift) >= 128) ++I.run_shift;
    return I;
}

// workgroups of the launch: whole rounds of a run per XCD, of which the last may hold more than `count`
constexpr uint32_t wave_blocks(const Items& I)
{
    const uint32_t round = 8u << I.run_shift;
    return (I.count + round - 1) / round * round;
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

}  // namespace qadam
