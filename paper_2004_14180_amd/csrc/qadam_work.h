// How the kernels' work is divided over their launches: arithmetic that the host and the kernels share.  Plain C++, so
// that it can be checked on the CPU at sizes no test allocates.
#pragma once

#include <stdint.h>

namespace qadam {

constexpr int64_t kMaxTiles = (int64_t)1 << 24;     // a handle has fewer: one 256-thread workgroup per tile must fit a launch

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
