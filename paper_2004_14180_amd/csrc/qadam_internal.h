// Shared declarations between the host-side C boundary (qadam_api.cpp) and the gfx950 kernels
// (qadam_kernels.hip).  Not part of the public interface.
#pragma once

#include <hip/hip_runtime_api.h>
#include <stdint.h>

#include "../../include/qadam.h"
#include "qadam_work.h"

namespace qadam {

// One unit of work of every kernel: a run of at most `tile_elems` consecutive elements that lies
// inside one layer segment.  Tiles start at a multiple of the tile size from the segment start, so
// the first element of a tile is the first element of a 32-element code group.
struct Tile {
    int64_t start;      // global flat index of the first element
    int64_t code_word;  // index of the tile's first uint32 in a worker's packed code buffer
    int32_t len;        // elements in the tile (1 .. tile_elems)
    int32_t seg;        // layer segment the tile belongs to
    int32_t flags;      // bit 0: start is not a multiple of 4 (no 128-bit accesses);
                        // bit 1: sampled tile of the filtered scale pass;
                        // bits 8..9: zero words to append after the tile's codes (segment padding)
    int32_t reserved;
};
static_assert(sizeof(Tile) == 32, "tile records are read as two 128-bit scalar loads");

constexpr int kTileUnaligned = 1;
constexpr int kTileSampled = 2;
constexpr int kSampleStride = 64;   // every 64th tile of a layer (from its first) is a sampled tile
constexpr int kBlockThreads = 256;

// Scalars of one launch, identical for every kernel.
struct StepScalars {
    int32_t  num_workers;
    int32_t  k_g, mu_bits, code_bits;   // Q_g: levels, bits of the level index, bits per code
    int32_t  k_x, wcode_bytes;          // Q_x
    int32_t  rounding, weight_ef, adam_flavor;
    uint32_t key0, key1;                // Philox key (seed)
    uint32_t step;                      // low 32 bits of t
    float    lr, beta1, beta2, eps;
    float    omb1, omb2;                // 1-beta, 1-theta_t (fp32 subtraction done on the host)
    float    lr1, sbc2;                 // flavour 1: lr / (1-beta^t), sqrt(1-theta^t)
    float    n_workers_f;               // (float)N
    float    inv_n;                     // 1/N, used when N is a power of two (then exact)
    int32_t  n_is_pow2;
};

// Pointer tables travel as kernel arguments.
struct WorkerPtrs {
    const float* grad[QADAM_MAX_WORKERS];
    float*       err[QADAM_MAX_WORKERS];
    uint32_t*    codes[QADAM_MAX_WORKERS];
    float*       scales[QADAM_MAX_WORKERS];
    float*       mw[QADAM_MAX_WORKERS];     // variant W only
    float*       vw[QADAM_MAX_WORKERS];
};

struct ServerPtrs {
    float* x;
    float* m;
    float* v;
    float* werr;        // may be null when weight_ef == 0
    void*  wcodes;
};

// Those of a handle's layers whose scales come from a pass of their own: all, or all but short_layers.  Tiles are counted
// within the section.
struct Section {
    const Tile* tiles;      // device
    const int32_t* seg_tile_begin;  // device, [num_segments + 1]: first tile of every layer
    const int32_t* layers;  // device: the layers, empty ones included; null: all
    int32_t     num_layers;
    int64_t     num_elems;
    ListShape   shape;
};

// A layer of k_parked, and a workgroup of it.
struct ParkedLayer {
    Tile    t;              // the whole layer
    int32_t num_units, first_unit;
    int32_t meeting, copies;    // first word of its meeting place, polled copies of the scale
};

struct ParkedUnit {
    int32_t layer, unit;
};

struct Parked {
    const ParkedUnit*  units;   // device
    const ParkedLayer* layers;  // device
    uint32_t* meeting;      // device, [num_workers][meeting_words], zero between launches but for the launches counted
    uint32_t* aside;        // device, [num_workers][num_units]
    int32_t   num_units, meeting_words;
    int64_t   num_elems, longest;   // elements of all of them, of the longest
    int32_t   polls;        // for a scale before a workgroup puts its unit aside
};

struct Launch {
    const Tile* tiles;      // device
    float*      inv_scales; // device, [num_workers][num_segments]: 1/s where the fast quotient is safe, else 0
    uint32_t*   tile_max;   // device, [num_workers][scaled tiles * moment_parts]: max |p| per tile (variant W: per piece of
                            // a tile) as a bit pattern; a worker's row begins at the same place in every call
    const int32_t* seg_tile_begin;  // device, [num_segments + 1]: first tile of every segment
    int32_t     num_tiles;
    ListShape   shape;
    Section     scaled;
    int64_t     off_grid_elems; // of `scaled`: of layers that start off the 16-byte grid
    int32_t     max_row;    // maxima from one worker's row to the next's, the same in every call and pass: calls for
                            // different workers may run on different streams
    Parked      parked;     // layers of `scaled` that k_parked can do; num_units == 0: none
    Section     rest;       // `scaled` without them
    const int32_t* rest_sample_tiles;
    int32_t     num_rest_sample_tiles;
    bool        parked_done;    // `scaled` is `rest`, k_parked does the others
    const Tile* served_tiles;   // the tiles of both
    ListShape   served;
    int32_t     longest_layer;  // tiles of the longest layer
    const Tile* short_layers;   // device: the layers that k_layers does, one tile each, by size; null: none
    ShortLayers apart;          // how many of each size
    const ListShape* short_shape;   // host, [kShortSizes]: their tiles
    int32_t     num_segments;
    int64_t     num_params;
    int64_t     code_words;     // of one worker
    double*     tile_sum;   // device, [num_tiles]: per-tile partial sums of the norm diagnostic
    float*      err_bound;  // device, [num_workers][num_segments]: bound on |e| left by the last step
    uint32_t*   thr;        // device, [num_workers][num_segments]: thresholds of the filtered scale pass
    const int32_t* sample_tiles;    // device: indices of the sampled tiles
    int32_t     num_sample_tiles;
    bool        empty_layers;   // some layer has no element: its scale (0) has no quantizing workgroup to write it
    uint32_t*   status;     // device status word
    hipStream_t stream;
};

// maxima per tile that the first pass of variant W leaves
inline int moment_parts(const Launch& L) { return (int)moment_cut(L.scaled.shape).parts; }

// maxima of one worker that a first pass over what k_parked leaves may write, in front of those of the units
inline int rest_maxima(const Section& rest) { return rest.shape.num_tiles * (int)moment_cut(rest.shape).parts; }

// the launch of what k_parked leaves
inline Launch without_parked(const Launch& L)
{
    Launch R = L;
    R.scaled = L.rest;
    R.sample_tiles = L.rest_sample_tiles; R.num_sample_tiles = L.num_rest_sample_tiles;
    R.parked_done = true;
    return R;
}

// Launchers (defined in qadam_kernels.hip).  `first_worker`/`num` select the workers a launch covers.
// scales in two stages without atomics: per-tile maxima, then one workgroup per (worker, layer)
// (of long lists: per 16 layers) reduces its tiles and also writes the reciprocal used by the fast quotient
hipError_t launch_amax(const Launch& L, const StepScalars& S, const WorkerPtrs& W, int first_worker, int num);
hipError_t launch_reduce_scales(const Launch& L, const StepScalars& S, const WorkerPtrs& W, int first_worker, int num,
                                int max_per_tile = 1);
hipError_t launch_amax_filtered(const Launch& L, const StepScalars& S, const WorkerPtrs& W, int first_worker, int num);
hipError_t launch_check_error_bounds(const Launch& L, const WorkerPtrs& W, int first_worker, int num);
bool use_parked(const Launch& L, const StepScalars& S, const WorkerPtrs& W, int first_worker, int num, bool call, bool variant_w);
hipError_t launch_parked(const Launch& L, const StepScalars& S, const WorkerPtrs& W, int first_worker, int num, bool variant_w);
hipError_t launch_worker_quantize(const Launch& L, const StepScalars& S, const WorkerPtrs& W, int worker);
// the short layers of the list, from the gradient (variant_w: through the local moments) to the codes, for one worker; or
// the whole step of all workers
hipError_t launch_short_layers(const Launch& L, const StepScalars& S, const WorkerPtrs& W, int worker, bool variant_w);
hipError_t launch_short_layers(const Launch& L, const StepScalars& S, const WorkerPtrs& W, const ServerPtrs& sp, bool variant_w);
hipError_t launch_server_step(const Launch& L, const StepScalars& S, const WorkerPtrs& W, const ServerPtrs& sp);
hipError_t launch_weight_quantize(const Launch& L, const StepScalars& S, const float* x, float* werr, void* wcodes);
hipError_t launch_weight_dequantize(const Launch& L, const StepScalars& S, const void* wcodes, void* xhat, bool half);
// whether the two below are one launch per worker and one for the server, which reads the codes
bool step_by_worker(const Launch& L, const StepScalars& S, const WorkerPtrs& W, const ServerPtrs& sp, bool variant_w);
hipError_t launch_fused(const Launch& L, const StepScalars& S, const WorkerPtrs& W, const ServerPtrs& sp);
// Q_g = identity: the messages are fp32 values (variant S: the gradients; variant W: the parked
// update + error, whose buffers are then cleared)
hipError_t launch_plain_messages(const Launch& L, const StepScalars& S, const WorkerPtrs& W, const ServerPtrs& sp,
                                 bool variant_w);
hipError_t launch_layer_sumsq(const Launch& L, const float* a, const float* b, double* out);
// variant W
hipError_t launch_worker_moments_w(const Launch& L, const StepScalars& S, const WorkerPtrs& W, int first_worker, int num);
hipError_t launch_fused_w(const Launch& L, const StepScalars& S, const WorkerPtrs& W, const ServerPtrs& sp);
hipError_t launch_server_apply_w(const Launch& L, const StepScalars& S, const WorkerPtrs& W, float* x);


// Handle-free quantization of one segment (qadam_quantize_segment_noalloc): the per-tile maxima, the
// reciprocal scale and a status word live in a static device array, so nothing is allocated.
// noalloc_prepare looks up that array's address on the current device (once per device).
constexpr int64_t kNoallocMaxElems = QADAM_NOALLOC_MAX_ELEMS;
hipError_t noalloc_prepare();
hipError_t noalloc_quantize_segment(const StepScalars& S, int64_t n, const float* grad, float* err, uint32_t* codes,
                                    float* scale_out, hipStream_t stream);

}  // namespace qadam
