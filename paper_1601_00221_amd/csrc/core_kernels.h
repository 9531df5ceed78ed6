// Launch interface of the core-based evaluation kernel.
#pragma once

#include <hip/hip_runtime_api.h>
#include <stdint.h>

#include "../../include/gp.h"
#include "gp_internal.h"
#ifdef __HIPCC__
#include <hip/hip_runtime.h>
#endif

namespace gpx {

// Exit operation that ends a program.  Its record's payload holds, in the low
// 24 bits, the number of records of the program that follows (0: none), and
// its constant the program's row.
enum : uint32_t { CORE_OP_LOAD = 14, CORE_OP_END = 15 };   // LOAD: a feature of the tile to stack level 0

enum : int32_t { CORE_TO_ROW = 5 };     // "fitness kind" of the programs that compute a block's rows

struct DatasetDesc {
    const float* X;
    const float* y;
    int64_t N;
};

struct JobDesc {
    int32_t ds;                 // dataset index
    int32_t kind;
    int32_t n_load;             // features the job's programs read
    int32_t pad;
    uint64_t part_base;         // the job's partial sums start here (see ReduceArgs)
};

struct UnitDesc {
    uint32_t job;
    uint32_t tile;
    uint32_t c0, c1;            // core records of its programs, one after another
};

// Partial sums are program-major: block b of program p (its row in the
// job) is partials[part_base + p * blocks + b], so one wave's blocks of one
// program are adjacent.
struct ReduceArgs {
    const double* partials;
    uint64_t part_base;
    int64_t n_prog;
    int64_t N;
    void* out;
    int32_t blocks;             // ceil(N / 256)
    int32_t kind;
};

struct CoreArgs {
    const uint32_t* code;       // core instructions, 16 bytes each
    // table of units (batched launches); null: implicit units over one dataset
    const UnitDesc* units;
    const JobDesc* jobs;
    const DatasetDesc* datasets;
    uint32_t* counter;          // next unit, persistent form
    // implicit units: block unit b = (the W groups from W (b div chunks) on, chunk b mod
    // chunks); a chunk is tiles_per_wave consecutive tiles
    const uint32_t* group_off;  // group g holds the core records group_off[g] .. group_off[g + 1)
    const float* X;
    const float* y;
    int64_t N;
    int32_t n_load;
    int32_t kind;
    int32_t tiles;
    int32_t n_units;            // table units, or implicit block units
    int32_t persistent;
    int32_t tiles_per_wave;
    int32_t chunks;
    int32_t prefetch;           // 64-byte lines of the next program's code loaded into the scalar cache at a
                                // time (1-14), or 0: none
    int32_t n_groups;           // program groups (implicit units)
    int32_t n_rows;             // rows (sin, cos, exp or log of a feature) each block computes for its tile into LDS,
                                // by the programs row_off[w] .. row_off[w + 1] of its wave w; 0: none
    const uint32_t* row_off;
    int32_t direct;             // implicit units, at most as many tiles as a block has waves: a block of that many
                                // waves runs one group on every tile and writes its programs' fitness to `out` itself
                                // (no reduction launch); 0: not so.
    const uint32_t* group_prog; // group g holds the programs order[group_prog[g] .. group_prog[g + 1])
    const uint32_t* order;
    void* out;
    int32_t same_group;         // implicit units: the waves of a block run one group on as many chunks
    int64_t n_bits;             // Boolean kernels: cases (bits) in the N words of each row
    uint32_t probe;             // nonzero: write the handler table address and return
    double* partials;
    float* cases_out;
    uint64_t* probe_out;
};

// Program p's fitness from the sum of its partials.
#ifdef __HIPCC__
__device__ __forceinline__ void finish_sum(int32_t kind, int64_t N, void* out, int64_t p, double s) {
    if (kind == GP_FIT_HITS || kind == GP_FIT_CLASS_ERR) ((int32_t*)out)[p] = (int32_t)s;
    else if (kind == GP_FIT_MSE) ((float*)out)[p] = (float)(s / (double)N);
    else ((float*)out)[p] = (float)s;
}
#endif

hipError_t core_launch(int variant, const CoreArgs& a, uint32_t blocks, hipStream_t s);
int core_blocks_per_cu(int variant);
hipError_t core_zero_counter(uint32_t* counter, hipStream_t s);
hipError_t core_reduce_jobs(const ReduceArgs* jobs_dev, int32_t n_jobs, int64_t max_prog, hipStream_t s);
hipError_t core_reduce_one(const ReduceArgs& r, hipStream_t s);

}  // namespace gpx
