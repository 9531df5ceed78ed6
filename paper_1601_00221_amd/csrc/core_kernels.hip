// Fitness reductions and the launchers of the evaluation kernel.  The
// kernel itself (core_body.h) is compiled once per variant, each in its own
// translation unit generated by gen_core.py (core_v_<variant>.hip).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/gp.h"
#include "core_kernels.h"

namespace gpx {
#include "core_dispatch.inc"

__global__ void k_zero_u32(uint32_t* p) { *p = 0u; }

// Reduction over blocks: program p sums its partials partial[base + p * blocks
// + b], in the order b = 0 .. blocks - 1 where they are binary64 sums (the
// result does not depend on what else a launch holds); counts are whole
// numbers, exact in any order.
//
// Bound by latency, not by bytes: one thread a program walking its row alone
// waits for a 32-byte sector every few additions (160 us for 1000 programs x
// 391 blocks, 0.52 ms for 4096 x 4096).  So a block takes kProgs programs, all
// its threads load the next kChunk partials of each in contiguous pieces while
// one thread a program adds up the chunk before, which lies in LDS.  Counts
// need no order: a wave a program, lanes side by side.
constexpr int kProgs = 16, kChunk = 128, kPer = kProgs * kChunk / 256;

__device__ __forceinline__ void reduce_block(const ReduceArgs& r) {
    const int64_t p0 = (int64_t)blockIdx.x * kProgs;
    if (p0 >= r.n_prog) return;
    const double* part = r.partials + r.part_base;
    const int t = (int)threadIdx.x, B = r.blocks;
    // (short rows go the other way: four programs a wave, one after another, wait for memory four times)
    if ((r.kind == GP_FIT_HITS || r.kind == GP_FIT_CLASS_ERR) && B > 4 * kChunk) {
        for (int k = t >> 6; k < kProgs; k += 4) {
            const int64_t p = p0 + k;
            if (p >= r.n_prog) break;
            double s = 0.0;
            for (int b = t & 63; b < B; b += 64) s += part[p * B + b];
#pragma unroll
            for (int d = 32; d >= 1; d >>= 1) s += __shfl_xor(s, d, 64);
            if ((t & 63) == 0) finish_sum(r.kind, r.N, r.out, p, s);
        }
        return;
    }
    // thread t loads partials (t & 15) + 16 i of program t >> 4, i = 0 .. kPer - 1
    __shared__ double buf[2][kProgs][kChunk + 1];
    const int64_t mine = p0 + (t >> 4);
    const double* src = part + (mine < r.n_prog ? mine : r.n_prog - 1) * B;
    double v[kPer];
    auto load = [&](int b0) {
#pragma unroll
        for (int i = 0; i < kPer; i++) {
            const int b = b0 + (t & 15) + 16 * i;
            v[i] = b < B ? src[b] : 0.0;
        }
    };
    load(0);
    double s = 0.0;
    for (int b0 = 0, h = 0; b0 < B; b0 += kChunk, h ^= 1) {
#pragma unroll
        for (int i = 0; i < kPer; i++) buf[h][t >> 4][(t & 15) + 16 * i] = v[i];
        __syncthreads();
        if (b0 + kChunk < B) load(b0 + kChunk);
        // the other half is written only after the next barrier, which every thread reaches after its sum here
        if (t < kProgs) {
            const int n = B - b0 < kChunk ? B - b0 : kChunk;
            const double* x = buf[h][t];
            int k = 0;
            for (; k + 8 <= n; k += 8) {
                double y[8];
#pragma unroll
                for (int i = 0; i < 8; i++) y[i] = x[k + i];
#pragma unroll
                for (int i = 0; i < 8; i++) s += y[i];
            }
            for (; k < n; k++) s += x[k];
        }
    }
    if (t < kProgs && p0 + t < r.n_prog) finish_sum(r.kind, r.N, r.out, p0 + t, s);
}

// Program block blockIdx.x of job blockIdx.y
__global__ __launch_bounds__(256) void k_reduce_jobs(const ReduceArgs* jobs) {
    const ReduceArgs r = jobs[blockIdx.y];
    reduce_block(r);
}

__global__ __launch_bounds__(256) void k_reduce_one(ReduceArgs r) { reduce_block(r); }

// --------------------------------------------------------------------------
// Launchers
// --------------------------------------------------------------------------
hipError_t core_launch(int vi, const CoreArgs& a, uint32_t blocks, hipStream_t s) {
    if (vi < 0 || vi >= (int)(sizeof(kCoreLaunch) / sizeof(kCoreLaunch[0]))) return hipErrorInvalidValue;
    return kCoreLaunch[vi](a, blocks, s);
}

int core_blocks_per_cu(int vi) {
    if (vi < 0 || vi >= (int)(sizeof(kCoreOccupancy) / sizeof(kCoreOccupancy[0]))) return 1;
    const int n = kCoreOccupancy[vi]();
    return n > 0 ? n : 1;
}

hipError_t core_zero_counter(uint32_t* counter, hipStream_t s) {
    hipLaunchKernelGGL(k_zero_u32, dim3(1), dim3(1), 0, s, counter);
    return hipGetLastError();
}

hipError_t core_reduce_jobs(const ReduceArgs* jobs_dev, int32_t n_jobs, int64_t max_prog, hipStream_t s) {
    if (n_jobs <= 0 || max_prog <= 0) return hipSuccess;
    const uint32_t bx = (uint32_t)((max_prog + kProgs - 1) / kProgs);
    hipLaunchKernelGGL(k_reduce_jobs, dim3(bx, (uint32_t)n_jobs), dim3(256), 0, s, jobs_dev);
    return hipGetLastError();
}

hipError_t core_reduce_one(const ReduceArgs& r, hipStream_t s) {
    if (r.n_prog <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_reduce_one, dim3((uint32_t)((r.n_prog + kProgs - 1) / kProgs)), dim3(256), 0, s, r);
    return hipGetLastError();
}

}  // namespace gpx
