// Evaluation kernel built around the hand-written interpreter core
// (gen_core.py).  One wavefront owns a case tile of 64 lanes x T slots
// (slot j of lane l is case tile*64*T + j*64 + l, so every feature row is
// read with contiguous 256-byte accesses, as the paper strides a thread's
// cases by the thread count, section 4.1).  The tile's features are loaded
// once into the core's VGPR range; then the wave interprets its programs on
// it.  The two-dimensional stack (section 4) is that VGPR range: one decoded
// instruction updates T slots of 64 lanes.
//
// The block runs a whole unit (a tile and consecutive programs): it loads the
// tile, interprets program after program, applies sin/cos/exp/log, and forms
// each program's fitness; the compiled code only finds the units.  sin, cos,
// exp and log are evaluated in binary64 and rounded once, with the arithmetic
// of gp_math.h: random GP trees chain many of them, and most such programs
// turn a last-place difference into a visible fitness difference, so a
// binary32 library result would make fitness depend on the evaluator.
//
// Fitness: per-slot error terms in binary32, per-lane binary64 sums over the
// 4 slots of each 256-case block, a fixed wavefront butterfly, one partial
// per (program, block), then a fixed-order reduction over blocks -- the
// result does not depend on the tile width, the grouping, or what else
// shared the launch.
//
// Kernel modes: 0 with the sin/cos/exp/log code, 1 without it (arithmetic
// programs), 3 like 1 for trees only, 4 like 0 for trees only, 2 the Boolean
// function set, whose slots are 32-bit words of bit-packed cases (32 cases
// per slot; a 256-slot block holds 8192 cases) and whose fitness is the
// number of output bits equal to the target bits.
//
// The classification fitness decodes an output to the class rint(o) and
// counts the cases whose class differs from y.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/gp.h"
#include "core_kernels.h"
#include "gp_internal.h"
#include "gp_math.h"

namespace gpx {
#include "core_gen.inc"

// Byte offsets in LDS that the block's sin/cos/exp/log address are built into
// it (LDS_SC .. LDS_PI in gen_core.py): the tables lie at offset 0, which the
// probe launch reports and the host checks.
static_assert(gmath::kTabSC == 0 && gmath::kTabExp == 256 && gmath::kTabLog == 320 &&
                  gmath::kTabPi == 320 + 2 * 257 && GPX_LOG_K0 == 0x7E6A,
              "the block's table offsets (gen_core.py)");

typedef __attribute__((address_space(3))) void* LdsPtr;
__device__ __forceinline__ uint32_t lds_address(const void* p) {
    return (uint32_t)(uintptr_t)(LdsPtr)(void*)p;
}

template <int T, int W, bool TABLES>
struct Shared {
    double tab[TABLES ? gmath::kTabSize + (gmath::kTabSize & 1) : 2];
    float y[W][64 * T];          // each wave's targets of its tile
};
// The rows of a block's tile (sin, cos, exp or log of a feature), behind Shared.
extern __shared__ __attribute__((aligned(16))) float s_rows[];

// A wave-uniform value in scalar registers.
__device__ __forceinline__ uint32_t uniform(uint32_t v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ uint64_t uniform(uint64_t v) {
    return (uint64_t)uniform((uint32_t)v) | ((uint64_t)uniform((uint32_t)(v >> 32)) << 32);
}

// Units come either from a table (batched launches: persistent waves pull
// them longest first from a counter, or one wave per unit) or implicitly
// over one dataset: block unit b = (W groups from W * (b div chunks) on, chunk
// b mod chunks); wave w of the block runs the w-th of those groups on tiles
// chunk * tiles_per_wave + i, i = 0 .. tiles_per_wave - 1.  The W waves of
// a block work on the same tiles with different instruction streams, so
// their scalar-cache misses do not fall on the same cycles.
template <int T, int D, int NF, int V0, int MODE, int W, bool ROWS>
__device__ __forceinline__ void k_core_body(const CoreArgs& a) {
    static_assert(T % 4 == 0, "a tile holds whole 256-case blocks");
    constexpr bool kTables = MODE == 0 || MODE == 4;
    __shared__ __attribute__((aligned(16))) Shared<T, W, kTables> sh;
    // the transcendentals' reduction tables, copied into LDS by the whole block
    if constexpr (kTables) {
        gmath::tab_fill(sh.tab, (int)threadIdx.x, (int)blockDim.x);
        __syncthreads();
    }
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t wib = uniform(threadIdx.x >> 6);
    const bool table = a.units != nullptr;
    uint32_t u, grp = 0, chunk = 0;
    if (table) {
        u = blockIdx.x * (uint32_t)W + wib;
    } else {
        // Blocks go to the 8 XCDs round robin; give each XCD a contiguous
        // range of block units so a program group's code stays in one L2.
        const uint32_t nb = gridDim.x, b = blockIdx.x;
        u = (b & 7u) * (nb >> 3) + (b >> 3);
        if (!a.probe) {
            if (u >= (uint32_t)a.n_units) return;
            if (a.direct) {
                // the block's waves run one group on all the tiles there are, and finish its fitness values
                grp = u;
                chunk = wib;
            } else if (a.same_group) {
                // wave w of the block runs group u div q on chunk W (u mod q) + w, q = chunks / W rounded up
                const uint32_t q = ((uint32_t)a.chunks + (uint32_t)W - 1u) / (uint32_t)W;
                grp = u / q;
                chunk = (u % q) * (uint32_t)W + wib;
                if (chunk >= (uint32_t)a.chunks) return;
            } else {
                grp = (u / (uint32_t)a.chunks) * (uint32_t)W + wib;
                chunk = u % (uint32_t)a.chunks;
            }
            // (a wave without a group still computes its share of the block's rows)
            if (grp >= (uint32_t)a.n_groups && !(ROWS && a.n_rows)) return;
        }
    }
    CoreUnit w;
    w.code = (uint64_t)a.code;
    w.coef = (uint64_t)gmath::kCoreCoef;
    w.lds_y = uniform(lds_address(sh.y[wib]));
    w.burst = (uint32_t)a.prefetch;
    for (uint32_t it = 0;; ++it) {
        uint32_t tile = 0, c0 = 0, c1 = 0;
        uint64_t pbase = 0;
        const float *X = nullptr, *y = nullptr;
        int64_t N = 1;
        int32_t n_load = 0, kind = 0;
        if (a.probe) {
            if (u != 0 || wib != 0) return;
        } else if (!table) {
            if (it >= (uint32_t)a.tiles_per_wave) break;
            tile = chunk * (uint32_t)a.tiles_per_wave + it;
            if (tile >= (uint32_t)a.tiles) break;
            if (grp < (uint32_t)a.n_groups) {
                c0 = a.group_off[grp];
                c1 = a.group_off[grp + 1];
            }
            X = a.X;
            y = a.y;
            N = a.N;
            n_load = a.n_load;
            kind = a.kind;
        } else {
            if (a.persistent) {
                uint32_t t = 0;
                if (lane == 0) t = atomicAdd(a.counter, 1u);
                u = uniform(t);
            } else if (it > 0) {
                return;
            }
            if (u >= (uint32_t)a.n_units) return;
            const UnitDesc ud = a.units[u];
            const JobDesc jd = a.jobs[ud.job];
            const DatasetDesc dd = a.datasets[jd.ds];
            tile = ud.tile;
            c0 = ud.c0;
            c1 = ud.c1;
            X = dd.X;
            y = dd.y;
            N = dd.N;
            n_load = jd.n_load;
            kind = jd.kind;
            pbase = jd.part_base;
        }
        const bool rows = ROWS && a.n_rows > 0;
        if (c0 >= c1 && !a.probe && !rows) continue;
        const int64_t tile0 = (int64_t)tile * (64 * T);        // first case of the tile
        const int64_t left = N - tile0, n_blocks = (N + 255) / 256;
        if constexpr (ROWS) {
            // first the wave's share of the rows: records row_off[w] .. row_off[w + 1)
            w.own_off = uniform(c0 * 16u);
            w.own_end = uniform(c1 * 16u);
            w.own_kind = rows ? uniform((uint32_t)kind) : 0xFFFFFFFFu;
            if (rows) {
                c0 = a.row_off[wib];
                c1 = a.row_off[wib + 1];
                kind = CORE_TO_ROW;
            }
        }
        w.off = uniform(c0 * 16u);
        w.end = uniform(c1 * 16u);
        w.X = uniform((uint64_t)(X + tile0));
        w.stride = uniform((uint64_t)N * 4u);
        // (per-case outputs need no targets, but a block that starts with rows loads some: a feature then)
        w.y = uniform((uint64_t)((y ? y : X) + tile0));
        w.n_load = uniform((uint32_t)n_load);
        w.left = uniform((uint32_t)(left < 64 * T ? left : 64 * T));
        w.kind = uniform((uint32_t)kind);
        w.partials = uniform((uint64_t)(a.partials + pbase + (int64_t)tile * (T / 4)));
        w.part_stride = uniform((uint32_t)(n_blocks * 8));
        w.cases = uniform((uint64_t)(a.cases_out + tile0));
        const int64_t bits = MODE == 2 ? a.n_bits - 32 * tile0 : 0;
        w.bits = uniform((uint32_t)(bits < 2048 * T ? bits : 2048 * T));
        // The block's asm (with its handler table and labels) must exist once
        // in the kernel (the assembler rejects a second copy): the probe flag
        // is laundered on every pass, so the loop is neither split nor peeled.
        uint32_t probe = a.probe;
        asm volatile("" : "+s"(probe));
        uint64_t handlers;
        Core<T, D, NF, V0, MODE>::run(w, probe, handlers);
        if (probe) {
            if (threadIdx.x == 0) {
                a.probe_out[0] = handlers;
                a.probe_out[1] = lds_address(sh.tab);
                a.probe_out[2] = ROWS ? lds_address(s_rows) : 0u;
            }
            return;
        }
    }
    if (!table && a.direct) {
        // The group's partial sums were written by this block (the stores have been waited for): a thread a program
        // adds them up in block order.  Read past the vector cache, which may not hold another wave's stores.
        __syncthreads();
        const uint32_t q1 = a.group_prog[grp + 1];
        const int32_t n_blocks = (int32_t)((a.N + 255) / 256);
        for (uint32_t q = a.group_prog[grp] + threadIdx.x; q < q1; q += blockDim.x) {
            const uint64_t p = a.order[q];
            double sum = 0.0;
            for (int32_t b = 0; b < n_blocks; b++)
                sum += __hip_atomic_load(a.partials + p * (uint64_t)n_blocks + b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            finish_sum(a.kind, a.N, a.out, (int64_t)p, sum);
        }
    }
}

// One kernel per variant.  amdgpu_num_vgpr(n) lets the compiler allocate 2n
// VGPRs on gfx950 (checked at build time against the compiler's
// reserved-register report); the core owns v[V0 ...].  MODE: 0 full, 1 no
// sin/cos/exp/log code (for programs without them), 2 Boolean, 3 trees only
// without sin/cos/exp/log code, 4 trees only with it.
// W: waves of a block; ROWS: the block computes rows for its tile first.
#define GPX_KERNEL(T, D, NF, V0, MODE, W, ROWS, NAME)                                                   \
    __global__ __launch_bounds__(64 * (W)) __attribute__((amdgpu_num_vgpr((V0) / 2))) void              \
        k_core_##NAME(CoreArgs a) {                                                                     \
        k_core_body<T, D, NF, V0, (MODE), (W), (ROWS)>(a);                                              \
    }

}  // namespace gpx
