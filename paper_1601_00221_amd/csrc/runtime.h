// Host runtime internals shared by the evaluation, batching and serving code.
#pragma once

#include <hip/hip_runtime_api.h>
#include <stddef.h>
#include <stdint.h>

#include <functional>
#include <map>
#include <memory>
#include <mutex>
#include <utility>
#include <vector>

#include "../../include/gp.h"
#include "gp_internal.h"

namespace gpx {

gp_status fail(gp_status s, const char* fmt, ...) __attribute__((format(printf, 2, 3)));
void clear_error();
const char* last_error();

// Grow-only device buffer.  It owns its allocation: moving hands it over,
// destruction frees it.
struct DevBuf {
    void* p = nullptr;
    size_t cap = 0;
    DevBuf() = default;
    DevBuf(const DevBuf&) = delete;
    DevBuf& operator=(const DevBuf&) = delete;
    DevBuf(DevBuf&& o) noexcept : p(o.p), cap(o.cap) { o.p = nullptr; o.cap = 0; }
    DevBuf& operator=(DevBuf&& o) noexcept {
        if (this != &o) {
            release();
            p = o.p;
            cap = o.cap;
            o.p = nullptr;
            o.cap = 0;
        }
        return *this;
    }
    ~DevBuf() { release(); }
    gp_status reserve(size_t n);
    void release();
};

// Pinned host staging for host-to-device copies, in four parts used in
// turn: begin() takes the next part and waits only until the copies of
// its previous use (four uses ago) have left it, so a call does not
// wait for its own copies or for the kernels queued before them.
struct Staging {
    struct Half {
        void* host = nullptr;
        size_t cap = 0;
        hipEvent_t ev = nullptr;
        bool pending = false;
    };
    Half half[4];
    int cur = 0;
    size_t used = 0;
    gp_status begin(size_t n);
    gp_status put(const void* src, size_t n, void* dst, hipStream_t s);
    gp_status end(hipStream_t s);
    void release();
};

// Words that are all written before they are read: growing does not clear
// them (a population's code is a megabyte or more, fresh on every call).
template <typename T>
struct RawAlloc : std::allocator<T> {
    template <typename U>
    struct rebind {
        typedef RawAlloc<U> other;
    };
    template <typename U>
    void construct(U* p) noexcept {
        ::new ((void*)p) U;
    }
    template <typename U, typename... A>
    void construct(U* p, A&&... a) {
        ::new ((void*)p) U(std::forward<A>(a)...);
    }
};
typedef std::vector<uint32_t, RawAlloc<uint32_t>> RawWords;

// Lowered programs on the host.
struct ProgData {
    int form = 0;
    int opset = OPSET_REAL;  // function set of trees (OPSET_BOOL: Boolean, 32 cases per slot)
    int32_t n_prog = 0;
    int32_t n_feat = 0;     // declared feature count (register initialisation wraps around it)
    int32_t n_reg = 0;
    int32_t n_load = 1;     // features the programs actually read (max index + 1)
    int32_t max_depth = 0;
    int64_t n_instr = 0;    // instructions that are run (register programs: those the result depends on)
    int64_t n_named = 0;    // instructions as given
    int64_t n_gpop = 0;     // GP operations per case: tree nodes or linear instructions, as given
    int64_t n_transc = 0;   // sin/cos/exp/log instructions, as given (evaluated in binary64)
    RawWords code;
    std::vector<DevProg> progs;
    std::vector<uint32_t> cost;
    int variant = -1;       // default_variant of the programs, once asked for
};

// Rows: sin, cos, exp or log of a feature, computed once a tile by a block for
// all its programs (ring cores with those functions).
struct RowPlan {
    std::vector<int32_t> row;      // by function and feature: the row, or -1
    std::vector<uint32_t> op;      // of each row: GP_SIN .. GP_PLOG, or OP_PUSH: the feature itself
    std::vector<int32_t> feat;
    std::vector<uint32_t> rec;     // first record of each wave's share of the rows' programs, and the end
    std::vector<uint32_t> cost;    // of each program, its rows read instead of computed
    double total = 0.0;            // of all of them
    int32_t first_lds = 0;         // the first rows are the features from here on, on cores that hold them in LDS
    // The number of blocks a tile found best for the last number of tiles (and of groups to begin with): the search
    // for it takes some 2 us.  Written under the lock of the programs it belongs to.
    mutable struct { int32_t tiles = -1; int64_t base = 0, blocks = 0; double est = 0.0; } shape;
    int32_t n() const { return (int32_t)op.size(); }
    int32_t feature(int f) const { return f - first_lds; }
    uint32_t longest = 0;          // the largest of them
    void sum() {
        total = 0.0;
        longest = 0;
        for (uint32_t c : cost) {
            total += c;
            if (c > longest) longest = c;
        }
    }
};

// Device copies of programs translated for one core variant, plus their
// group layouts (the first record of each group) by group count.  `ready`
// is recorded on the stream of the last upload into these buffers; a launch
// on any stream waits for it.
struct DevProgs {
    bool uploaded = false;
    DevBuf code;
    std::vector<uint32_t> order;   // programs in the order of the code (host)
    std::vector<int64_t> rec;      // first record of each, in that order, and the end (host)
    RowPlan rows;
    std::map<int32_t, DevBuf> groups_by_G;
    DevBuf groups_once;        // one-shot calls: the group layout of the current programs
    hipEvent_t ready = nullptr;
    bool settled = false;          // `ready` has been seen to have passed: no launch waits for it any more
    DevProgs() = default;
    DevProgs(const DevProgs&) = delete;
    DevProgs& operator=(const DevProgs&) = delete;
    ~DevProgs() { release(); }
    void release() {
        uploaded = false;
        code.release();
        groups_by_G.clear();
        groups_once.release();
        if (ready) (void)hipEventDestroy(ready);
        ready = nullptr;
    }
};

// Per-stream scratch: partial sums, staging and the one-shot program buffers.
struct Workspace {
    std::mutex mu;
    DevBuf partials;
    Staging staging;
    std::map<int, DevProgs> oneshot;   // by core variant
    DevBuf bg_code, bg_meta;           // programs of the one-dimensional-stack comparator
};

// Consecutive programs of an evaluation whose results go to an array of their own.
struct EvalSegment {
    int32_t first, n_prog;
    void* out;
};

constexpr int kNoRows = 1 << 16;   // added to a variant's index: the key of its translation without rows

struct EvalOptions {
    int variant = -1;            // core variant index, -1 = chosen from the programs
    int32_t group_instr = 0;     // core instructions per program group, 0 = automatic
    int32_t tiles_per_wave = 0;  // tiles each wave walks per group, 0 = automatic
    int32_t target_blocks = 0;   // blocks the launch should have at least, 0 = automatic
    // Evaluation without any allocation or upload: the programs and the group
    // layout for `groups` groups are already on the device (a program set),
    // and the partial sums go to `partials` (at most `partials_bytes`).
    bool no_alloc = false;
    int32_t groups = 0;
    double* partials = nullptr;
    size_t partials_bytes = 0;
    // Several populations evaluated as one (not for GP_OUT_CASES): their parts of the programs, in order.
    const std::vector<EvalSegment>* segments = nullptr;
};

Workspace& workspace(hipStream_t s);
// Run fn over [0, n) split into chunks on a pool of host threads (the caller
// takes part); small ranges run on the calling thread.  Calls take turns.
void parallel_for(int64_t n, const std::function<void(int64_t, int64_t)>& fn);
int32_t code_prefetch();
// Programs by falling cost, and such a sequence cut into G groups of about
// equal cost (goff: G + 1 record offsets, from rec, each program's first
// record in that order and the end; gprog: the same as places in the order).
void cost_order(const std::vector<uint32_t>& cost, std::vector<uint32_t>& order);
void cut_groups(const std::vector<uint32_t>& cost, const std::vector<uint32_t>& order, const std::vector<int64_t>& rec,
                int32_t G, std::vector<uint32_t>& goff, std::vector<uint32_t>* gprog = nullptr);

// Kernel timing brackets (active only while gp_timing_enable(1)).
hipError_t timed_launch_begin(hipStream_t s, int* slot);
hipError_t timed_launch_end(hipStream_t s, int slot);

// The lowering of one population in steps, so that several are lowered in one
// walk of the host threads: begin checks the arrays' lengths and makes room
// (no program is read before), lower takes ranges of its n() programs in any
// order, side by side, and finish reports the first that failed.  The
// caller's arrays and pd are used until then.
class ProgBuild {
public:
    gp_status begin_tree(const int32_t* tok, const float* cst, const int64_t* off, int32_t P, int32_t n_feat, ProgData& pd,
                         int opset = OPSET_REAL);
    gp_status begin_linear(const uint32_t* code, const int64_t* off, const float* cst, const int64_t* cst_off, int32_t P,
                           int32_t n_reg, int32_t n_feat, ProgData& pd);
    int64_t n() const { return pd_ ? pd_->n_prog : 0; }
    void lower(int64_t p0, int64_t p1);
    gp_status finish();

private:
    void start(ProgData& pd, const int64_t* off);
    void lower_trees(int64_t p0, int64_t p1);
    void lower_linear(int64_t p0, int64_t p1);
    gp_status finish_trees();
    gp_status finish_linear();
    ProgData* pd_ = nullptr;       // null: nothing to lower
    const int64_t *off_ = nullptr, *cst_off_ = nullptr;
    const int32_t* tok_ = nullptr;
    const uint32_t* code_ = nullptr;
    const float *tcst_ = nullptr, *lcst_ = nullptr;
    std::vector<TreeLowering> lst;
    std::vector<int32_t> pfeat, prc, ptransc;   // of each program: highest feature, status, sin/cos/exp/log
};
gp_status build_tree(const int32_t* tok, const float* cst, const int64_t* off, int32_t P, int32_t n_feat,
                     ProgData& pd, int opset = OPSET_REAL);
gp_status build_linear(const uint32_t* code, const int64_t* off, const float* cst, const int64_t* cst_off,
                       int32_t P, int32_t n_reg, int32_t n_feat, ProgData& pd);
// The kernel variant an evaluation of these programs uses by default.
int default_variant(const ProgData& pd);
// Evaluate lowered programs on one case matrix.  dps caches the programs
// translated per core variant; fresh forces a new translation and upload.
// Boolean programs (pd.opset == OPSET_BOOL) take X and y as 32-bit words, N
// words per row, and n_bits > 0 cases; every other call passes n_bits = 0.
gp_status eval_core(const ProgData& pd, std::map<int, DevProgs>& dps, bool fresh, const float* X, int32_t n_feat,
                    int64_t N, const float* y, int32_t kind, void* out, hipStream_t s, Workspace* w,
                    const EvalOptions* opt, int64_t n_bits = 0);
}  // namespace gpx

struct gp_progset;

namespace gpx {
// Evaluate a program set as gp_progset_eval does, with nothing allocated or
// uploaded: the partial sums go to `partials` (device memory of
// `partials_bytes`); the set's programs and group layout were uploaded when
// it was created.
gp_status progset_eval_no_alloc(gp_progset* ps, const float* X, int32_t n_feat, int64_t n_cases, const float* y,
                                int32_t kind, void* out, hipStream_t s, double* partials, size_t partials_bytes);
// Program groups of a launch of variant vi over plentiful case tiles (the
// layout a program set uploads when it is created).
int32_t base_groups(const ProgData& pd, int vi, const EvalOptions* opt);

}  // namespace gpx
