// Host runtime of the GP population evaluator: argument checks, program
// lowering and upload, scheduling of (case tile, program group) units, and
// the C ABI declared in include/gp.h.
#include <hip/hip_runtime_api.h>
#include <stdarg.h>
#include <stdlib.h>
#include <stdio.h>
#include <string.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <condition_variable>
#include <exception>
#include <functional>
#include <map>
#include <memory>
#include <mutex>
#include <numeric>
#include <thread>
#include <unordered_map>
#include <vector>

#include "../../include/gp.h"
#include "core_host.h"
#include "core_kernels.h"
#include "gp_internal.h"
#include "runtime.h"

namespace gpx {

// ---------------------------------------------------------------------------
// Errors
// ---------------------------------------------------------------------------
static thread_local char t_err[512] = "";

gp_status fail(gp_status s, const char* fmt, ...) {
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(t_err, sizeof t_err, fmt, ap);
    va_end(ap);
    return s;
}
void clear_error() { t_err[0] = 0; }
const char* last_error() { return t_err; }

// ---------------------------------------------------------------------------
// Buffers
// ---------------------------------------------------------------------------
gp_status DevBuf::reserve(size_t n) {
    if (n <= cap) return GP_OK;
    if (p) {
        hipError_t e = hipFree(p);  // waits for the device before releasing
        p = nullptr;
        cap = 0;
        if (e != hipSuccess) return fail(GP_E_DEVICE, "hipFree: %s", hipGetErrorString(e));
    }
    size_t want = n < 4096 ? 4096 : n + n / 4;
    hipError_t e = hipMalloc(&p, want);
    if (e != hipSuccess) {
        p = nullptr;
        return fail(e == hipErrorOutOfMemory ? GP_E_NOMEM : GP_E_DEVICE, "hipMalloc(%zu): %s", want,
                    hipGetErrorString(e));
    }
    cap = want;
    return GP_OK;
}

void DevBuf::release() {
    if (p) (void)hipFree(p);
    p = nullptr;
    cap = 0;
}

gp_status Staging::begin(size_t n) {
    cur = (cur + 1) & 3;
    Half& h = half[cur];
    if (h.pending) {
        hipError_t e = hipEventSynchronize(h.ev);
        if (e != hipSuccess) return fail(GP_E_DEVICE, "hipEventSynchronize: %s", hipGetErrorString(e));
        h.pending = false;
    }
    if (!h.ev) {
        hipError_t e = hipEventCreateWithFlags(&h.ev, hipEventDisableTiming);
        if (e != hipSuccess) return fail(GP_E_DEVICE, "hipEventCreate: %s", hipGetErrorString(e));
    }
    if (n > h.cap) {
        if (h.host) (void)hipHostFree(h.host);
        h.host = nullptr;
        h.cap = 0;
        size_t want = n < 65536 ? 65536 : n + n / 4;
        hipError_t e = hipHostMalloc(&h.host, want, hipHostMallocDefault);
        if (e != hipSuccess) {
            h.host = nullptr;
            return fail(GP_E_NOMEM, "hipHostMalloc(%zu): %s", want, hipGetErrorString(e));
        }
        h.cap = want;
    }
    used = 0;
    return GP_OK;
}

void parallel_for(int64_t n, const std::function<void(int64_t, int64_t)>& fn);

gp_status Staging::put(const void* src, size_t n, void* dst, hipStream_t s) {
    if (n == 0) return GP_OK;
    Half& h = half[cur];
    if (used + n > h.cap) return fail(GP_E_INVAL, "internal: staging overflow (%zu + %zu > %zu)", used, n, h.cap);
    char* to = (char*)h.host + used;
    if (n >= ((size_t)1 << 22)) {
        // a large program set: copy into the pinned buffer on the host threads, 64 KiB apiece
        const int64_t pieces = (int64_t)((n + ((size_t)1 << 16) - 1) >> 16);
        parallel_for(pieces, [&](int64_t i0, int64_t i1) {
            const size_t a = (size_t)i0 << 16, b = std::min(n, (size_t)i1 << 16);
            memcpy(to + a, (const char*)src + a, b - a);
        });
    } else {
        memcpy(to, src, n);
    }
    hipError_t e = hipMemcpyAsync(dst, to, n, hipMemcpyHostToDevice, s);
    if (e != hipSuccess) return fail(GP_E_DEVICE, "hipMemcpyAsync: %s", hipGetErrorString(e));
    used += (n + 255) & ~(size_t)255;
    return GP_OK;
}

gp_status Staging::end(hipStream_t s) {
    Half& h = half[cur];
    hipError_t e = hipEventRecord(h.ev, s);
    if (e != hipSuccess) return fail(GP_E_DEVICE, "hipEventRecord: %s", hipGetErrorString(e));
    h.pending = true;
    return GP_OK;
}

void Staging::release() {
    for (Half& h : half) {
        if (h.pending && h.ev) (void)hipEventSynchronize(h.ev);
        if (h.host) (void)hipHostFree(h.host);
        if (h.ev) (void)hipEventDestroy(h.ev);
        h = Half();
    }
    used = 0;
}

static std::mutex g_ws_mu;
static std::unordered_map<hipStream_t, Workspace*> g_ws;

Workspace& workspace(hipStream_t s) {
    std::lock_guard<std::mutex> g(g_ws_mu);
    auto it = g_ws.find(s);
    if (it != g_ws.end()) return *it->second;
    Workspace* w = new Workspace();  // lives until process exit
    g_ws[s] = w;
    return *w;
}

// ---------------------------------------------------------------------------
// Host threads: a fixed pool that splits a range of programs
// ---------------------------------------------------------------------------
namespace {
// One range being worked on.  Threads hold it by shared pointer: one that
// wakes up late finds nothing left to take and never touches `fn`, which is
// the caller's and is used only while items are outstanding.
struct Work {
    const std::function<void(int64_t, int64_t)>* fn;
    int64_t n, chunk;
    std::atomic<int64_t> next{0}, done{0};
    std::atomic<bool> failed{false};
    std::exception_ptr error;   // the first one, thrown again by the caller when every item has ended
    Work(const std::function<void(int64_t, int64_t)>* f, int64_t count, int64_t c) : fn(f), n(count), chunk(c) {}
    void take() {
        for (;;) {
            const int64_t lo = next.fetch_add(chunk);
            if (lo >= n) return;
            const int64_t hi = std::min(n, lo + chunk);
            try {
                (*fn)(lo, hi);
            } catch (...) {
                if (!failed.exchange(true)) error = std::current_exception();
            }
            done.fetch_add(hi - lo, std::memory_order_acq_rel);
        }
    }
};

// The caller works from the start and returns when every item is done, however
// many threads have woken up by then (waiting for all fifteen to report took
// 100-200 us a range).  A thread that has run out of work looks for the next
// range for some 50 us before it sleeps: lowering and translation follow each
// other within one call.
struct Pool {
    std::mutex mu;
    std::condition_variable cv;
    std::vector<std::thread> th;
    std::shared_ptr<Work> work;
    std::atomic<uint64_t> gen{0};
    bool stop = false;

    explicit Pool(int k) {
        for (int i = 0; i < k; i++) th.emplace_back([this] { worker(); });
    }
    ~Pool() {
        {
            std::lock_guard<std::mutex> g(mu);
            stop = true;
            gen++;
        }
        cv.notify_all();
        for (auto& t : th) t.join();
    }
    void worker() {
        uint64_t seen = 0;
        for (;;) {
            for (int spin = 0; spin < 2000 && gen.load(std::memory_order_acquire) == seen; spin++) __builtin_ia32_pause();
            std::shared_ptr<Work> w;
            {
                std::unique_lock<std::mutex> lk(mu);
                cv.wait(lk, [&] { return stop || gen.load() != seen; });
                if (stop) return;
                seen = gen.load();
                w = work;
            }
            if (w) w->take();
        }
    }
    void run(int64_t count, const std::function<void(int64_t, int64_t)>& f) {
        auto w = std::make_shared<Work>(&f, count, std::max<int64_t>(1, count / (8 * (int64_t)(th.size() + 1))));
        {
            std::lock_guard<std::mutex> g(mu);
            work = w;
            gen++;
        }
        cv.notify_all();
        w->take();
        while (w->done.load(std::memory_order_acquire) < count) __builtin_ia32_pause();   // the last chunks of others
        {
            std::lock_guard<std::mutex> g(mu);
            if (work == w) work.reset();
        }
        if (w->failed) std::rethrow_exception(w->error);
    }
};

std::mutex g_pool_mu;   // one parallel_for at a time (calls from several host threads take turns)
}  // namespace

void parallel_for(int64_t n, const std::function<void(int64_t, int64_t)>& fn) {
    if (n <= 0) return;
    if (n < 64) {
        fn(0, n);
        return;
    }
    static Pool* pool = [] {
        const unsigned hc = std::thread::hardware_concurrency();
        return new Pool((int)std::max(1u, std::min(16u, hc ? hc : 1u)) - 1);   // the caller is the last thread
    }();
    std::lock_guard<std::mutex> g(g_pool_mu);
    pool->run(n, fn);
}

// ---------------------------------------------------------------------------
// Program building
// ---------------------------------------------------------------------------
// Relative cost of one instruction, used only to balance program groups:
// the vector instructions it issues per slot, plus one for its dispatch.
// Protected division takes 13 to 15 a slot, the compares, IF and AND/OR a
// compare or two and a select, sin and cos some 34, exp and log 24 (binary64).
// Every Boolean function is one bitwise instruction per slot.
static uint32_t op_cost(uint32_t op, int opset) {
    if (opset == OPSET_BOOL) return 2;
    switch (op) {
        case GP_PDIV: return 16;
        case GP_GT: case GP_LT: case GP_EQ: case OP_IF: return 3;
        case GP_AND: case GP_OR: return 4;
        case GP_SIN: case GP_COS: return 35;
        case GP_EXPC: case GP_PLOG: return 25;
        default: return 2;
    }
}

gp_status ProgBuild::begin_tree(const int32_t* tok, const float* cst, const int64_t* off, int32_t P, int32_t n_feat,
                                ProgData& pd, int opset) {
    if (P < 0) return fail(GP_E_INVAL, "n_prog < 0");
    if (P > 0 && (!tok || (!cst && opset != OPSET_BOOL) || !off)) return fail(GP_E_INVAL, "null program array");
    if (n_feat < 1) return fail(GP_E_INVAL, "n_feat < 1");
    pd = ProgData();
    pd.form = FORM_TREE;
    pd.opset = opset;
    pd.n_prog = P;
    pd.n_feat = n_feat;
    if (P == 0) return GP_OK;
    if (off[0] != 0) return fail(GP_E_INVAL, "off[0] must be 0");
    int64_t total = 0;
    for (int32_t p = 0; p < P; p++) {
        const int64_t n = off[p + 1] - off[p];
        if (n < 1) return fail(GP_E_INVAL, "program %d is empty", p);
        if (n > GP_MAX_LEN) return fail(GP_E_DEPTH, "program %d: %lld nodes exceeds %d", p, (long long)n, GP_MAX_LEN);
        total += n;
    }
    if (total > 0x7FFFFFFFll) return fail(GP_E_INVAL, "programs exceed 2^31 nodes");
    // Program p is lowered at word 2 * off[p] (at most one instruction per
    // node), so the programs are independent: they are lowered in parallel.
    pd.code.resize((size_t)total * 2);
    start(pd, off);
    lst.resize(P);
    tok_ = tok;
    tcst_ = cst;
    return GP_OK;
}

void ProgBuild::start(ProgData& pd, const int64_t* off) {
    pd_ = &pd;
    off_ = off;
    pd.progs.resize(pd.n_prog);
    pd.cost.resize(pd.n_prog);
    pfeat.assign(pd.n_prog, -1);
    prc.assign(pd.n_prog, GP_OK);
    ptransc.assign(pd.n_prog, 0);
}

void ProgBuild::lower_trees(int64_t p0, int64_t p1) {
    ProgData& pd = *pd_;
    const int64_t* off = off_;
    const int opset = pd.opset;
    char err[256];
    for (int64_t p = p0; p < p1; p++) {
        const int64_t n = off[p + 1] - off[p];
        uint32_t* words = pd.code.data() + 2 * off[p];
        const int rc = lower_tree(tok_ + off[p], tcst_ ? tcst_ + off[p] : nullptr, n, pd.n_feat, words, &lst[p], err, opset);
        if (rc != GP_OK) {
            prc[p] = rc;
            return;
        }
        int32_t mf = -1;
        for (int64_t i = 0; i < n; i++) {
            const int32_t t = tok_[off[p] + i];
            if ((t & 0xFF) == GP_VAR) mf = std::max<int32_t>(mf, (int32_t)((uint32_t)t >> 8));
        }
        pfeat[p] = mf;
        uint32_t cost = 0;
        int32_t nt = 0;
        for (int32_t i = 0; i < lst[p].n_instr; i++) {
            const uint32_t op = words[2 * i] & 15u;
            cost += op_cost(op, opset);
            nt += opset != OPSET_BOOL && op >= GP_SIN && op <= GP_PLOG;
        }
        ptransc[p] = nt;
        pd.cost[p] = cost + 16;
    }
}

gp_status ProgBuild::finish_trees() {
    ProgData& pd = *pd_;
    const int64_t* off = off_;
    int32_t max_feat = -1;
    for (int32_t p = 0; p < pd.n_prog; p++) {
        if (prc[p] != GP_OK) {
            // lower the first failing program again on this thread for its message
            char err[256];
            TreeLowering st;
            lower_tree(tok_ + off[p], tcst_ ? tcst_ + off[p] : nullptr, off[p + 1] - off[p], pd.n_feat, nullptr, &st, err,
                       pd.opset);
            return fail((gp_status)prc[p], "program %d: %s", p, err);
        }
        const TreeLowering& st = lst[p];
        DevProg& d = pd.progs[p];
        d.code_off = (uint32_t)(2 * off[p]);
        d.len = (uint32_t)st.n_instr;
        d.meta = FORM_TREE | ((uint32_t)st.max_depth << 8);
        d.live = 0;
        d.reserved1 = 0;
        d.row = (uint64_t)p;
        max_feat = std::max(max_feat, pfeat[p]);
        pd.n_transc += ptransc[p];
        pd.max_depth = std::max(pd.max_depth, st.max_depth);
        pd.n_instr += st.n_instr;
        pd.n_gpop += st.n_nodes;
    }
    pd.n_named = pd.n_instr;
    pd.n_load = max_feat + 1 > 0 ? max_feat + 1 : 1;
    return GP_OK;
}

gp_status ProgBuild::begin_linear(const uint32_t* code, const int64_t* off, const float* cst, const int64_t* cst_off,
                                  int32_t P, int32_t n_reg, int32_t n_feat, ProgData& pd) {
    if (P < 0) return fail(GP_E_INVAL, "n_prog < 0");
    if (P > 0 && (!code || !off)) return fail(GP_E_INVAL, "null program array");
    if (n_reg < 1 || n_reg > GP_MAX_REG) return fail(GP_E_INVAL, "n_reg %d outside [1, %d]", n_reg, GP_MAX_REG);
    if (n_feat < 1 || n_reg + n_feat > GP_SRC_CONST)
        return fail(GP_E_INVAL, "n_feat %d: registers plus features must stay below %d", n_feat, GP_SRC_CONST);
    pd = ProgData();
    pd.form = FORM_LINEAR;
    pd.n_prog = P;
    pd.n_feat = n_feat;
    pd.n_reg = n_reg;
    if (P == 0) return GP_OK;
    if (off[0] != 0) return fail(GP_E_INVAL, "off[0] must be 0");
    if (cst_off && cst_off[0] != 0) return fail(GP_E_INVAL, "cst_off[0] must be 0");
    int64_t total = 0;
    for (int32_t p = 0; p < P; p++) {
        const int64_t n = off[p + 1] - off[p];
        const int64_t nc = cst_off ? cst_off[p + 1] - cst_off[p] : 0;
        if (n < 1) return fail(GP_E_INVAL, "program %d is empty", p);
        if (n > GP_MAX_LEN) return fail(GP_E_DEPTH, "program %d: %lld instructions exceeds %d", p, (long long)n, GP_MAX_LEN);
        if (nc < 0 || nc > 256 - GP_SRC_CONST) return fail(GP_E_INVAL, "program %d: %lld constants", p, (long long)nc);
        if (nc > 0 && !cst) return fail(GP_E_INVAL, "null constant array");
        total += n + nc;
    }
    if (total > 0xFFFFFFFFll) return fail(GP_E_INVAL, "programs exceed 2^32 device words");
    // Program p lies at word off[p] plus the constants before it, so the programs are independent: they are checked,
    // freed of the instructions that the result does not depend on, and copied in parallel.
    pd.code.resize((size_t)total);
    start(pd, off);
    code_ = code;
    lcst_ = cst;
    cst_off_ = cst_off;
    return GP_OK;
}

void ProgBuild::lower_linear(int64_t p0, int64_t p1) {
    ProgData& pd = *pd_;
    const int64_t *off = off_, *cst_off = cst_off_;
    const int32_t n_reg = pd.n_reg;
    char err[256];
    for (int64_t p = p0; p < p1; p++) {
        const int64_t n = off[p + 1] - off[p];
        const int64_t c0 = cst_off ? cst_off[p] : 0, nc = cst_off ? cst_off[p + 1] - c0 : 0;
        const uint32_t* src = code_ + off[p];
        if ((prc[p] = check_linear(src, n, nc, n_reg, pd.n_feat, err)) != GP_OK) return;
        for (int64_t i = 0; i < n; i++) {
            const uint32_t wd = src[i];
            const bool unary = (wd & 0xFF) >= GP_SIN && (wd & 0xFF) <= GP_PLOG;
            ptransc[p] += unary;
            for (int q = 0; q < (unary ? 1 : 2); q++) {
                const int32_t id = (int32_t)((wd >> (16 + 8 * q)) & 0xFF);
                if (id >= n_reg && id < GP_SRC_CONST) pfeat[p] = std::max(pfeat[p], id - n_reg);
            }
        }
        uint32_t* dst = pd.code.data() + off[p] + c0;
        DevProg& d = pd.progs[p];
        d.code_off = (uint32_t)(off[p] + c0);
        d.len = (uint32_t)needed_linear(src, n, n_reg, dst, &d.live);
        if (nc) memcpy(dst + d.len, lcst_ + c0, sizeof(float) * (size_t)nc);
        d.meta = FORM_LINEAR | ((uint32_t)n_reg << 8);
        d.reserved1 = 0;
        d.row = (uint64_t)p;
        uint32_t cost = 2u * (uint32_t)__builtin_popcount(d.live);
        for (uint32_t i = 0; i < d.len; i++) cost += op_cost(dst[i] & 0xFF, OPSET_REAL);
        pd.cost[p] = cost + 16;
    }
}

gp_status ProgBuild::finish_linear() {
    ProgData& pd = *pd_;
    const int64_t *off = off_, *cst_off = cst_off_;
    int32_t max_feat = std::min(pd.n_feat, pd.n_reg) - 1;  // registers start from these features
    for (int32_t p = 0; p < pd.n_prog; p++) {
        const int64_t n = off[p + 1] - off[p];
        if (prc[p] != GP_OK) {
            // check the first failing program again on this thread for its message
            char err[256];
            check_linear(code_ + off[p], n, cst_off ? cst_off[p + 1] - cst_off[p] : 0, pd.n_reg, pd.n_feat, err);
            return fail((gp_status)prc[p], "program %d: %s", p, err);
        }
        max_feat = std::max(max_feat, pfeat[p]);
        pd.n_transc += ptransc[p];
        pd.n_instr += pd.progs[p].len;
        pd.n_named += n;
        pd.n_gpop += n;
    }
    pd.n_load = max_feat + 1;
    return GP_OK;
}

void ProgBuild::lower(int64_t p0, int64_t p1) {
    if (pd_->form == FORM_TREE) lower_trees(p0, p1);
    else lower_linear(p0, p1);
}

gp_status ProgBuild::finish() {
    if (!pd_) return GP_OK;   // no programs
    return pd_->form == FORM_TREE ? finish_trees() : finish_linear();
}

static gp_status run_build(gp_status begun, ProgBuild& b) {
    if (begun != GP_OK) return begun;
    parallel_for(b.n(), [&](int64_t p0, int64_t p1) { b.lower(p0, p1); });
    return b.finish();
}

gp_status build_tree(const int32_t* tok, const float* cst, const int64_t* off, int32_t P, int32_t n_feat, ProgData& pd,
                     int opset) {
    ProgBuild b;
    return run_build(b.begin_tree(tok, cst, off, P, n_feat, pd, opset), b);
}

gp_status build_linear(const uint32_t* code, const int64_t* off, const float* cst, const int64_t* cst_off, int32_t P,
                       int32_t n_reg, int32_t n_feat, ProgData& pd) {
    ProgBuild b;
    return run_build(b.begin_linear(code, off, cst, cst_off, P, n_reg, n_feat, pd), b);
}

// Programs by falling cost: the order their code lies in on the device.
void cost_order(const std::vector<uint32_t>& cost, std::vector<uint32_t>& order) {
    order.resize(cost.size());
    std::iota(order.begin(), order.end(), 0u);
    std::stable_sort(order.begin(), order.end(), [&](uint32_t a, uint32_t b) { return cost[a] > cost[b]; });
}

// Cut the programs, in that order, into G runs of about equal cost: a group
// is a range of records, so a wave walks one stream of code.  Each group takes
// programs up to the mean of what is left (at least one), so with as many
// groups as programs each holds one.
void cut_groups(const std::vector<uint32_t>& cost, const std::vector<uint32_t>& order, const std::vector<int64_t>& rec,
                int32_t G, std::vector<uint32_t>& goff, std::vector<uint32_t>* gprog) {
    const int32_t P = (int32_t)cost.size();
    double left = 0.0;
    for (int32_t i = 0; i < P; i++) left += cost[order[i]];
    goff.assign(1, (uint32_t)rec[0]);
    if (gprog) gprog->assign(1, 0u);
    int32_t i = 0;
    for (int32_t g = 0; g < G; g++) {
        const double want = left / (G - g);
        const int32_t most = P - (G - g - 1);     // leave one program for each later group
        double got = 0.0;
        while (i < most && (got == 0.0 || got + 0.5 * cost[order[i]] <= want)) got += cost[order[i++]];
        if (g == G - 1) i = P;
        left -= got;
        goff.push_back((uint32_t)rec[i]);
        if (gprog) gprog->push_back((uint32_t)i);
    }
}

// Order a launch on stream s after the upload of dp, on whichever stream that
// was, unless the upload is known to have passed.  The event is not queried
// while s is being captured (that would end the capture), and otherwise in the
// relaxed capture mode: in the default mode a query is refused while any thread
// captures a stream in the global mode, and ends that capture.  A wait for an
// event from outside a capture may be refused too: a captured evaluation relies
// on an earlier one's having seen the upload pass.
static gp_status wait_for_upload(DevProgs& dp, hipStream_t s) {
    if (dp.settled) return GP_OK;
    hipStreamCaptureStatus cap = hipStreamCaptureStatusActive;
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    if (hipStreamIsCapturing(s, &cap) == hipSuccess && cap == hipStreamCaptureStatusNone &&
        hipThreadExchangeStreamCaptureMode(&mode) == hipSuccess) {
        dp.settled = hipEventQuery(dp.ready) == hipSuccess;
        (void)hipThreadExchangeStreamCaptureMode(&mode);
    }
    if (dp.settled) return GP_OK;
    (void)hipGetLastError();   // "not yet" is no error: it must not be taken for a launch's
    const hipError_t e = hipStreamWaitEvent(s, dp.ready, 0);
    if (e == hipSuccess) return GP_OK;
    (void)hipGetLastError();
    return fail(GP_E_DEVICE, "hipStreamWaitEvent: %s", hipGetErrorString(e));
}

// Translate and upload the programs for variant vi (when `fresh` or not yet
// uploaded; dp.rows is planned) and the group layout for G groups (when not cached), all in one
// staging pass on stream s, then record dp.ready on s.  One-shot calls
// (`fresh`) keep a single group layout, replaced on every call.  G <= 0:
// programs only.
static gp_status prepare_programs(const ProgData& pd, int vi, DevProgs& dp, bool fresh, int32_t G, hipStream_t s,
                                  Workspace& w, const uint32_t** goff) {
    RawWords code;
    std::vector<uint32_t> g, gprog;
    gp_status st;
    const bool upload = fresh || !dp.uploaded;
    if (!upload && (st = wait_for_upload(dp, s)) != GP_OK) return st;
    if (upload) {
        std::vector<DevProg> progs;
        cost_order(dp.rows.cost, dp.order);
        if ((st = core_translate(pd, vi, dp.order.data(), &dp.rows, code, progs)) != GP_OK) return st;
        dp.rec.resize((size_t)pd.n_prog + 1);
        for (int32_t i = 0; i < pd.n_prog; i++) dp.rec[i] = progs[dp.order[i]].code_off / 4;
        const DevProg& last = progs[dp.order[pd.n_prog - 1]];
        dp.rec[pd.n_prog] = last.code_off / 4 + last.len;
    }
    DevBuf made;   // a new layout of a program set: kept once it has been uploaded
    DevBuf* gb = nullptr;
    if (fresh) {
        gb = &dp.groups_once;
    } else {
        auto it = dp.groups_by_G.find(G);
        if (it != dp.groups_by_G.end()) gb = &it->second;
    }
    const bool new_groups = G > 0 && (fresh || gb == nullptr);
    if (new_groups) {
        // the groups' records, each wave's share of the rows, the groups' programs and the programs' order
        cut_groups(dp.rows.cost, dp.order, dp.rec, G, g, &gprog);
        g.insert(g.end(), dp.rows.rec.begin(), dp.rows.rec.end());
        g.insert(g.end(), gprog.begin(), gprog.end());
        g.insert(g.end(), dp.order.begin(), dp.order.end());
        if (!fresh) gb = &made;
        if ((st = gb->reserve(g.size() * 4)) != GP_OK) return st;
    }
    if (upload || new_groups) {
        if (upload && (st = dp.code.reserve(std::max<size_t>(16, code.size() * 4))) != GP_OK) return st;
        const size_t bytes = code.size() * 4 + g.size() * 4 + 1024;
        if ((st = w.staging.begin(bytes)) != GP_OK) return st;
        if (upload && (st = w.staging.put(code.data(), code.size() * 4, dp.code.p, s)) != GP_OK) return st;
        if (new_groups && (st = w.staging.put(g.data(), g.size() * 4, gb->p, s)) != GP_OK) return st;
        if ((st = w.staging.end(s)) != GP_OK) return st;
        if (!dp.ready) {
            hipError_t e = hipEventCreateWithFlags(&dp.ready, hipEventDisableTiming);
            if (e != hipSuccess) return fail(GP_E_DEVICE, "hipEventCreate: %s", hipGetErrorString(e));
        }
        hipError_t e = hipEventRecord(dp.ready, s);
        if (e != hipSuccess) return fail(GP_E_DEVICE, "hipEventRecord: %s", hipGetErrorString(e));
        dp.uploaded = true;
        dp.settled = false;
        if (gb == &made) gb = &(dp.groups_by_G[G] = std::move(made));
    }
    if (goff) *goff = gb ? (const uint32_t*)gb->p : nullptr;
    return GP_OK;
}

// Launch shape of one evaluation.  Programs are cut into G groups; each block
// runs W groups (one per wave) on a chunk of tiles_per_wave tiles.  With tiles
// enough for the chip a group holds about `group_instr` core instructions.  A
// block takes one tile (two or more were no faster anywhere: 1, 2, 4 tiles took
// 38.2, 38.5, 39.2 ms on 41-feature classification trees x 494021 cases, 6.30,
// 6.40, 7.04 ms on 8-feature trees x 65536), until there are 2^24 blocks.  With
// fewer tiles the programs are cut into more groups, by the
// estimate below.  (Cutting them until there were those 4096 blocks had waves
// of one or two programs that mostly loaded their tile: the estimate takes
// 158 -> 109 us for 100 programs of up to 512 nodes x 30000 cases, 235 -> 160
// for 4096 programs x 1000 cases, 433 -> 336 for 4096 classification trees over 41 features x 3000, 53 -> 30 for 1024 Boolean programs x 32000, and over 100
// pairs of a population and a number of cases it is within 4 % of the best
// number of blocks, where the old rule was 22 % above it.)
struct LaunchShape {
    int32_t G, tiles_per_wave, chunks;
    double est;   // launch_time of G, 0: not asked for
};

static int32_t env_int(const char* name, int32_t dflt) {
    const char* v = getenv(name);
    if (!v || !*v) return dflt;
    const long x = strtol(v, nullptr, 10);
    return x > 0 && x < (1L << 30) ? (int32_t)x : dflt;
}

int32_t code_prefetch() {
    // GP2D_CODE_PREFETCH: 0 = no burst load, n = n lines in flight beside the next records (at most 14:
    // the scalar memory counter holds 15 loads), unset = 14
    const char* v = getenv("GP2D_CODE_PREFETCH");
    if (!v || !*v) return 14;
    const long n = strtol(v, nullptr, 10);
    return n <= 0 ? 0 : (n > 14 ? 14 : (int32_t)n);
}

// Groups of a launch with tiles enough for them.
int32_t base_groups(const ProgData& pd, int vi, const EvalOptions* opt) {
    // Program groups of about 1536 core instructions when the programs read at most 12 features, else 6144 (4096 of
    // Boolean programs, 2048 where features lie in LDS): every wave loads the features of its tile before it runs its group, and a longer
    // group spreads those loads over more instructions; a block's rows, too, are computed for all its groups.
    // Measured on the 4096-program workloads (1024, 1536, 2048, 4096): 8-feature trees 6.34, 6.29, 6.29, 6.4 ms
    // (sin/cos/exp/log) and 587, 578, 582, 600 us (+, -, *), 9-feature classification trees 1.48, 1.47, 1.47, 1.51 ms;
    // 16-feature linear programs 3.17, 3.16, 3.16, 3.02 ms (2.96 with 6144), 16-feature classification trees without
    // sin/cos/exp/log 1.61 and 1.58 ms (4096, 6144), 20-input multiplexer trees 455, 452, 453, 449 us, and
    // 41-feature classification trees with features in LDS 2048 against 4096: 39.5, 40.1 ms.
    const int32_t usual = core_variant_cap(vi) > core_variant_nf(vi) ? 2048
                          : pd.n_load <= 12 ? 1536 : pd.opset == OPSET_BOOL ? 4096 : 6144;
    const int32_t group_instr = opt && opt->group_instr > 0 ? opt->group_instr : env_int("GP2D_GROUP_INSTR", usual);
    // (the end of a program takes about as long as four instructions)
    const int64_t G = (pd.n_instr + 4 * (int64_t)pd.n_prog + group_instr - 1) / group_instr;
    // (whole blocks: 836 trees x 200000 cases, 20 groups of eight waves' blocks 2.68 ms, 16 or 24 groups 1.98)
    const int64_t W = core_variant_waves(vi);
    return (int32_t)std::max<int64_t>(1, std::min<int64_t>(W * ((G + W / 2) / W + (G < W / 2)), pd.n_prog));
}

// An estimate of how long `blocks` blocks a tile take, in the time of one
// vector instruction a slot (4 T cycles), fitted to the times of 100 launches
// at 12 numbers of blocks each.  A SIMD that holds 1, 2, 3 or 4 waves runs at
// `rate` of its peak.  A wave loads its tile (2.2 a feature) after a fixed
// start, and computes its share of the rows (35 a row as work of the chip; the
// wait for them is some 100 a row and wave).  The longest program bounds a
// wave from below.  Waves beyond those that fit at once take the SIMDs as they
// come free, and the last of them leave others idle for half their time.
static double launch_time(const ProgData& pd, int vi, int32_t tiles, int32_t tpw, int64_t blocks, const RowPlan& rows) {
    static constexpr double rate[5] = {0.0, 0.47, 0.60, 0.75, 1.0};
    const double W = core_variant_waves(vi), T = core_variant_t(vi), G = std::min<double>(blocks * W, pd.n_prog);
    const int K = std::min(4, core_variant_simd(vi));
    const double chunks = (tiles + tpw - 1) / tpw;
    const double fix = 190.0 / T + 2.2 * pd.n_load * tpw;
    const double mean = fix + tpw * (35.0 * rows.n() / W + rows.total / G);
    const double most = fix + tpw * (100.0 * std::ceil(rows.n() / W) + std::max(rows.total / G, 0.7 * rows.longest));
    const double waves = G * chunks, start = 1.8 * blocks * chunks / T;
    if (waves <= 1024.0 * K) {
        const int k = std::max(1, (int)((waves + 1023) / 1024));
        return start + std::max(k * mean / rate[k], most / rate[1]);
    }
    return start + waves * mean / (1024.0 * rate[K]) + 0.55 * most / rate[1];
}

static LaunchShape launch_shape(const ProgData& pd, int vi, int32_t tiles, const EvalOptions* opt, const RowPlan& rows,
                                int32_t force_G = 0) {
    // (a block counts as four waves)
    const int64_t W = core_variant_waves(vi);
    const int32_t forced = opt && opt->target_blocks > 0 ? opt->target_blocks : env_int("GP2D_TARGET_BLOCKS", 0);
    const int32_t target_blocks = (int32_t)((4 * (int64_t)(forced > 0 ? forced : 4096) + W - 1) / W);
    LaunchShape L;
    L.est = 0.0;
    int64_t G = base_groups(pd, vi, opt);
    if (force_G <= 0 && ((G + W - 1) / W) * tiles < target_blocks) {
        const int64_t most = (pd.n_prog + W - 1) / W;
        int64_t best = (G + W - 1) / W;
        if (forced > 0) {
            best = (target_blocks + tiles - 1) / tiles;
        } else if (rows.shape.tiles == tiles && rows.shape.base == G) {
            best = rows.shape.blocks;
            L.est = rows.shape.est;
        } else {
            const int64_t base = G;
            for (int64_t b = best; b <= most; b += std::max<int64_t>(1, b / 16)) {
                const double t = launch_time(pd, vi, tiles, 1, b, rows);
                if (L.est == 0.0 || t < L.est) L.est = t, best = b;
            }
            rows.shape = {tiles, base, best, L.est};
        }
        G = std::min<int64_t>(best * W, pd.n_prog);
    }
    if (force_G > 0) G = force_G;
    const int64_t quads = (G + W - 1) / W;
    int32_t tpw = opt && opt->tiles_per_wave > 0 ? opt->tiles_per_wave : env_int("GP2D_TILES_PER_WAVE", 0);
    if (tpw <= 0) {
        tpw = 1;
        while (tpw < 16 && quads * ((tiles + tpw - 1) / tpw) >= (1 << 24)) tpw *= 2;
    }
    L.G = (int32_t)G;
    L.tiles_per_wave = tpw;
    L.chunks = (int32_t)((tiles + tpw - 1) / tpw);
    return L;
}

// ---------------------------------------------------------------------------
// Kernel timing
// ---------------------------------------------------------------------------
static std::mutex g_tm_mu;
static bool g_tm_on = false;
static std::vector<std::pair<hipEvent_t, hipEvent_t>> g_tm_events;
static std::vector<std::pair<hipEvent_t, hipEvent_t>> g_tm_free;

hipError_t timed_launch_begin(hipStream_t s, int* slot) {
    *slot = -1;
    std::lock_guard<std::mutex> g(g_tm_mu);
    if (!g_tm_on) return hipSuccess;
    std::pair<hipEvent_t, hipEvent_t> ev;
    if (!g_tm_free.empty()) {
        ev = g_tm_free.back();
        g_tm_free.pop_back();
    } else {
        hipError_t e = hipEventCreate(&ev.first);
        if (e != hipSuccess) return e;
        e = hipEventCreate(&ev.second);
        if (e != hipSuccess) return e;
    }
    hipError_t e = hipEventRecord(ev.first, s);
    if (e != hipSuccess) return e;
    g_tm_events.push_back(ev);
    *slot = (int)g_tm_events.size() - 1;
    return hipSuccess;
}

hipError_t timed_launch_end(hipStream_t s, int slot) {
    if (slot < 0) return hipSuccess;
    std::lock_guard<std::mutex> g(g_tm_mu);
    return hipEventRecord(g_tm_events[slot].second, s);
}


static void plan_rows_for(const ProgData& pd, int vi, RowPlan& rows) {
    const int32_t W = core_variant_waves(vi);
    plan_rows(pd, vi, (base_groups(pd, vi, nullptr) + W - 1) / W, rows);
}

// Translate and upload a program set for variant vi, with the layout for G
// groups (0: none): with rows, and, if over some number of cases it is faster
// so, without them as well (translation_for says which an evaluation takes; a
// set is uploaded once).  The fewer the tiles, the less rows pay: in a sweep of
// 125 sets (5 to 5000 programs, 1 to 44 features) rows that were worth it over
// one tile were so over every number of tiles.  So only small sets hold both:
// 100 programs of up to 64 nodes, but not 300 of up to 200.  (For want of
// memory for both, the one with rows serves.)
static gp_status upload_set(const ProgData& pd, int vi, std::map<int, DevProgs>& dps, int32_t G, hipStream_t s, Workspace& w) {
    DevProgs& dp = dps[vi];
    plan_rows_for(pd, vi, dp.rows);
    const gp_status st = prepare_programs(pd, vi, dp, false, G, s, w, nullptr);
    if (st != GP_OK) return st;
    RowPlan none;
    no_rows(pd, vi, none);
    if (dp.rows.n() == none.n() ||
        launch_shape(pd, vi, 1, nullptr, dp.rows).est <= launch_shape(pd, vi, 1, nullptr, none).est)
        return GP_OK;
    DevProgs& plain = dps[vi + kNoRows];
    plain.rows = std::move(none);
    if (prepare_programs(pd, vi, plain, false, 0, s, w, nullptr) != GP_OK) {
        dps.erase(vi + kNoRows);
        clear_error();
    }
    return GP_OK;
}

// The translation that an evaluation takes, as a key of dps: with rows (vi) or without (vi + kNoRows).  Every block
// computes the rows of its tile, so with few tiles, and thus blocks of few programs, they can cost more than they save
// (1148 classification programs with 41 rows x 1000 cases: 29 us with them, 18 without; x 8000: 65 and 61; x 383000:
// 1.72 ms and 1.89): the shorter estimate is taken.  Where the tiles are enough for whole groups both estimates are
// zero, and the rows stay.
static int translation_for(const ProgData& pd, int vi, std::map<int, DevProgs>& dps, bool fresh, int32_t tiles,
                           const EvalOptions* opt) {
    DevProgs& dp = dps[vi];
    if (fresh) {
        plan_rows_for(pd, vi, dp.rows);
        if (dp.rows.n() == 0) return vi;
        RowPlan none;
        no_rows(pd, vi, none);
        if (launch_shape(pd, vi, tiles, opt, dp.rows).est > launch_shape(pd, vi, tiles, opt, none).est) dp.rows = std::move(none);
        return vi;
    }
    auto plain = dps.find(vi + kNoRows);
    if (plain == dps.end()) return vi;
    return launch_shape(pd, vi, tiles, opt, dp.rows).est <= launch_shape(pd, vi, tiles, opt, plain->second.rows).est
               ? vi : vi + kNoRows;
}

int default_variant(const ProgData& pd) {
    if (pd.variant >= 0) return pd.variant;
    return pick_core_variant(pd.n_load, pd.max_depth, pd.n_named ? (double)pd.n_transc / pd.n_named : 0.0,
                             pd.n_transc > 0, pd.opset == OPSET_BOOL, pd.form == FORM_TREE, true);
}

// The variant an evaluation without an explicit one launches: GP2D_VARIANT
// (tuning: a kernel variant index + 1) when that variant can hold the
// programs, else the default.
static int tuned_variant(const ProgData& pd) {
    const int32_t ev = env_int("GP2D_VARIANT", 0) - 1;
    if (ev >= 0 && ev < core_variants() && core_variant_fits(ev, pd))
        return ev;
    return default_variant(pd);
}

gp_status eval_core(const ProgData& pd, std::map<int, DevProgs>& dps, bool fresh, const float* X, int32_t n_feat,
                    int64_t N, const float* y, int32_t kind, void* out, hipStream_t s, Workspace* w,
                    const EvalOptions* opt, int64_t n_bits) {
    if (!X) return fail(GP_E_INVAL, "X is null");
    if (!out) return fail(GP_E_INVAL, "out is null");
    if (N < 1) return fail(GP_E_INVAL, "n_cases must be >= 1");
    if (kind < GP_FIT_SUM_ABS || kind > GP_FIT_CLASS_ERR) return fail(GP_E_INVAL, "unknown fitness kind %d", kind);
    if (kind != GP_OUT_CASES && !y) return fail(GP_E_INVAL, "y is null");
    if (n_feat < pd.n_feat) return fail(GP_E_INVAL, "case matrix has %d features, programs need %d", n_feat, pd.n_feat);
    if (pd.n_prog == 0) return GP_OK;
    if (pd.n_load > GP_MAX_FEAT)
        return fail(GP_E_INVAL, "programs read feature %d; at most %d features are supported", pd.n_load - 1, GP_MAX_FEAT);
    const bool boolean = pd.opset == OPSET_BOOL;
    if (boolean != (n_bits > 0)) return fail(GP_E_INVAL, "internal: Boolean programs need a bit count");
    if (boolean && kind != GP_FIT_HITS && kind != GP_OUT_CASES)
        return fail(GP_E_INVAL, "Boolean programs take GP_FIT_HITS or GP_OUT_CASES, not kind %d", kind);
    const int vi = opt && opt->variant >= 0 ? opt->variant
                   : opt && opt->no_alloc   ? default_variant(pd)
                                            : tuned_variant(pd);
    if (vi < 0 || vi >= core_variants())
        return fail(GP_E_DEPTH, "no kernel variant for %d features and depth %d", pd.n_load, pd.max_depth);
    if (!core_variant_fits(vi, pd))
        return fail(GP_E_INVAL, "variant %d cannot hold these programs", vi);
    const bool no_alloc = opt && opt->no_alloc;
    gp_status st;
    if (no_alloc) {
        if (!core_is_ready(vi)) return fail(GP_E_DEVICE, "kernel variant %d is not set up on this device", vi);
    } else if ((st = core_ready(vi, s)) != GP_OK) {
        return st;
    }
    const int T = core_variant_t(vi);
    const int64_t tiles64 = (N + 64LL * T - 1) / (64LL * T);
    if (tiles64 > (1LL << 30)) return fail(GP_E_INVAL, "n_cases too large");
    const int32_t tiles = (int32_t)tiles64;
    if (!no_alloc && !w) return fail(GP_E_INVAL, "internal: no workspace");
    // (a set is uploaded when it is created, and here for another kernel than its own)
    if (!no_alloc && !fresh && !dps[vi].uploaded && (st = upload_set(pd, vi, dps, 0, s, *w)) != GP_OK) return st;
    const int key = no_alloc ? vi : translation_for(pd, vi, dps, fresh, tiles, opt);
    auto dit = dps.find(key);
    if (no_alloc && dit == dps.end()) return fail(GP_E_INVAL, "programs are not on the device for variant %d", vi);
    DevProgs& dp = no_alloc ? dit->second : dps[key];
    const LaunchShape L = launch_shape(pd, vi, tiles, opt, dp.rows, no_alloc ? opt->groups : 0);
    const int32_t G = L.G;
    // (rows are those of the one tile that a block's waves share)
    const int32_t same_group = dp.rows.n() == 0 && env_int("GP2D_SAME_GROUP", 0) > 0 ? 1 : 0;
    const int32_t W = core_variant_waves(vi);
    // Few tiles: a block takes a group on all of them and finishes its fitness values, without the reduction launch
    // (100 trees x 1024 cases: 10.6 -> 7.4 us of host time a call, and 1 us less from call to result).
    const std::vector<EvalSegment>* seg = opt ? opt->segments : nullptr;
    const bool direct = kind != GP_OUT_CASES && !seg && dp.rows.n() == 0 && !same_group && tiles <= W && L.tiles_per_wave == 1;
    const int64_t units = direct ? (int64_t)G : same_group ? (int64_t)G * ((L.chunks + W - 1) / W) : (int64_t)L.chunks * ((G + W - 1) / W);
    if (units > (1LL << 31) - 64) return fail(GP_E_INVAL, "too many work units");
    const int64_t n_blocks = (N + 255) / 256;
    const size_t part_bytes = kind == GP_OUT_CASES ? 0 : (size_t)n_blocks * pd.n_prog * sizeof(double);
    const uint32_t* goff;
    double* partials = nullptr;
    if (no_alloc) {
        auto git = dp.groups_by_G.find(G);
        if (!dp.uploaded || git == dp.groups_by_G.end() || !dp.ready)
            return fail(GP_E_INVAL, "programs or their group layout are not on the device");
        if (part_bytes > opt->partials_bytes)
            return fail(GP_E_NOMEM, "%lld programs x %lld blocks of 256 cases need %zu bytes of partial sums; "
                        "this entry point has %zu", (long long)pd.n_prog, (long long)n_blocks, part_bytes,
                        opt->partials_bytes);
        if ((st = wait_for_upload(dp, s)) != GP_OK) return st;
        goff = (const uint32_t*)git->second.p;
        partials = opt->partials;
    } else {
        if ((st = prepare_programs(pd, vi, dp, fresh, G, s, *w, &goff)) != GP_OK) return st;
        if (part_bytes && (st = w->partials.reserve(part_bytes)) != GP_OK) return st;
        partials = (double*)w->partials.p;
    }
    CoreArgs a;
    memset(&a, 0, sizeof a);
    a.code = (const uint32_t*)dp.code.p;
    a.group_off = goff;
    a.X = X;
    a.y = kind == GP_OUT_CASES ? nullptr : y;
    a.N = N;
    a.n_load = std::min(pd.n_load, core_variant_nf(vi));
    a.kind = kind;
    a.tiles = tiles;
    a.n_units = (int32_t)units;
    a.tiles_per_wave = L.tiles_per_wave;
    a.chunks = L.chunks;
    a.prefetch = code_prefetch();
    a.n_groups = G;
    a.same_group = same_group;
    a.n_rows = dp.rows.n();
    a.row_off = goff + G + 1;
    a.direct = direct ? tiles : 0;
    a.group_prog = a.row_off + W + 1;
    a.order = a.group_prog + G + 1;
    a.out = out;
    a.n_bits = n_bits;
    a.partials = partials;
    a.cases_out = kind == GP_OUT_CASES ? (float*)out : nullptr;
    uint32_t blocks = (uint32_t)units;
    blocks = (blocks + 7u) & ~7u;
    int slot = -1;
    hipError_t e = no_alloc ? hipSuccess : timed_launch_begin(s, &slot);
    if (e == hipSuccess) e = core_launch(vi, a, blocks, s);
    if (e == hipSuccess) e = timed_launch_end(s, slot);
    if (e != hipSuccess) return fail(GP_E_DEVICE, "evaluation launch: %s", hipGetErrorString(e));
    if (kind == GP_OUT_CASES || direct) return GP_OK;
    ReduceArgs r;
    memset(&r, 0, sizeof r);
    r.partials = partials;
    r.part_base = 0;
    r.n_prog = pd.n_prog;
    r.N = N;
    r.out = out;
    r.blocks = (int32_t)n_blocks;
    r.kind = kind;
    const EvalSegment all{0, pd.n_prog, out};
    for (size_t k = 0; k < (seg ? seg->size() : 1); k++) {
        const EvalSegment& g = seg ? (*seg)[k] : all;
        r.part_base = (uint64_t)g.first * (uint64_t)n_blocks;
        r.n_prog = g.n_prog;
        r.out = g.out;
        e = core_reduce_one(r, s);
        if (e != hipSuccess) return fail(GP_E_DEVICE, "reduction launch: %s", hipGetErrorString(e));
    }
    return GP_OK;
}

}  // namespace gpx

// ===========================================================================
// C ABI
// ===========================================================================
using namespace gpx;

struct gp_progset {
    ProgData pd;
    std::map<int, DevProgs> dps;   // translated per core variant
    int32_t groups = 0;            // the group layout uploaded at creation
    std::mutex mu;
};

// Evaluate a program set with nothing allocated or uploaded (see runtime.h).
gp_status gpx::progset_eval_no_alloc(gp_progset* ps, const float* X, int32_t n_feat, int64_t n_cases, const float* y,
                                int32_t kind, void* out, hipStream_t s, double* partials, size_t partials_bytes) {
    if (!ps) return fail(GP_E_INVAL, "ps is null");
    std::lock_guard<std::mutex> g(ps->mu);
    EvalOptions o;
    o.no_alloc = true;
    o.groups = ps->groups;
    o.partials = partials;
    o.partials_bytes = partials_bytes;
    if (ps->pd.opset == OPSET_BOOL) {
        if (n_cases < 1) return fail(GP_E_INVAL, "n_cases must be >= 1");
        if (n_cases > 0x7FFFFFFF) return fail(GP_E_INVAL, "n_cases above 2^31 - 1 (hit counts are int32)");
        return eval_core(ps->pd, ps->dps, false, X, n_feat, (n_cases + 31) / 32, y, kind, out, s, nullptr, &o,
                         n_cases);
    }
    return eval_core(ps->pd, ps->dps, false, X, n_feat, n_cases, y, kind, out, s, nullptr, &o);
}

extern "C" {

const char* gp_last_error(void) { return last_error(); }

const char* gp_version(void) { return "gp2d 0.1 (gfx950)"; }

gp_status gp_eval_tree(const int32_t* tok, const float* cst, const int64_t* off, int32_t n_prog,
                       const float* X, int32_t n_feat, int64_t n_cases, const float* y, int32_t kind,
                       void* out, void* stream) {
    clear_error();
    ProgData pd;
    gp_status st = build_tree(tok, cst, off, n_prog, n_feat, pd);
    if (st != GP_OK || n_prog == 0) return st;
    hipStream_t s = (hipStream_t)stream;
    Workspace& w = workspace(s);
    std::lock_guard<std::mutex> g(w.mu);
    return eval_core(pd, w.oneshot, true, X, n_feat, n_cases, y, kind, out, s, &w, nullptr);
}

gp_status gp_eval_linear(const uint32_t* code, const int64_t* off, const float* cst, const int64_t* cst_off,
                         int32_t n_prog, int32_t n_reg, const float* X, int32_t n_feat, int64_t n_cases,
                         const float* y, int32_t kind, void* out, void* stream) {
    clear_error();
    ProgData pd;
    gp_status st = build_linear(code, off, cst, cst_off, n_prog, n_reg, n_feat, pd);
    if (st != GP_OK || n_prog == 0) return st;
    hipStream_t s = (hipStream_t)stream;
    Workspace& w = workspace(s);
    std::lock_guard<std::mutex> g(w.mu);
    return eval_core(pd, w.oneshot, true, X, n_feat, n_cases, y, kind, out, s, &w, nullptr);
}

gp_status gp_eval_bool(const int32_t* tok, const int64_t* off, int32_t n_prog, const uint32_t* X, int32_t n_feat,
                       int64_t n_cases, const uint32_t* y, int32_t kind, void* out, void* stream) {
    clear_error();
    if (n_cases < 1) return fail(GP_E_INVAL, "n_cases must be >= 1");
    if (n_cases > 0x7FFFFFFF) return fail(GP_E_INVAL, "n_cases above 2^31 - 1 (hit counts are int32)");
    if (kind != GP_FIT_HITS && kind != GP_OUT_CASES)
        return fail(GP_E_INVAL, "Boolean programs take GP_FIT_HITS or GP_OUT_CASES, not kind %d", kind);
    ProgData pd;
    gp_status st = build_tree(tok, nullptr, off, n_prog, n_feat, pd, OPSET_BOOL);
    if (st != GP_OK || n_prog == 0) return st;
    hipStream_t s = (hipStream_t)stream;
    Workspace& w = workspace(s);
    std::lock_guard<std::mutex> g(w.mu);
    // one slot per 32-bit word: the kernel sees n_words "cases"
    const int64_t n_words = (n_cases + 31) / 32;
    return eval_core(pd, w.oneshot, true, (const float*)X, n_feat, n_words, (const float*)y, kind, out, s, &w,
                     nullptr, n_cases);
}

static gp_status progset_finish(ProgData&& pd, void* stream, gp_progset** ps) {
    // Translate the programs for the kernel variant evaluations will use and
    // upload them on `stream` now; an evaluation on any stream waits for it.
    std::unique_ptr<gp_progset> p(new gp_progset());
    p->pd = std::move(pd);
    if (p->pd.n_prog > 0) {
        const int vi = p->pd.variant = default_variant(p->pd);
        if (vi < 0) return fail(GP_E_DEPTH, "no kernel variant for %d features and depth %d", p->pd.n_load,
                                p->pd.max_depth);
        hipStream_t s = (hipStream_t)stream;
        gp_status st;
        if ((st = core_ready(vi, s)) != GP_OK) return st;
        Workspace& w = workspace(s);
        std::lock_guard<std::mutex> g(w.mu);
        p->groups = base_groups(p->pd, vi, nullptr);
        if ((st = upload_set(p->pd, vi, p->dps, p->groups, s, w)) != GP_OK) return st;
    }
    *ps = p.release();
    return GP_OK;
}

gp_status gp_progset_tree(const int32_t* tok, const float* cst, const int64_t* off, int32_t n_prog,
                          int32_t n_feat, void* stream, gp_progset** ps) {
    clear_error();
    if (!ps) return fail(GP_E_INVAL, "ps is null");
    ProgData pd;
    gp_status st = build_tree(tok, cst, off, n_prog, n_feat, pd);
    if (st != GP_OK) return st;
    return progset_finish(std::move(pd), stream, ps);
}

gp_status gp_progset_bool(const int32_t* tok, const int64_t* off, int32_t n_prog, int32_t n_feat, void* stream,
                          gp_progset** ps) {
    clear_error();
    if (!ps) return fail(GP_E_INVAL, "ps is null");
    ProgData pd;
    gp_status st = build_tree(tok, nullptr, off, n_prog, n_feat, pd, OPSET_BOOL);
    if (st != GP_OK) return st;
    return progset_finish(std::move(pd), stream, ps);
}

gp_status gp_progset_linear(const uint32_t* code, const int64_t* off, const float* cst,
                            const int64_t* cst_off, int32_t n_prog, int32_t n_reg, int32_t n_feat,
                            void* stream, gp_progset** ps) {
    clear_error();
    if (!ps) return fail(GP_E_INVAL, "ps is null");
    ProgData pd;
    gp_status st = build_linear(code, off, cst, cst_off, n_prog, n_reg, n_feat, pd);
    if (st != GP_OK) return st;
    return progset_finish(std::move(pd), stream, ps);
}

gp_status gp_progset_eval(gp_progset* ps, const float* X, int32_t n_feat, int64_t n_cases, const float* y,
                          int32_t kind, void* out, void* stream) {
    clear_error();
    if (!ps) return fail(GP_E_INVAL, "ps is null");
    hipStream_t s = (hipStream_t)stream;
    Workspace& w = workspace(s);
    std::lock_guard<std::mutex> g(w.mu);
    std::lock_guard<std::mutex> g2(ps->mu);
    if (ps->pd.opset == OPSET_BOOL) {
        // Boolean set: X and y are 32-bit words, n_cases counts bits
        if (n_cases < 1) return fail(GP_E_INVAL, "n_cases must be >= 1");
        if (n_cases > 0x7FFFFFFF) return fail(GP_E_INVAL, "n_cases above 2^31 - 1 (hit counts are int32)");
        return eval_core(ps->pd, ps->dps, false, X, n_feat, (n_cases + 31) / 32, y, kind, out, s, &w, nullptr,
                         n_cases);
    }
    return eval_core(ps->pd, ps->dps, false, X, n_feat, n_cases, y, kind, out, s, &w, nullptr);
}

gp_status gp_progset_get_info(const gp_progset* ps, gp_progset_info* info) {
    clear_error();
    if (!ps || !info) return fail(GP_E_INVAL, "null argument");
    info->n_prog = ps->pd.n_prog;
    info->form = ps->pd.form;
    info->n_feat = ps->pd.n_feat;
    info->max_depth = ps->pd.max_depth;
    info->n_instr = ps->pd.n_named;
    info->n_gpop = ps->pd.n_gpop;
    info->variant = tuned_variant(ps->pd);
    info->pad = 0;
    return GP_OK;
}

gp_status gp_progset_destroy(gp_progset* ps) {
    clear_error();
    if (!ps) return GP_OK;
    for (auto& kv : ps->dps) kv.second.release();
    delete ps;
    return GP_OK;
}

static gp_status core_lower_common(ProgData& pd, int32_t variant, uint64_t table_base, uint32_t* words,
                                   int64_t max_words, int64_t* prog_off, int64_t* n_words) {
    RawWords code;
    std::vector<DevProg> progs;
    gp_status st = core_translate_at(pd, variant, table_base, code, progs);
    if (st != GP_OK) return st;
    if (n_words) *n_words = (int64_t)code.size();
    if (words) {
        if (max_words < (int64_t)code.size()) return fail(GP_E_INVAL, "words buffer too small");
        memcpy(words, code.data(), code.size() * 4);
    }
    if (prog_off) {
        for (int32_t p = 0; p < pd.n_prog; p++) prog_off[p] = progs[p].code_off;
        prog_off[pd.n_prog] = (int64_t)code.size();
    }
    return GP_OK;
}

gp_status gp_core_lower_tree(const int32_t* tok, const float* cst, const int64_t* off, int32_t n_prog, int32_t n_feat,
                             int32_t variant, uint64_t table_base, uint32_t* words, int64_t max_words,
                             int64_t* prog_off, int64_t* n_words) {
    clear_error();
    if (variant < 0 || variant >= core_variants()) return fail(GP_E_INVAL, "variant %d does not exist", variant);
    // a Boolean kernel takes trees of the Boolean function set
    ProgData pd;
    gp_status st = build_tree(tok, cst, off, n_prog, n_feat, pd, core_variant_bool(variant) ? OPSET_BOOL : OPSET_REAL);
    if (st != GP_OK) return st;
    return core_lower_common(pd, variant, table_base, words, max_words, prog_off, n_words);
}

gp_status gp_core_lower_linear(const uint32_t* code, const int64_t* off, const float* cst, const int64_t* cst_off,
                               int32_t n_prog, int32_t n_reg, int32_t n_feat, int32_t variant, uint64_t table_base,
                               uint32_t* words, int64_t max_words, int64_t* prog_off, int64_t* n_words) {
    clear_error();
    if (variant < 0 || variant >= core_variants()) return fail(GP_E_INVAL, "variant %d does not exist", variant);
    if (core_variant_trees_only(variant)) return fail(GP_E_INVAL, "variant %d runs trees only", variant);
    ProgData pd;
    gp_status st = build_linear(code, off, cst, cst_off, n_prog, n_reg, n_feat, pd);
    if (st != GP_OK) return st;
    return core_lower_common(pd, variant, table_base, words, max_words, prog_off, n_words);
}

gp_status gp_timing_enable(int on) {
    clear_error();
    std::lock_guard<std::mutex> g(g_tm_mu);
    g_tm_on = on != 0;
    return GP_OK;
}

gp_status gp_timing_read(int64_t* launches, double* total_ms, int reset) {
    clear_error();
    std::lock_guard<std::mutex> g(g_tm_mu);
    double ms = 0.0;
    for (auto& ev : g_tm_events) {
        hipError_t e = hipEventSynchronize(ev.second);
        if (e != hipSuccess) return fail(GP_E_DEVICE, "hipEventSynchronize: %s", hipGetErrorString(e));
        float t = 0.0f;
        e = hipEventElapsedTime(&t, ev.first, ev.second);
        if (e != hipSuccess) return fail(GP_E_DEVICE, "hipEventElapsedTime: %s", hipGetErrorString(e));
        ms += t;
    }
    if (launches) *launches = (int64_t)g_tm_events.size();
    if (total_ms) *total_ms = ms;
    if (reset) {
        g_tm_free.insert(g_tm_free.end(), g_tm_events.begin(), g_tm_events.end());
        g_tm_events.clear();
    }
    return GP_OK;
}

gp_status gp_lower_tree(const int32_t* tok, const float* cst, int64_t n, int32_t n_feat, uint32_t* words,
                        int64_t max_words, gp_lower_stats* stats) {
    clear_error();
    if (!tok || !cst) return fail(GP_E_INVAL, "null program");
    if (n_feat < 1) return fail(GP_E_INVAL, "n_feat < 1");
    if (n > GP_MAX_LEN) return fail(GP_E_DEPTH, "program of %lld nodes exceeds %d", (long long)n, GP_MAX_LEN);
    std::vector<uint32_t> buf(2 * (size_t)std::max<int64_t>(n, 1));
    TreeLowering st;
    char err[256];
    int rc = lower_tree(tok, cst, n, n_feat, buf.data(), &st, err);
    if (rc != GP_OK) return fail((gp_status)rc, "%s", err);
    if (words) {
        if (max_words < 2 * (int64_t)st.n_instr) return fail(GP_E_INVAL, "words buffer too small");
        memcpy(words, buf.data(), sizeof(uint32_t) * 2 * (size_t)st.n_instr);
    }
    if (stats) {
        stats->n_nodes = st.n_nodes;
        stats->n_instr = st.n_instr;
        stats->max_depth = st.max_depth;
        stats->stack_fetches = st.stack_fetches;
        stats->n_values = st.n_values;
        stats->n_reversed = st.n_reversed;
    }
    return GP_OK;
}

}  // extern "C"
