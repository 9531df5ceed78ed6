// Batched evaluation: several program populations (tree and linear) over
// several resident case matrices, large sets of alike ones as one population,
// the others in one persistent launch over a table of units; and the
// autotuner that picks kernel variant, unit size and schedule of such a launch
// for a batch shape.
#include <hip/hip_runtime_api.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <functional>
#include <map>
#include <mutex>
#include <numeric>
#include <string>
#include <tuple>
#include <vector>

#include "../../include/gp.h"
#include "batch.h"
#include "core_host.h"
#include "core_kernels.h"
#include "runtime.h"

namespace gpx {

static int device_cus() {
    static int cus = 0;
    if (cus == 0) {
        int dev = 0;
        hipDeviceProp_t prop;
        if (hipGetDevice(&dev) == hipSuccess && hipGetDeviceProperties(&prop, dev) == hipSuccess)
            cus = prop.multiProcessorCount;
        if (cus <= 0) cus = 256;
    }
    return cus;
}

static double transc_fraction(const std::vector<BatchJobRef>& jobs) {
    int64_t e = 0, n = 0;
    for (const BatchJobRef& j : jobs) {
        e += j.pd->n_transc;
        n += j.pd->n_named;
    }
    return n ? (double)e / (double)n : 0.0;
}

// Whether a configuration's kernel can run the jobs.
static gp_status check_config(const std::vector<BatchJobRef>& jobs, const gp_batch_config& cfg) {
    int n_load = 1, depth = 0;
    bool any_transc = false;
    for (const BatchJobRef& j : jobs) {
        n_load = std::max(n_load, j.pd->n_load);
        depth = std::max(depth, j.pd->max_depth);
        any_transc = any_transc || j.pd->n_transc > 0;
    }
    const int vi = cfg.variant;
    if (vi < 0 || vi >= core_variants()) return fail(GP_E_INVAL, "kernel variant %d does not exist", vi);
    if (core_variant_nf(vi) < n_load || core_variant_d(vi) < depth)
        return fail(GP_E_INVAL, "variant %d (%d features, depth %d) cannot hold %d features / depth %d", vi,
                    core_variant_nf(vi), core_variant_d(vi), n_load, depth);
    if (core_variant_arith(vi) && any_transc)
        return fail(GP_E_INVAL, "variant %d has no sin/cos/exp/log code", vi);
    if (core_variant_bool(vi)) return fail(GP_E_INVAL, "variant %d is a Boolean kernel", vi);
    if (core_variant_trees_only(vi))
        for (const BatchJobRef& j : jobs)
            if (j.pd->form != FORM_TREE) return fail(GP_E_INVAL, "variant %d runs trees only", vi);
    return GP_OK;
}

gp_status plan_batch(const std::vector<BatchJobRef>& jobs, const std::vector<gp_dataset>& ds,
                     const gp_batch_config& cfg, BatchPlan& plan) {
    plan = BatchPlan();
    const gp_status fits = check_config(jobs, cfg);
    if (fits != GP_OK) return fits;
    const int vi = cfg.variant, vt = core_variant_t(vi);
    plan.vi = vi;
    const int32_t unit_prog = std::max(1, cfg.unit_programs);
    int64_t n_prog = 0;
    for (const BatchJobRef& j : jobs) n_prog += j.pd->n_prog;
    if (n_prog > 0x7FFFFFFFll) return fail(GP_E_INVAL, "batch too large");
    uint64_t part_base = 0;
    std::vector<std::pair<double, UnitDesc>> units;
    for (size_t ji = 0; ji < jobs.size(); ji++) {
        const BatchJobRef& j = jobs[ji];
        const ProgData& pd = *j.pd;
        const gp_dataset& d = ds[j.ds];
        const int64_t N = d.n_cases;
        const int64_t blocks = (N + 255) / 256;
        const int64_t tiles = (N + 64LL * vt - 1) / (64LL * vt);
        RawWords jcode;
        std::vector<DevProg> jprogs;
        // programs of this job by falling cost, in G groups of about equal cost
        std::vector<uint32_t> order, goff;
        std::vector<int64_t> rec((size_t)pd.n_prog + 1);
        cost_order(pd.cost, order);
        gp_status st = core_translate(pd, vi, order.data(), nullptr, jcode, jprogs);
        if (st != GP_OK) return st;
        if ((plan.code.size() + jcode.size()) * 4 > 0xFFFFFFF0ull) return fail(GP_E_INVAL, "batch code exceeds 4 GiB");
        const int64_t base = (int64_t)plan.code.size() / 4;
        plan.code.insert(plan.code.end(), jcode.begin(), jcode.end());
        for (int32_t i = 0; i < pd.n_prog; i++) rec[i] = base + jprogs[order[i]].code_off / 4;
        rec[pd.n_prog] = rec[pd.n_prog - 1] + jprogs[order[pd.n_prog - 1]].len;
        const int32_t G = std::max<int32_t>(1, (pd.n_prog + unit_prog - 1) / unit_prog);
        cut_groups(pd.cost, order, rec, G, goff);
        std::vector<double> gcost(G, 0.0);
        for (int32_t g = 0, i = 0; g < G; g++)
            for (; i < pd.n_prog && rec[i] < goff[g + 1]; i++) gcost[g] += pd.cost[order[i]];
        for (int64_t t = 0; t < tiles; t++) {
            for (int32_t g = 0; g < G; g++) {
                if (goff[g] == goff[g + 1]) continue;
                UnitDesc u{(uint32_t)ji, (uint32_t)t, goff[g], goff[g + 1]};
                // every slot of a tile is interpreted, ragged or not; add the tile load
                units.push_back({gcost[g] + 8.0 * pd.n_load, u});
            }
        }
        JobDesc jd;
        memset(&jd, 0, sizeof jd);
        jd.ds = j.ds;
        jd.kind = j.kind;
        jd.n_load = pd.n_load;
        jd.part_base = part_base;
        plan.jobs.push_back(jd);
        ReduceArgs r;
        memset(&r, 0, sizeof r);
        r.part_base = part_base;
        r.n_prog = pd.n_prog;
        r.N = N;
        r.out = j.out;
        r.blocks = (int32_t)blocks;
        r.kind = j.kind;
        plan.reduce.push_back(r);
        plan.max_prog = std::max<int64_t>(plan.max_prog, pd.n_prog);
        plan.gpop += pd.n_gpop * N;
        part_base += (uint64_t)blocks * (uint64_t)pd.n_prog;
    }
    if (units.size() > 0x7FFFFFF0ull) return fail(GP_E_INVAL, "batch has too many work units");
    if (cfg.persistent)
        std::stable_sort(units.begin(), units.end(),
                         [](const std::pair<double, UnitDesc>& a, const std::pair<double, UnitDesc>& b) {
                             return a.first > b.first;
                         });
    plan.units.reserve(units.size());
    for (auto& u : units) plan.units.push_back(u.second);
    plan.partial_doubles = (int64_t)part_base;
    plan.persistent = cfg.persistent != 0;
    for (const gp_dataset& d : ds) {
        DatasetDesc dd;
        dd.X = d.X;
        dd.y = d.y;
        dd.N = d.n_cases;
        plan.datasets.push_back(dd);
    }
    return GP_OK;
}

size_t plan_device_bytes(const BatchPlan& p) {
    return p.code.size() * 4 + p.units.size() * sizeof(UnitDesc) + p.jobs.size() * sizeof(JobDesc) +
           p.datasets.size() * sizeof(DatasetDesc) + p.reduce.size() * sizeof(ReduceArgs) +
           (size_t)p.partial_doubles * sizeof(double) + 4096;
}

gp_status upload_plan(BatchPlan& p, BatchScratch& sc, hipStream_t s) {
    gp_status st;
    if ((st = sc.code.reserve(std::max<size_t>(4, p.code.size() * 4))) != GP_OK) return st;
    if ((st = sc.units.reserve(std::max<size_t>(1, p.units.size()) * sizeof(UnitDesc))) != GP_OK) return st;
    if ((st = sc.jobs.reserve(std::max<size_t>(1, p.jobs.size()) * sizeof(JobDesc))) != GP_OK) return st;
    if ((st = sc.datasets.reserve(std::max<size_t>(1, p.datasets.size()) * sizeof(DatasetDesc))) != GP_OK) return st;
    if ((st = sc.reduce.reserve(std::max<size_t>(1, p.reduce.size()) * sizeof(ReduceArgs))) != GP_OK) return st;
    if ((st = sc.partials.reserve(std::max<size_t>(1, (size_t)p.partial_doubles) * sizeof(double))) != GP_OK) return st;
    if ((st = sc.counter.reserve(256)) != GP_OK) return st;
    for (ReduceArgs& r : p.reduce) r.partials = (const double*)sc.partials.p;
    const size_t total = plan_device_bytes(p) - (size_t)p.partial_doubles * sizeof(double) + 8 * 256;
    if ((st = sc.staging.begin(total)) != GP_OK) return st;
    if ((st = sc.staging.put(p.code.data(), p.code.size() * 4, sc.code.p, s)) != GP_OK) return st;
    if ((st = sc.staging.put(p.units.data(), p.units.size() * sizeof(UnitDesc), sc.units.p, s)) != GP_OK) return st;
    if ((st = sc.staging.put(p.jobs.data(), p.jobs.size() * sizeof(JobDesc), sc.jobs.p, s)) != GP_OK) return st;
    if ((st = sc.staging.put(p.datasets.data(), p.datasets.size() * sizeof(DatasetDesc), sc.datasets.p, s)) != GP_OK)
        return st;
    if ((st = sc.staging.put(p.reduce.data(), p.reduce.size() * sizeof(ReduceArgs), sc.reduce.p, s)) != GP_OK)
        return st;
    return sc.staging.end(s);
}

gp_status launch_plan(const BatchPlan& p, BatchScratch& sc, hipStream_t s) {
    if (p.units.empty()) return GP_OK;
    CoreArgs a;
    memset(&a, 0, sizeof a);
    a.code = (const uint32_t*)sc.code.p;
    a.units = (const UnitDesc*)sc.units.p;
    a.jobs = (const JobDesc*)sc.jobs.p;
    a.datasets = (const DatasetDesc*)sc.datasets.p;
    a.partials = (double*)sc.partials.p;
    a.counter = (uint32_t*)sc.counter.p;
    a.n_units = (int32_t)p.units.size();
    a.persistent = p.persistent ? 1 : 0;
    a.prefetch = code_prefetch();
    const size_t waves = (size_t)core_variant_waves(p.vi);
    const uint32_t grid = p.persistent ? (uint32_t)(device_cus() * core_blocks_per_cu(p.vi))
                                       : (uint32_t)((p.units.size() + waves - 1) / waves);
    int slot;
    hipError_t e = hipSuccess;
    if (p.persistent) e = core_zero_counter(a.counter, s);
    if (e == hipSuccess) e = timed_launch_begin(s, &slot);
    if (e == hipSuccess) e = core_launch(p.vi, a, grid, s);
    if (e == hipSuccess) e = timed_launch_end(s, slot);
    if (e != hipSuccess) return fail(GP_E_DEVICE, "batch launch: %s", hipGetErrorString(e));
    e = core_reduce_jobs((const ReduceArgs*)sc.reduce.p, (int32_t)p.reduce.size(), p.max_prog, s);
    if (e != hipSuccess) return fail(GP_E_DEVICE, "batch reduction launch: %s", hipGetErrorString(e));
    return GP_OK;
}

// ---------------------------------------------------------------------------
// Autotuning
// ---------------------------------------------------------------------------
// What is stored for a shape.  In the file the kernel goes by its name: it may
// have been written by another release, with kernels that this one has not.
struct Tuned {
    std::string kernel;
    int unit_programs, persistent;
    int variant;                   // of that name, -1: none
    Tuned() = default;
    Tuned(const std::string& name, int unit, int pers)
        : kernel(name), unit_programs(unit), persistent(pers), variant(core_variant_named(name)) {}
};
static std::mutex g_tune_mu;
static std::map<std::string, Tuned> g_tune_cache;
static bool g_tune_loaded = false;

static const char* tune_cache_path() { return getenv("GP2D_TUNE_CACHE"); }

static void tune_load_locked() {
    if (g_tune_loaded) return;
    g_tune_loaded = true;
    const char* path = tune_cache_path();
    if (!path) return;
    FILE* f = fopen(path, "r");
    if (!f) return;
    // one entry per line: "key": ["kernel", unit_programs, persistent], or, in files of earlier releases, the kernel's
    // number
    char line[4096];
    while (fgets(line, sizeof line, f)) {
        char* q1 = strchr(line, '"');
        if (!q1) continue;
        char* q2 = strchr(q1 + 1, '"');
        if (!q2) continue;
        std::string key(q1 + 1, q2);
        char name[64];
        int vi, unit, pers;
        if (sscanf(q2 + 1, " : [ \"%63[^\"]\" , %d , %d ]", name, &unit, &pers) == 3)
            g_tune_cache[key] = Tuned(name, unit, pers);
        else if (sscanf(q2 + 1, " : [ %d , %d , %d ]", &vi, &unit, &pers) == 3)
            g_tune_cache[key] = Tuned(vi >= 0 && vi < core_variants() ? core_variant_name(vi) : std::to_string(vi), unit, pers);
    }
    fclose(f);
}

static void tune_save_locked() {
    const char* path = tune_cache_path();
    if (!path) return;
    std::string tmp = std::string(path) + ".tmp";
    FILE* f = fopen(tmp.c_str(), "w");
    if (!f) return;
    fprintf(f, "{\n");
    size_t i = 0;
    for (auto& kv : g_tune_cache) {
        fprintf(f, "\"%s\": [\"%s\", %d, %d]%s\n", kv.first.c_str(), kv.second.kernel.c_str(), kv.second.unit_programs,
                kv.second.persistent, ++i < g_tune_cache.size() ? "," : "");
    }
    fprintf(f, "}\n");
    fclose(f);
    rename(tmp.c_str(), path);
}

// Shape signature of a batch: what the best configuration depends on.
static std::string batch_key(const std::vector<BatchJobRef>& jobs, const std::vector<gp_dataset>& ds) {
    std::string k;
    char buf[128];
    for (const gp_dataset& d : ds) {
        snprintf(buf, sizeof buf, "d%lldx%d;", (long long)d.n_cases, d.n_feat);
        k += buf;
    }
    for (const BatchJobRef& j : jobs) {
        // program counts and mean lengths rounded to powers of two
        const int64_t P = j.pd->n_prog;
        const int64_t mean = P ? j.pd->n_named / P : 0;
        int lp = 0, lm = 0;
        while ((1LL << lp) < P) lp++;
        while ((1LL << lm) < mean) lm++;
        snprintf(buf, sizeof buf, "j%d,%d,%d,%d,%d,%d;", j.pd->form, j.ds, lp, lm, j.pd->n_load, j.pd->max_depth);
        k += buf;
    }
    return k;
}

static gp_status time_config(const std::vector<BatchJobRef>& jobs, const std::vector<gp_dataset>& ds,
                             const gp_batch_config& c, int reps, BatchScratch& sc, hipStream_t s, double* ms) {
    gp_status st = core_ready(c.variant, s);
    if (st != GP_OK) return st;
    BatchPlan plan;
    st = plan_batch(jobs, ds, c, plan);
    if (st != GP_OK) return st;
    if ((st = upload_plan(plan, sc, s)) != GP_OK) return st;
    if ((st = launch_plan(plan, sc, s)) != GP_OK) return st;  // warm-up
    hipEvent_t e0, e1;
    if (hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess)
        return fail(GP_E_DEVICE, "hipEventCreate failed");
    std::vector<float> t;
    for (int r = 0; r < reps; r++) {
        hipError_t e = hipEventRecord(e0, s);
        st = launch_plan(plan, sc, s);
        if (e == hipSuccess) e = hipEventRecord(e1, s);
        if (st != GP_OK) break;
        if (e == hipSuccess) e = hipEventSynchronize(e1);
        if (e != hipSuccess) {
            st = fail(GP_E_DEVICE, "hipEventSynchronize: %s", hipGetErrorString(e));
            break;
        }
        float x = 0;
        e = hipEventElapsedTime(&x, e0, e1);
        if (e != hipSuccess) {
            st = fail(GP_E_DEVICE, "hipEventElapsedTime: %s", hipGetErrorString(e));
            break;
        }
        t.push_back(x);
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (st != GP_OK) return st;
    std::sort(t.begin(), t.end());
    *ms = t[t.size() / 2];
    return GP_OK;
}

gp_status tune_batch(const std::vector<BatchJobRef>& jobs, const std::vector<gp_dataset>& ds, int reps,
                     BatchScratch& sc, hipStream_t s, gp_batch_config* best, double* best_ms) {
    int n_load = 1, depth = 0;
    bool any_transc = false;
    for (const BatchJobRef& j : jobs) {
        n_load = std::max(n_load, j.pd->n_load);
        depth = std::max(depth, j.pd->max_depth);
        any_transc = any_transc || j.pd->n_transc > 0;
    }
    double best_t = 1e300;
    gp_batch_config b;
    memset(&b, 0, sizeof b);
    b.variant = -1;
    const int unit_sizes[] = {8, 32, 128};
    for (int vi = 0; vi < core_variants(); vi++) {
        if (core_variant_nf(vi) < n_load || core_variant_d(vi) < depth) continue;
        if (core_variant_arith(vi) && any_transc) continue;
        if (core_variant_bool(vi) || core_variant_trees_only(vi)) continue;
        for (int us : unit_sizes) {
            for (int pers = 1; pers >= 0; pers--) {
                gp_batch_config c;
                memset(&c, 0, sizeof c);
                c.variant = vi;
                c.unit_programs = us;
                c.persistent = pers;
                double ms = 0;
                gp_status st = time_config(jobs, ds, c, reps, sc, s, &ms);
                if (st != GP_OK) return st;
                if (ms < best_t) {
                    best_t = ms;
                    b = c;
                }
            }
        }
    }
    if (b.variant < 0) return fail(GP_E_DEPTH, "no kernel variant holds %d features and depth %d", n_load, depth);
    *best = b;
    if (best_ms) *best_ms = best_t;
    std::lock_guard<std::mutex> g(g_tune_mu);
    tune_load_locked();
    g_tune_cache[batch_key(jobs, ds)] = Tuned(core_variant_name(b.variant), b.unit_programs, b.persistent);
    tune_save_locked();
    return GP_OK;
}

// Forget what was tuned for this shape: the launches without a configuration are faster.
static void drop_tuned(const std::vector<BatchJobRef>& jobs, const std::vector<gp_dataset>& ds) {
    std::lock_guard<std::mutex> g(g_tune_mu);
    g_tune_cache.erase(batch_key(jobs, ds));
    tune_save_locked();
}

bool tuned_config(const std::vector<BatchJobRef>& jobs, const std::vector<gp_dataset>& ds, gp_batch_config* c) {
    std::lock_guard<std::mutex> g(g_tune_mu);
    tune_load_locked();
    if (g_tune_cache.empty()) return false;
    auto it = g_tune_cache.find(batch_key(jobs, ds));
    if (it == g_tune_cache.end()) return false;
    // a kernel that does not exist (any more) or cannot run these programs (the shape's key does not say whether they use
    // sin/cos/exp/log) is not taken
    memset(c, 0, sizeof *c);
    c->variant = it->second.variant;
    c->unit_programs = it->second.unit_programs;
    c->persistent = it->second.persistent;
    if (check_config(jobs, *c) == GP_OK) return true;
    clear_error();
    return false;
}

gp_batch_config default_config(const std::vector<BatchJobRef>& jobs) {
    int n_load = 1, depth = 0;
    for (const BatchJobRef& j : jobs) {
        n_load = std::max(n_load, j.pd->n_load);
        depth = std::max(depth, j.pd->max_depth);
    }
    gp_batch_config c;
    memset(&c, 0, sizeof c);
    bool any_transc = false;
    for (const BatchJobRef& j : jobs) any_transc = any_transc || j.pd->n_transc > 0;
    c.variant = pick_core_variant(n_load, depth, transc_fraction(jobs), any_transc);
    c.unit_programs = 32;
    c.persistent = 1;
    return c;
}

// ---------------------------------------------------------------------------
// Job intake shared by the batch API and the server
// ---------------------------------------------------------------------------
gp_status check_datasets(const gp_dataset* ds, int32_t n_ds) {
    if (n_ds < 1 || !ds) return fail(GP_E_INVAL, "no datasets");
    for (int32_t i = 0; i < n_ds; i++) {
        if (!ds[i].X) return fail(GP_E_INVAL, "dataset %d: X is null", i);
        if (ds[i].n_cases < 1) return fail(GP_E_INVAL, "dataset %d: n_cases < 1", i);
        if (ds[i].n_feat < 1) return fail(GP_E_INVAL, "dataset %d: n_feat < 1", i);
    }
    return GP_OK;
}

static gp_status begin_job(const gp_job& j, const gp_dataset* ds, int32_t n_ds, ProgData& pd, ProgBuild& b) {
    if (j.dataset < 0 || j.dataset >= n_ds) return fail(GP_E_NOTFOUND, "dataset %d does not exist", j.dataset);
    if (j.kind != GP_FIT_SUM_ABS && j.kind != GP_FIT_MSE && j.kind != GP_FIT_HITS && j.kind != GP_FIT_CLASS_ERR)
        return fail(GP_E_INVAL, "batched jobs take GP_FIT_SUM_ABS, GP_FIT_MSE, GP_FIT_HITS or GP_FIT_CLASS_ERR (got %d)",
                    j.kind);
    if (!j.out && j.n_prog > 0) return fail(GP_E_INVAL, "job output is null");
    if (!ds[j.dataset].y) return fail(GP_E_INVAL, "dataset %d has no targets", j.dataset);
    const int32_t F = ds[j.dataset].n_feat;
    if (j.form == FORM_TREE) return b.begin_tree(j.tok, j.tcst, j.toff, j.n_prog, F, pd);
    if (j.form == FORM_LINEAR) return b.begin_linear(j.code, j.loff, j.lcst, j.lcst_off, j.n_prog, j.n_reg, F, pd);
    return fail(GP_E_INVAL, "unknown program form %d", j.form);
}

static gp_status finish_job(const ProgData& pd, ProgBuild& b) {
    const gp_status st = b.finish();
    if (st != GP_OK) return st;
    if (pd.n_load > GP_MAX_FEAT)
        return fail(GP_E_INVAL, "programs read feature %d; at most %d features are supported", pd.n_load - 1,
                    GP_MAX_FEAT);
    return GP_OK;
}

gp_status build_job(const gp_job& j, const gp_dataset* ds, int32_t n_ds, ProgData& pd) {
    ProgBuild b;
    const gp_status st = begin_job(j, ds, n_ds, pd, b);
    if (st != GP_OK) return st;
    parallel_for(b.n(), [&](int64_t p0, int64_t p1) { b.lower(p0, p1); });
    return finish_job(pd, b);
}

// Calls fn(part, first, end) for the parts of [p0, p1) that lie in each of
// consecutive ranges; range k is [start[k], start[k + 1]).
template <typename Fn>
static void each_part(const std::vector<int64_t>& start, int64_t p0, int64_t p1, Fn&& fn) {
    size_t k = (size_t)(std::upper_bound(start.begin(), start.end(), p0) - start.begin()) - 1;
    while (p0 < p1) {
        const int64_t e = std::min(p1, start[k + 1]);
        if (p0 < e) fn(k, p0 - start[k], e - start[k]);
        p0 = e;
        k++;
    }
}

}  // namespace gpx

// ===========================================================================
// C ABI
// ===========================================================================
using namespace gpx;

namespace {
std::mutex g_batch_mu;
std::map<hipStream_t, BatchScratch*> g_batch_scratch;

BatchScratch& batch_scratch(hipStream_t s) {
    std::lock_guard<std::mutex> g(g_batch_mu);
    auto it = g_batch_scratch.find(s);
    if (it != g_batch_scratch.end()) return *it->second;
    BatchScratch* sc = new BatchScratch();  // lives until process exit
    g_batch_scratch[s] = sc;
    return *sc;
}

gp_status intake(const gp_dataset* ds, int32_t n_ds, const gp_job* jobs, int32_t n_jobs,
                 std::vector<ProgData>& pds, std::vector<BatchJobRef>& refs, std::vector<gp_dataset>& dv) {
    gp_status st = check_datasets(ds, n_ds);
    if (st != GP_OK) return st;
    if (n_jobs < 0 || (n_jobs > 0 && !jobs)) return fail(GP_E_INVAL, "bad job array");
    // The jobs' programs are lowered in one walk of the host threads (a call with 40 jobs of 250 programs took 5.4 ms of
    // host time with a walk a job, 4.0 so).  The first job that is wrong is the one reported: its arrays (number `begun`)
    // or one of its programs.
    pds.resize(n_jobs);
    std::vector<ProgBuild> builds(n_jobs);
    std::vector<int64_t> start(1, 0);
    int32_t begun = 0;
    while (begun < n_jobs && (st = begin_job(jobs[begun], ds, n_ds, pds[begun], builds[begun])) == GP_OK)
        start.push_back(start.back() + builds[begun++].n());
    char msg[512];
    snprintf(msg, sizeof msg, "%s", st == GP_OK ? "" : last_error());
    parallel_for(start.back(), [&](int64_t p0, int64_t p1) {
        each_part(start, p0, p1, [&](size_t k, int64_t a, int64_t b) { builds[k].lower(a, b); });
    });
    for (int32_t i = 0; i < begun; i++) {
        const gp_status done = finish_job(pds[i], builds[i]);
        if (done != GP_OK) {
            snprintf(msg, sizeof msg, "%s", last_error());
            return fail(done, "job %d: %s", i, msg);
        }
    }
    if (st != GP_OK) return fail(st, "job %d: %s", begun, msg);
    for (int32_t i = 0; i < n_jobs; i++) {
        if (pds[i].n_prog == 0) continue;
        refs.push_back(BatchJobRef{&pds[i], jobs[i].dataset, jobs[i].kind, jobs[i].out});
    }
    dv.assign(ds, ds + n_ds);
    return GP_OK;
}

// Jobs that share form, table, fitness kind and registers, as one population.
struct MergedSet {
    const BatchJobRef* job;                // the first of them
    std::vector<EvalSegment> segments;
    ProgData pd;
};

// The work (tokens x cases) from which a merged set is launched by itself.  It
// then takes the kernel and the launch shape its programs call for (trees
// their ring cores, with rows); below, a launch's own time shows (some 10 us,
// and a tail in which the chip empties), and such sets share one launch over
// a table of units, which must hold trees and register programs alike.
// Measured on 40 populations of 250 over 4,096, 65,536 and 1,048,576 cases:
// 128 ms a call all in one launch, 95 ms by sets.
// GP2D_MERGED_WORK sets another limit (0: every set by itself).
double merged_work() {
    const char* v = getenv("GP2D_MERGED_WORK");
    return v && *v ? strtod(v, nullptr) : 2e9;
}

// Lowered populations of one form, table and register count as one.  False:
// more than its offsets reach.
bool merge_programs(const std::vector<const ProgData*>& parts, ProgData& m) {
    std::vector<int64_t> prog0(1, 0), word0(1, 0);
    for (const ProgData* a : parts) {
        prog0.push_back(prog0.back() + a->n_prog);
        word0.push_back(word0.back() + (int64_t)a->code.size());
    }
    if (prog0.back() > 0x7FFFFFFFll || word0.back() > 0xFFFFFFFFll) return false;
    m = ProgData();
    const ProgData& first = *parts[0];
    m.form = first.form;
    m.opset = first.opset;
    m.n_feat = first.n_feat;
    m.n_reg = first.n_reg;
    m.n_prog = (int32_t)prog0.back();
    for (const ProgData* a : parts) {
        m.n_load = std::max(m.n_load, a->n_load);
        m.max_depth = std::max(m.max_depth, a->max_depth);
        m.n_instr += a->n_instr;
        m.n_named += a->n_named;
        m.n_gpop += a->n_gpop;
        m.n_transc += a->n_transc;
    }
    m.code.resize((size_t)word0.back());
    m.progs.resize((size_t)m.n_prog);
    m.cost.resize((size_t)m.n_prog);
    parallel_for(m.n_prog, [&](int64_t p0, int64_t p1) {
        each_part(prog0, p0, p1, [&](size_t k, int64_t i0, int64_t i1) {
            const ProgData& a = *parts[k];
            for (int64_t i = i0; i < i1; i++) {
                const int64_t p = prog0[k] + i;
                DevProg d = a.progs[i];
                const size_t w0 = d.code_off, w1 = i + 1 < a.n_prog ? a.progs[i + 1].code_off : a.code.size();
                memcpy(m.code.data() + word0[k] + w0, a.code.data() + w0, (w1 - w0) * sizeof(uint32_t));
                d.code_off = (uint32_t)(word0[k] + (int64_t)w0);
                d.row = (uint64_t)p;
                m.progs[p] = d;
                m.cost[p] = a.cost[i];
            }
        });
    });
    return true;
}

// Sort the jobs of a batch into such sets, and the jobs of no set into `rest`.
// False: a set cannot be built, or no kernel holds it, or there is none.
bool merge_jobs(const std::vector<BatchJobRef>& refs, const std::vector<gp_dataset>& ds, std::vector<MergedSet>& sets,
                std::vector<BatchJobRef>& rest) {
    std::map<std::tuple<int32_t, int32_t, int32_t, int32_t>, std::vector<size_t>> by;
    for (size_t i = 0; i < refs.size(); i++)
        by[{refs[i].pd->form, refs[i].ds, refs[i].kind, refs[i].pd->n_reg}].push_back(i);
    std::vector<size_t> left;
    const double limit = merged_work();
    for (auto& kv : by) {
        double work = 0.0;
        int64_t progs = 0;
        for (size_t i : kv.second) {
            work += (double)refs[i].pd->n_gpop * (double)ds[refs[i].ds].n_cases;
            progs += refs[i].pd->n_prog;
        }
        if (work < limit || progs > 0x7FFFFFFFll) {
            left.insert(left.end(), kv.second.begin(), kv.second.end());
            continue;
        }
        sets.emplace_back();
        MergedSet& m = sets.back();
        m.job = &refs[kv.second[0]];
        std::vector<const ProgData*> parts;
        int32_t at = 0;
        for (size_t i : kv.second) {
            parts.push_back(refs[i].pd);
            m.segments.push_back(EvalSegment{at, refs[i].pd->n_prog, refs[i].out});
            at += refs[i].pd->n_prog;
        }
        if (!merge_programs(parts, m.pd)) return false;
        m.pd.variant = default_variant(m.pd);
        if (m.pd.variant < 0) return false;
    }
    std::sort(left.begin(), left.end());
    for (size_t i : left) rest.push_back(refs[i]);
    return !sets.empty();
}

// The jobs in one launch over a table of units.
gp_status eval_table(const std::vector<BatchJobRef>& refs, const std::vector<gp_dataset>& dv, const gp_batch_config& c,
                     hipStream_t s) {
    if (c.variant < 0) return fail(GP_E_DEPTH, "no kernel variant can hold these programs");
    gp_status st;
    if ((st = check_config(refs, c)) != GP_OK) return st;   // (before the kernel is looked for by its number)
    BatchScratch& sc = batch_scratch(s);
    std::lock_guard<std::mutex> g(sc.mu);
    if ((st = core_ready(c.variant, s)) != GP_OK) return st;
    BatchPlan plan;
    if ((st = plan_batch(refs, dv, c, plan)) != GP_OK) return st;
    if ((st = upload_plan(plan, sc, s)) != GP_OK) return st;
    return launch_plan(plan, sc, s);
}

// The batch without a configuration of its own.
gp_status eval_default(const std::vector<BatchJobRef>& refs, const std::vector<gp_dataset>& dv, hipStream_t s) {
    gp_status st;
    std::vector<MergedSet> sets;
    std::vector<BatchJobRef> rest;
    if (!merge_jobs(refs, dv, sets, rest)) {
        sets.clear();
        rest = refs;
    }
    // (looked at before anything is launched, so a call that fails here has done nothing)
    gp_batch_config c;
    if (!rest.empty()) {
        c = default_config(rest);
        if (c.variant < 0) return fail(GP_E_DEPTH, "no kernel variant can hold these programs");
    }
    for (MergedSet& m : sets) {
        Workspace& w = workspace(s);
        std::lock_guard<std::mutex> g(w.mu);
        EvalOptions o;
        o.segments = &m.segments;
        const gp_dataset& d = dv[m.job->ds];
        st = eval_core(m.pd, w.oneshot, true, d.X, d.n_feat, d.n_cases, d.y, m.job->kind, m.job->out, s, &w, &o);
        if (st != GP_OK) return st;
    }
    return rest.empty() ? GP_OK : eval_table(rest, dv, c, s);
}

// Median time on the stream of a whole evaluation, preparation on the host included.
gp_status time_whole(const std::function<gp_status()>& eval, int32_t reps, hipStream_t s, double* ms) {
    gp_status st = eval();   // warm-up
    if (st != GP_OK) return st;
    hipEvent_t e0, e1;
    if (hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess)
        return fail(GP_E_DEVICE, "hipEventCreate failed");
    std::vector<float> t;
    for (int r = 0; r < reps && st == GP_OK; r++) {
        float x = 0;
        hipError_t e = hipEventRecord(e0, s);
        st = eval();
        if (e == hipSuccess) e = hipEventRecord(e1, s);
        if (e == hipSuccess) e = hipEventSynchronize(e1);
        if (e == hipSuccess) e = hipEventElapsedTime(&x, e0, e1);
        if (st == GP_OK && e != hipSuccess) st = fail(GP_E_DEVICE, "timing the batch: %s", hipGetErrorString(e));
        t.push_back(x);
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (st != GP_OK) return st;
    std::sort(t.begin(), t.end());
    *ms = t[t.size() / 2];
    return GP_OK;
}

}  // namespace

extern "C" {

gp_status gp_eval_batch(const gp_dataset* ds, int32_t n_ds, const gp_job* jobs, int32_t n_jobs,
                        const gp_batch_config* cfg, void* stream) {
    clear_error();
    hipStream_t s = (hipStream_t)stream;
    std::vector<ProgData> pds;
    std::vector<BatchJobRef> refs;
    std::vector<gp_dataset> dv;
    gp_status st = intake(ds, n_ds, jobs, n_jobs, pds, refs, dv);
    if (st != GP_OK || refs.empty()) return st;
    gp_batch_config c;
    if (cfg) c = *cfg;
    else if (!tuned_config(refs, dv, &c)) return eval_default(refs, dv, s);
    return eval_table(refs, dv, c, s);
}

gp_status gp_tune_batch(const gp_dataset* ds, int32_t n_ds, const gp_job* jobs, int32_t n_jobs, int32_t reps,
                        gp_batch_config* best, double* best_ms, void* stream) {
    clear_error();
    if (!best) return fail(GP_E_INVAL, "best is null");
    std::vector<ProgData> pds;
    std::vector<BatchJobRef> refs;
    std::vector<gp_dataset> dv;
    gp_status st = intake(ds, n_ds, jobs, n_jobs, pds, refs, dv);
    if (st != GP_OK) return st;
    if (refs.empty()) return fail(GP_E_INVAL, "nothing to tune");
    hipStream_t s = (hipStream_t)stream;
    if (reps < 1) reps = 3;
    double ms = 0.0, dflt = 0.0, whole = 0.0;
    {
        BatchScratch& sc = batch_scratch(s);
        std::lock_guard<std::mutex> g(sc.mu);
        if ((st = tune_batch(refs, dv, reps, sc, s, best, &ms)) != GP_OK) return st;
    }
    if (best_ms) *best_ms = ms;
    // the candidates were timed by their launches; the default prepares several launches, so whole calls are compared
    if ((st = time_whole([&] { return eval_table(refs, dv, *best, s); }, reps, s, &whole)) != GP_OK) return st;
    if (time_whole([&] { return eval_default(refs, dv, s); }, reps, s, &dflt) == GP_OK) {
        if (dflt < whole) drop_tuned(refs, dv);
    } else {
        clear_error();   // (no memory for it: the configuration serves)
    }
    return GP_OK;
}

int32_t gp_num_variants(void) { return core_variants(); }

gp_status gp_variant_info(int32_t i, int32_t* t, int32_t* depth, int32_t* n_feat, int32_t* vgprs,
                          int32_t* flags) {
    clear_error();
    if (i < 0 || i >= core_variants()) return fail(GP_E_INVAL, "variant %d does not exist", i);
    if (t) *t = core_variant_t(i);
    if (depth) *depth = core_variant_d(i);
    if (n_feat) *n_feat = core_variant_nf(i);
    if (vgprs) *vgprs = core_variant_ncv(i);
    if (flags)
        *flags = (core_variant_arith(i) ? GP_VARIANT_NO_TRANSC : 0) | (core_variant_bool(i) ? GP_VARIANT_BOOLEAN : 0) |
                 (core_variant_trees_only(i) && !core_variant_bool(i) ? GP_VARIANT_TREES_ONLY : 0);
    return GP_OK;
}

}  // extern "C"
