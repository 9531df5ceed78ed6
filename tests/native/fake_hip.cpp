// A HIP runtime of host memory, and kernel launchers that record what they
// are given, so that the library's host code (uploads, layouts, batches) runs
// without a device.  Copies take place at once; an allocation can be made to
// fail.  Nothing is evaluated: outputs keep what they held.
#include <hip/hip_runtime_api.h>
#include <stdlib.h>
#include <string.h>

#include <atomic>
#include <mutex>

#include "blockgp.h"
#include "core_kernels.h"
#include "gp.h"
#include "runtime.h"

namespace gpx {
#include "core_gen.inc"
}

struct FakeState {
    int fail_malloc = 0;       // the n-th allocation from now on fails (0: none)
    int launches = 0;          // evaluation launches
    int last_rows = 0, last_groups = 0, last_variant = -1, last_table = 0;
    int null_layout = 0;       // launches whose group layout was null or not a layout
    int uploads = 0;           // copies to the device
    int capturing = 0;         // streams are being captured
    double now_ms = 0.0;       // the clock of events: advanced by launches and by copies to the device
    double launch_ms = 1.0, table_ms = 1.0, copy_ms = 0.0;
};
static FakeState g;
static std::mutex g_mu;
static std::atomic<int> g_lowered{0};   // programs lowered

// lower.cpp is compiled with these two functions under other names, so that calls are counted
namespace gpx {
int real_lower_tree(const int32_t*, const float*, int64_t, int32_t, uint32_t*, TreeLowering*, char*, int);
int64_t real_needed_linear(const uint32_t*, int64_t, int32_t, uint32_t*, uint32_t*);
int lower_tree(const int32_t* tok, const float* cst, int64_t n, int32_t n_feat, uint32_t* words, TreeLowering* st, char* err,
               int opset) {
    g_lowered++;
    return real_lower_tree(tok, cst, n, n_feat, words, st, err, opset);
}
int64_t needed_linear(const uint32_t* code, int64_t n, int32_t n_reg, uint32_t* out, uint32_t* live) {
    g_lowered++;
    return real_needed_linear(code, n, n_reg, out, live);
}
}  // namespace gpx

extern "C" {
FakeState* fake_state() { return &g; }
void fake_fail_malloc(int n) { g.fail_malloc = n; }
int fake_int(int what) {
    const int v[] = {g.launches, g.last_rows, g.last_groups, g.last_variant, g.last_table, g.null_layout, g.uploads,
                     g_lowered.load()};
    return v[what];
}
void fake_capturing(int on) { g.capturing = on; }
void fake_times(double launch, double table, double copy) {
    g.launch_ms = launch;
    g.table_ms = table;
    g.copy_ms = copy;
}

hipError_t hipMalloc(void** p, size_t n) {
    std::lock_guard<std::mutex> l(g_mu);
    *p = nullptr;
    if (g.fail_malloc > 0 && --g.fail_malloc == 0) return hipErrorOutOfMemory;
    *p = malloc(n ? n : 1);
    return *p ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipFree(void* p) { free(p); return hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { return hipMalloc(p, n); }
hipError_t hipHostFree(void* p) { free(p); return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind kind, hipStream_t) {
    memcpy(d, s, n);
    if (kind == hipMemcpyHostToDevice) {
        g.uploads++;
        g.now_ms += g.copy_ms;
    }
    return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t* e) { *e = (hipEvent_t) new double(0.0); return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e) { delete (double*)e; return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t) { *(double*)e = g.now_ms; return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventQuery(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t a, hipEvent_t b) {
    *ms = (float)(*(double*)b - *(double*)a);
    return hipSuccess;
}
hipError_t hipStreamCreate(hipStream_t* s) { *s = (hipStream_t)malloc(1); return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { return hipStreamCreate(s); }
hipError_t hipStreamDestroy(hipStream_t s) { free(s); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* c) {
    *c = g.capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode*) { return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipGetDeviceProperties(hipDeviceProp_t* p, int) {
    memset(p, 0, sizeof *p);
    p->multiProcessorCount = 256;
    return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t e) { return e == hipErrorOutOfMemory ? "out of memory" : "error"; }

gp_status gp_progset_eval_noalloc(gp_progset*, const float*, int32_t, int64_t, const float*, int32_t, void*, void*) {
    return GP_E_DEVICE;
}
}  // extern "C"

namespace gpx {
hipError_t core_launch(int vi, const CoreArgs& a, uint32_t, hipStream_t) {
    if (a.probe) {
        a.probe_out[0] = 0x7F0000000000ull;
        a.probe_out[1] = 0;
        a.probe_out[2] = (uint64_t)kCoreVariants[vi].rows_base;
        return hipSuccess;
    }
    g.launches++;
    g.last_variant = vi;
    g.last_table = a.units != nullptr;
    g.last_rows = a.n_rows;
    g.last_groups = a.n_groups;
    g.now_ms += a.units ? g.table_ms : g.launch_ms;
    if (!a.units) {
        // the layout is read as the kernel reads it: groups, rows, and the programs' order
        if (!a.group_off || (uintptr_t)a.group_off < 4096) {
            g.null_layout++;
            return hipSuccess;
        }
        if (a.group_prog[0] != 0) g.null_layout++;   // never written
        for (int k = 0; k < a.n_groups; k++)
            if (a.group_off[k] > a.group_off[k + 1] || a.group_prog[k] > a.group_prog[k + 1]) g.null_layout++;
    }
    return hipSuccess;
}
int core_blocks_per_cu(int) { return 1; }
hipError_t core_zero_counter(uint32_t*, hipStream_t) { return hipSuccess; }
hipError_t core_reduce_jobs(const ReduceArgs*, int32_t, int64_t, hipStream_t) { return hipSuccess; }
hipError_t core_reduce_one(const ReduceArgs&, hipStream_t) { return hipSuccess; }
hipError_t blockgp_launch(int, const BgArgs&, int32_t, hipStream_t) { return hipSuccess; }
}  // namespace gpx
