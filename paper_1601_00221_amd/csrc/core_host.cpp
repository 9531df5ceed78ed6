// Host side of the interpreter core: find each kernel variant's handler
// table on the device, and translate lowered programs into core
// instructions (handler address, operand offsets, constant).
#include <hip/hip_runtime_api.h>
#include <stdio.h>
#include <string.h>

#include <algorithm>
#include <functional>
#include <memory>
#include <mutex>
#include <string>
#include <unordered_map>
#include <vector>

#include "../../include/gp.h"
#include "core_host.h"
#include "core_kernels.h"
#include "gp_internal.h"
#include "gp_math.h"
#include "runtime.h"

namespace gpx {
#include "core_gen.inc"

namespace {

// Handler slot by key: an open-addressing table (a few thousand keys, one
// lookup per translated instruction).
struct SlotTable {
    std::vector<uint32_t> keys;   // 0xFFFFFFFF = empty (no handler key has it)
    std::vector<uint16_t> slots;
    uint32_t mask = 0;
    static uint32_t hash(uint32_t k) { return (k * 0x9E3779B1u) ^ (k >> 15); }
    void build(const std::vector<std::pair<uint32_t, uint16_t>>& kv) {
        uint32_t cap = 16;
        while (cap < 2 * kv.size()) cap <<= 1;
        keys.assign(cap, 0xFFFFFFFFu);
        slots.assign(cap, 0);
        mask = cap - 1;
        for (auto& e : kv) {
            uint32_t i = hash(e.first) & mask;
            while (keys[i] != 0xFFFFFFFFu && keys[i] != e.first) i = (i + 1) & mask;
            keys[i] = e.first;
            slots[i] = e.second;
        }
    }
    bool find(uint32_t k, uint16_t* out) const {
        if (keys.empty()) return false;
        for (uint32_t i = hash(k) & mask;; i = (i + 1) & mask) {
            if (keys[i] == k) {
                *out = slots[i];
                return true;
            }
            if (keys[i] == 0xFFFFFFFFu) return false;
        }
    }
};

struct VariantMap {
    bool ready = false;
    int device = -1;
    uint64_t base = 0;
    SlotTable slot;
};

std::mutex g_mu;
std::vector<std::shared_ptr<const VariantMap>> g_maps;   // by variant, once its table is found

uint32_t key_of(int kind, int op, int p1, int p2) {
    return (uint32_t)kind | ((uint32_t)op << 8) | ((uint32_t)(uint8_t)(int8_t)p1 << 16) |
           ((uint32_t)(uint8_t)(int8_t)p2 << 24);
}

}  // namespace

static SlotTable variant_slots(int vi) {
    const CoreVariantDesc& v = kCoreVariants[vi];
    std::vector<std::pair<uint32_t, uint16_t>> kv;
    kv.reserve(v.n);
    for (int i = 0; i < v.n; i++)
        kv.push_back({key_of(v.keys[i].kind, v.keys[i].op, v.keys[i].p1, v.keys[i].p2), v.slots[i]});
    SlotTable t;
    t.build(kv);
    return t;
}

const CoreVariantDesc& core_desc(int vi) { return kCoreVariants[vi]; }
int core_variants() { return (int)(sizeof(kCoreVariants) / sizeof(kCoreVariants[0])); }
int core_reg_levels(int vi) {
    // Boolean kernels run trees only: no linear registers before the features
    const CoreVariantDesc& v = kCoreVariants[vi];
    return v.arith >= 2 || v.d > GPX_LIN_REGS ? v.d : GPX_LIN_REGS;
}

// Kernel modes (gen_core.py): 0 full, 1 without sin/cos/exp/log code, 2 Boolean, 3 trees only without
// sin/cos/exp/log code, 4 trees only with it.
static bool mode_no_transc(int mode) { return mode == 1 || mode == 2 || mode == 3; }

static constexpr int kShallowDepth = 12;

int pick_core_variant(int n_load, int depth, double transc_frac, bool has_transc, bool boolean, bool trees_only, bool wide) {
    // Programs rich in sin/cos/exp/log (binary64) run best where two slots of
    // them are computed side by side, and with as many waves per SIMD as that
    // leaves, to hide the latency; the others with
    // the widest tile, on a kernel without that code if they use none of it.  Ties go to the fewest feature slots, then the fewest
    // handlers (least code).  (Measured on the 4096 x 65,536 tree workloads.)
    const bool heavy = transc_frac > 0.2;
    // (ring cores before pair cores of the same shape)
    int best = -1;
    auto waves = [](const CoreVariantDesc& v) {
        const int lv = v.arith >= 2 || v.d > GPX_LIN_REGS ? v.d : GPX_LIN_REGS;
        const int vg = (v.ncv + lv * v.t + v.nf * v.t + 7) / 8 * 8;
        return 512 / vg;
    };
    auto score = [&](const CoreVariantDesc& v) {
        if (heavy) return (v.ncv >= 48) * 100000000 + waves(v) * 1000000 + v.ring * 100000 + v.t * 10000 - v.nf * 100 - v.n / 100;
        // trees-only kernels first (the smallest handler tables), then those without sin/cos/exp/log code, the
        // widest tile, then the most waves per SIMD (4 against 3 at T = 4: 13-16 % on the linear and Shuttle-shaped
        // workloads)
        return (v.arith == 3) * 400000000 + mode_no_transc(v.arith) * 200000000 + (v.ncv <= 64) * 100000000 + v.t * 10000 +
               waves(v) * 1000 - v.nf * 100 - v.n / 100;
    };
    // Boolean programs: the most slots in flight per SIMD (waves x tile width); ties go to more waves (they
    // hide the dispatch chain of the one-instruction handlers: measured 5 % on the 20-multiplexer), then to
    // fewer feature slots
    auto score_bool = [&](const CoreVariantDesc& v) {
        return waves(v) * v.t * 100000 + waves(v) * 1000 + v.ncv * 10 - v.nf;
    };
    for (int i = 0; i < core_variants(); i++) {
        const CoreVariantDesc& v = kCoreVariants[i];
        if (v.by_number_only || (v.arith == 2) != boolean) continue;
        if (v.arith >= 3 && !trees_only) continue;
        // Features in LDS: where fewer than four waves a SIMD would hold them in registers (13 and more with
        // sin/cos/exp/log: 4096 trees x 30000 cases over 13, 24, 41 features 3.63, 4.02, 4.95 ms in registers, 3.34,
        // 3.87, 4.26 so; without those functions 25 and more: 1.27 and 1.11 ms).
        if (v.cap > v.nf) {
            if (!wide || n_load <= (has_transc ? 12 : 24) || v.cap < n_load || v.d <= depth) continue;
            return i;
        } else if (v.nf < n_load || v.d < depth || (mode_no_transc(v.arith) && has_transc)) {
            continue;
        }
        // the deep variants (fewer waves per SIMD) serve only programs that need them
        if (v.d > kShallowDepth && depth <= kShallowDepth) continue;
        if (best < 0) { best = i; continue; }
        const bool better = boolean ? score_bool(v) > score_bool(kCoreVariants[best])
                                    : score(v) > score(kCoreVariants[best]);
        if (better) best = i;
    }
    return best;
}

gp_status core_ready(int vi, hipStream_t s) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return fail(GP_E_DEVICE, "hipGetDevice: %s", hipGetErrorString(e));
    std::lock_guard<std::mutex> g(g_mu);
    if ((int)g_maps.size() < core_variants()) g_maps.resize(core_variants());
    if (g_maps[vi] && g_maps[vi]->device == dev) return GP_OK;
    uint64_t* d = nullptr;
    e = hipMalloc(&d, 256);
    if (e != hipSuccess) return fail(GP_E_DEVICE, "hipMalloc: %s", hipGetErrorString(e));
    CoreArgs a;
    memset(&a, 0, sizeof a);
    a.probe = 1;
    a.probe_out = d;
    e = core_launch(vi, a, 1, s);
    uint64_t probed[3] = {0, 1, 1};   // the handler table, and where the reduction tables and the rows lie in LDS
    if (e == hipSuccess) e = hipMemcpyAsync(probed, d, 24, hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    (void)hipFree(d);
    if (e != hipSuccess) return fail(GP_E_DEVICE, "handler table probe: %s", hipGetErrorString(e));
    const uint64_t base = probed[0];
    if (probed[1] != 0 || probed[2] != (uint64_t)kCoreVariants[vi].rows_base)
        return fail(GP_E_DEVICE, "reduction tables at LDS offset %llu, rows at %llu", (unsigned long long)probed[1],
                    (unsigned long long)probed[2]);
    if (base == 0 || (base & (GPX_SLOT - 1)) != 0) return fail(GP_E_DEVICE, "handler table probe returned %llx",
                                                               (unsigned long long)base);
    auto m = std::make_shared<VariantMap>();
    m->slot = variant_slots(vi);
    m->base = base;
    m->device = dev;
    m->ready = true;
    g_maps[vi] = m;
    return GP_OK;
}

bool core_is_ready(int vi) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return false;
    std::lock_guard<std::mutex> g(g_mu);
    return vi >= 0 && vi < (int)g_maps.size() && g_maps[vi] && g_maps[vi]->device == dev;
}

namespace {

// Handlers come in two phases (records are fetched two at a time, see
// gen_core.py): instructions alternate A, B, A, ... and every entry into the
// core -- a program's start, the return from an exit -- begins with A.  Ring
// cores have four, taken in turn.
constexpr int kPhaseB = 0x80;

// Writes core instructions (4 words each) to `out`, at most `cap` of them.
struct Emitter {
    const CoreVariantDesc& v;
    const VariantMap& m;
    uint32_t* out;
    int64_t cap;
    char* err;
    int64_t n = 0;
    bool ok = true;
    int phase = 0;

    void put(int kind, int op, int p1, int p2, uint32_t pay, uint32_t cst) {
        uint16_t slot = 0;
        const bool have = m.slot.find(key_of(kind | phase, op, p1, p2), &slot);
        phase = v.ring ? (phase + (1 << GPX_RING_PHASE)) & (3 << GPX_RING_PHASE) : phase ^ kPhaseB;
        if (!have) {
            snprintf(err, 256, "no core handler for kind %d op %d (%d, %d)", kind, op, p1, p2);
            ok = false;
            return;
        }
        if (n >= cap) {
            snprintf(err, 256, "internal: core code longer than counted");
            ok = false;
            return;
        }
        const uint64_t addr = m.base + (uint64_t)slot * v.slot_bytes;
        uint32_t* o = out + 4 * n++;
        o[0] = (uint32_t)addr;
        o[1] = (uint32_t)(addr >> 32);
        o[2] = pay;
        o[3] = cst;
    }
    // leave the handlers for the block's tail: operation op on A (offset or constant), B, into D
    void exit(uint32_t op, int oa, int ob, int od, bool a_const, bool b_const, uint32_t cst) {
        const uint32_t fl = (a_const ? 1u : 0u) | (b_const ? 2u : 0u);
        put(CK_EXIT, 0, 0, 0,
            (uint32_t)(oa & 255) | ((uint32_t)(ob & 255) << 8) | ((uint32_t)(od & 255) << 16) |
                ((op | (fl << 4)) << 24),
            cst);
        phase = 0;   // the core is entered again after an exit
    }
    // feature f of the tile to stack level 0 (programs of rows)
    void load(int f) {
        put(CK_EXIT, 0, 0, 0, (CORE_OP_LOAD << 24) | (uint32_t)f, 0);
        phase = 0;
    }
    // the end of a program: its row, and the records of the program that follows it
    void end(uint32_t row, uint32_t next) {
        if (ok) put(CK_EXIT, 0, 0, 0, (CORE_OP_END << 24) | (next & 0xFFFFFFu), row);
    }
    // protected division, in the core (every arithmetic kernel has its
    // handlers): the exit's payload layout, without leaving
    void fail_two_constants() {
        // lowering pushes one of two constant operands first, and register programs move one into the
        // destination: no function of two constants reaches the handlers
        snprintf(err, 256, "internal: a function of two constants reached core translation");
        ok = false;
    }
    void div(int oa, int ob, int od, bool a_const, bool b_const, uint32_t cst) {
        if (a_const && b_const) return fail_two_constants();
        const int kind = a_const ? CK_DCV : b_const ? CK_DVC : CK_DVV;
        put(kind, GP_PDIV, 0, 0,
            (uint32_t)(oa & 255) | ((uint32_t)(ob & 255) << 8) | ((uint32_t)(od & 255) << 16), cst);
    }
    // >, <, ==, logical AND and OR in the core: 1 or 0 per slot
    void cmp(uint32_t op, int oa, int ob, int od, bool a_const, bool b_const, uint32_t cst) {
        if (a_const && b_const) return fail_two_constants();
        const int kind = a_const ? CK_CCV : b_const ? CK_CVC : CK_CVV;
        put(kind, (int)op, 0, 0,
            (uint32_t)(oa & 255) | ((uint32_t)(ob & 255) << 8) | ((uint32_t)(od & 255) << 16), cst);
    }
    // ring cores: functions of a stack entry and the one above it or a variable, at level l = offset / T
    static uint32_t swapped(uint32_t op) { return op == GP_GT ? (uint32_t)GP_LT : op == GP_LT ? (uint32_t)GP_GT : op; }
    bool ring_apply(uint32_t op, uint32_t mode, int h, int xa, int xb) {
        if (!v.ring || v.arith == 2) return false;
        const int T = v.t;
        if (op == GP_PDIV) {
            // the level above the operand holds a variable's copy, so the top level takes the general form
            switch (mode) {
                case M_SS: put(CK_DSS, (int)op, h - 2, 0, 0, 0); return true;
                case M_SSR: put(CK_DSSR, (int)op, h - 2, 0, 0, 0); return true;
                case M_SX: case M_XS:
                    if (h - 1 > v.d - 2) return false;
                    put(mode == M_SX ? CK_DSX : CK_DXS, (int)op, h - 1, 0, (uint32_t)(mode == M_SX ? xb : xa), 0);
                    return true;
                default: return false;
            }
        }
        switch (mode) {
            case M_SS: put(CK_CSS, (int)op, 0, 0, (uint32_t)((h - 2) * T), 0); return true;
            case M_SSR: put(CK_CSS, (int)swapped(op), 0, 0, (uint32_t)((h - 2) * T), 0); return true;
            case M_SX: put(CK_CSX, (int)op, h - 1, 0, (uint32_t)xb, 0); return true;
            case M_XS: put(CK_CSX, (int)swapped(op), h - 1, 0, (uint32_t)xa, 0); return true;
            default: return false;
        }
    }
    // protected division and the binary classification functions in their general form: operands at any offsets, or
    // one of them the constant
    void apply(uint32_t op, bool boolean, int oa, int ob, int od, bool a_const, bool b_const, uint32_t cst) {
        if (!boolean && op == GP_PDIV) {
            div(oa, ob, od, a_const, b_const, cst);
        } else if (!boolean && (op == GP_GT || op == GP_LT || op == GP_EQ || op == GP_AND || op == GP_OR)) {
            cmp(op, oa, ob, od, a_const, b_const, cst);
        } else {
            snprintf(err, 256, "no core handler for binary function %u", op);
            ok = false;
        }
    }
};

// Functions with a handler for every operand mode: + - * and, in Boolean
// kernels, the four bitwise functions (in arithmetic trees opcodes 8 and 9 are
// the logical AND and OR, which go with the compares).
bool is_core_op(uint32_t op, bool boolean) {
    return op == GP_ADD || op == GP_SUB || op == GP_MUL || (boolean && op >= GP_AND && op <= GP_NOR);
}

}  // namespace

// sin, cos, exp or log of a constant, as the kernel computes it
static uint32_t unary_of_constant(uint32_t op, uint32_t bits) {
    static const std::vector<double> tab = [] {
        std::vector<double> t(gmath::kTabSize);
        gmath::tab_fill(t.data(), 0, 1);
        return t;
    }();
    float a[1] = {gmath::float_of(bits)};
    switch (op) {
        case GP_SIN: gmath::sincos_n<1>(a, false, tab.data(), 0); break;
        case GP_COS: gmath::sincos_n<1>(a, true, tab.data(), 0); break;
        case GP_EXPC: gmath::expc_n<1>(a, tab.data(), 0); break;
        default: gmath::plog_n<1>(a, tab.data(), 0); break;
    }
    return gmath::bits_of(a[0]);
}

static int row_key(uint32_t op, int f) { return (int)(op - GP_SIN) * GP_MAX_FEAT + f; }

static int translate_tree(const uint32_t* w, int64_t n_instr, int vi, const VariantMap& m, const RowPlan* rows,
                          uint32_t row, uint32_t next, uint32_t* out, int64_t cap, int64_t* n_out, char* err) {
    const CoreVariantDesc& v = kCoreVariants[vi];
    const int T = v.t, FO = core_reg_levels(vi) * T;
    Emitter e{v, m, out, cap, err};
    auto push_row = [&](int r, int h) { e.put(CK_PUSHR, 0, h, 0, (uint32_t)(r * 256 * T), 0); };
    for (int64_t i = 0; i < n_instr && e.ok; i++) {
        const uint32_t w0 = w[2 * i], c = w[2 * i + 1];
        const uint32_t op = w0 & 15u;
        uint32_t mode = (w0 >> 4) & 15u;
        const int fa = (int)((w0 >> 8) & 255u), fb = (int)((w0 >> 16) & 255u), ha = (int)(w0 >> 24);
        int h;  // stack height before the instruction
        switch (mode) {
            case M_SS: case M_SSR: h = ha + 1; break;
            case M_S3: h = ha + 2; break;
            case M_XX: case M_XC: case M_CX: case M_X: case M_C: h = ha - 1; break;
            default: h = ha; break;
        }
        const int xa = FO + fa * T, xb = FO + fb * T;
        if (v.cap > v.nf && op != OP_IF) {
            // features in LDS are pushed, and the instruction takes them from the stack
            const bool la = fa >= v.nf, lb = fb >= v.nf;
            switch (mode) {
                case M_SX: if (lb) push_row(rows->feature(fb), h++), mode = M_SS; break;
                case M_XS: if (la) push_row(rows->feature(fa), h++), mode = M_SSR; break;
                case M_XC: if (la) push_row(rows->feature(fa), h++), mode = M_SC; break;
                case M_CX: if (lb) push_row(rows->feature(fb), h++), mode = M_CS; break;
                case M_XX:
                    if (la) {
                        push_row(rows->feature(fa), h++);
                        mode = M_SX;
                        if (lb) push_row(rows->feature(fb), h++), mode = M_SS;
                    } else if (lb) {
                        push_row(rows->feature(fb), h++);
                        mode = M_XS;
                    }
                    break;
                case M_X:
                    if (!la) break;
                    if (op == OP_PUSH) {
                        push_row(rows->feature(fa), h);
                        continue;
                    }
                    if (rows->row[row_key(op, fa)] < 0) push_row(rows->feature(fa), h++), mode = M_S;
                    break;
                default: break;
            }
        }
        if (op == OP_PUSH) {
            if (mode == M_X) {
                // Boolean kernels push a variable only as a whole program, at the bottom
                if (v.arith == 2 && h != 0) {
                    snprintf(err, 256, "push of a variable above the stack bottom");
                    return GP_E_INVAL;
                }
                e.put(CK_PUSHX, 0, h, 0, (uint32_t)xa, 0);
            } else {
                e.put(CK_PUSHC, 0, 0, 0, (uint32_t)(h * T), c);
            }
            continue;
        }
        if (mode == M_S3) {
            // IF: operands at positions fa, fb and the third of s[h-3 .. h-1]; the exit writes
            // the lowest of the three offsets
            const int pc = 3 - fa - fb;
            if (op != OP_IF || fa > 2 || fb > 2 || pc < 0 || pc > 2 || fa == fb || h < 3) {
                snprintf(err, 256, "malformed three-operand instruction");
                return GP_E_INVAL;
            }
            // IF runs in the core: operands at three offsets, the result to the lowest, s[h-3]
            if (v.ring) {
                e.put(CK_IF3, GP_IF, 3 * fa + fb, 0, (uint32_t)((h - 3) * T), 0);
                continue;
            }
            e.put(CK_IF3, GP_IF, 0, 0,
                  (uint32_t)((h - 3 + fa) * T) | ((uint32_t)((h - 3 + fb) * T) << 8) |
                      ((uint32_t)((h - 3 + pc) * T) << 16) | ((uint32_t)((h - 3) * T) << 24),
                  0);
            continue;
        }
        if (is_core_op(op, v.arith == 2)) {
            const bool comm = op != GP_SUB;
            switch (mode) {
                case M_SS: e.put(CK_SS, op, 0, 0, (uint32_t)((h - 2) * T), 0); break;
                case M_SSR:
                    if (comm) e.put(CK_SS, op, 0, 0, (uint32_t)((h - 2) * T), 0);
                    else e.put(CK_SSR, op, 0, 0, (uint32_t)((h - 2) * T), 0);
                    break;
                case M_SX: e.put(CK_SX, op, h - 1, 0, (uint32_t)xb, 0); break;
                case M_XS:
                    if (comm) e.put(CK_SX, op, h - 1, 0, (uint32_t)xa, 0);
                    else e.put(CK_XS, op, h - 1, 0, (uint32_t)xa, 0);
                    break;
                case M_SC: e.put(CK_SC, op, 0, 0, (uint32_t)((h - 1) * T), c); break;
                case M_CS:
                    if (comm) e.put(CK_SC, op, 0, 0, (uint32_t)((h - 1) * T), c);
                    else e.put(CK_CS, op, 0, 0, (uint32_t)((h - 1) * T), c);
                    break;
                case M_XX:
                    if (h < v.xx) {
                        if (comm) {
                            const int a = fa < fb ? fa : fb, b = fa < fb ? fb : fa;
                            e.put(CK_XX, op, h, b - a, (uint32_t)(a * T), 0);
                        } else {
                            e.put(CK_XX, op, h, fb - fa, (uint32_t)(fa * T), 0);
                        }
                    } else {
                        e.put(CK_XX2, op, h, 0, (uint32_t)xa | ((uint32_t)xb << 8), 0);
                    }
                    break;
                case M_XC: e.put(CK_XC, op, h, 0, (uint32_t)xa, c); break;
                case M_CX:
                    if (comm) e.put(CK_XC, op, h, 0, (uint32_t)xb, c);
                    else e.put(CK_CX, op, h, 0, (uint32_t)xb, c);
                    break;
                default:
                    snprintf(err, 256, "mode %u is not a binary mode", mode);
                    return GP_E_INVAL;
            }
            continue;
        }
        // protected division and the classification functions: a ring core's forms for operands on the stack, else the
        // general one.  sin/cos/exp/log are exits to the block's tail (or a row, or, of a constant, a push).
        const bool bl = v.arith == 2;
        if (!bl && (op == GP_PDIV || op == GP_GT || op == GP_LT || op == GP_EQ || op == GP_AND || op == GP_OR) &&
            e.ring_apply(op, mode, h, xa, xb))
            continue;
        switch (mode) {
            case M_SS: e.apply(op, bl, (h - 2) * T, (h - 1) * T, (h - 2) * T, false, false, 0); break;
            case M_SSR: e.apply(op, bl, (h - 1) * T, (h - 2) * T, (h - 2) * T, false, false, 0); break;
            case M_SX: e.apply(op, bl, (h - 1) * T, xb, (h - 1) * T, false, false, 0); break;
            case M_XS: e.apply(op, bl, xa, (h - 1) * T, (h - 1) * T, false, false, 0); break;
            case M_SC: e.apply(op, bl, (h - 1) * T, 0, (h - 1) * T, false, true, c); break;
            case M_CS: e.apply(op, bl, 0, (h - 1) * T, (h - 1) * T, true, false, c); break;
            case M_XX: e.apply(op, bl, xa, xb, h * T, false, false, 0); break;
            case M_XC: e.apply(op, bl, xa, 0, h * T, false, true, c); break;
            case M_CX: e.apply(op, bl, 0, xb, h * T, true, false, c); break;
            case M_S: e.exit(op, (h - 1) * T, 0, (h - 1) * T, false, false, 0); break;
            case M_X: {
                const int r = rows && rows->n() > 0 ? rows->row[row_key(op, fa)] : -1;
                if (r >= 0) push_row(r, h);
                else e.exit(op, xa, 0, h * T, false, false, 0);
                break;
            }
            default:  // M_C
                if (v.ring) e.put(CK_PUSHC, 0, 0, 0, (uint32_t)(h * T), unary_of_constant(op, c));
                else e.exit(op, 0, 0, h * T, true, false, c);
                break;
        }
    }
    e.end(row, next);
    *n_out = e.n;
    return e.ok ? GP_OK : GP_E_INVAL;
}

// Core instructions of a register program: the set-up of the registers whose
// starting value it reads, one or two per instruction, and the end.
static int64_t linear_records(const uint32_t* w, int64_t n, uint32_t live) {
    int64_t k = __builtin_popcount(live) + n + 1;
    for (int64_t i = 0; i < n; i++) {
        const uint32_t op = w[i] & 255u;
        const bool c1 = ((w[i] >> 16) & 255u) >= GP_SRC_CONST, c2 = (w[i] >> 24) >= GP_SRC_CONST;
        k += (c1 && c2 && !(op >= GP_SIN && op <= GP_PLOG));
    }
    return k;
}

static int translate_linear(const uint32_t* w, int64_t n, uint32_t live, const uint32_t* cst, int32_t n_reg, int32_t n_feat, int vi,
                            const VariantMap& m, uint32_t row, uint32_t next, uint32_t* out, int64_t cap,
                            int64_t* n_out, char* err) {
    const CoreVariantDesc& v = kCoreVariants[vi];
    const int T = v.t, FO = core_reg_levels(vi) * T;
    Emitter e{v, m, out, cap, err};
    auto off = [&](int id) { return id < n_reg ? id * T : FO + (id - n_reg) * T; };
    // registers start as r[k] = x[k mod n_feat]
    for (int k = 0; k < n_reg && e.ok; k++)
        if ((live >> k) & 1u) e.put(CK_MOVX, 0, k, 0, (uint32_t)(FO + (k % n_feat) * T), 0);
    for (int64_t i = 0; i < n && e.ok; i++) {
        const uint32_t wd = w[i];
        const uint32_t op = wd & 255u;
        const int d = (int)((wd >> 8) & 255u), s1 = (int)((wd >> 16) & 255u), s2 = (int)(wd >> 24);
        const bool c1 = s1 >= GP_SRC_CONST, c2 = s2 >= GP_SRC_CONST;
        const uint32_t v1 = c1 ? cst[s1 - GP_SRC_CONST] : 0u, v2 = c2 ? cst[s2 - GP_SRC_CONST] : 0u;
        if (op >= GP_SIN && op <= GP_PLOG) {  // in the block's tail
            e.exit(op, c1 ? 0 : off(s1), 0, d * T, c1, false, v1);
            continue;
        }
        if (!is_core_op(op, false)) {   // protected division and the classification functions
            if (c1 && c2) {
                e.put(CK_MOVC, 0, d, 0, 0, v1);
                e.apply(op, false, d * T, 0, d * T, false, true, v2);
            } else {
                e.apply(op, false, c1 ? 0 : off(s1), c2 ? 0 : off(s2), d * T, c1, c2, c1 ? v1 : v2);
            }
            continue;
        }
        const bool comm = op != GP_SUB;
        if (c1 && c2) {
            e.put(CK_MOVC, 0, d, 0, 0, v1);
            if (comm) e.put(CK_CR, op, d, 0, (uint32_t)(d * T), v2);
            else e.put(CK_RC, op, d, 0, (uint32_t)(d * T), v2);
        } else if (c1) {
            e.put(CK_CR, op, d, 0, (uint32_t)off(s2), v1);
        } else if (c2) {
            if (comm) e.put(CK_CR, op, d, 0, (uint32_t)off(s1), v2);
            else e.put(CK_RC, op, d, 0, (uint32_t)off(s1), v2);
        } else if (s1 < n_reg) {
            e.put(CK_RR, op, d, s1, (uint32_t)off(s2), 0);
        } else if (s2 < n_reg) {
            if (comm) e.put(CK_RR, op, d, s2, (uint32_t)off(s1), 0);
            else e.put(CK_XR, op, d, s2, (uint32_t)off(s1), 0);
        } else {
            e.put(CK_FF, op, d, 0, (uint32_t)off(s1) | ((uint32_t)off(s2) << 8), 0);
        }
    }
    e.end(row, next);
    *n_out = e.n;
    return e.ok ? GP_OK : GP_E_INVAL;
}

static VariantMap map_at(int vi, uint64_t base) {
    VariantMap m;
    m.slot = variant_slots(vi);
    m.base = base;
    m.ready = true;
    return m;
}

constexpr int kCodePadding = 32;   // words

// Operands of a tree that lie in LDS and are pushed by a record of their own.
static int64_t pushes_of_features(const uint32_t* w, int64_t n, const CoreVariantDesc& v, const RowPlan& rows) {
    int64_t k = 0;
    for (int64_t i = 0; i < n; i++) {
        const uint32_t w0 = w[2 * i], op = w0 & 15u, mode = (w0 >> 4) & 15u;
        const int fa = (int)((w0 >> 8) & 255u), fb = (int)((w0 >> 16) & 255u);
        if (op == OP_IF) continue;
        if (mode == M_XS || mode == M_XC || mode == M_XX) k += fa >= v.nf;
        if (mode == M_SX || mode == M_CX || mode == M_XX) k += fb >= v.nf;
        if (mode == M_X && op != OP_PUSH) k += fa >= v.nf && rows.row[row_key(op, fa)] < 0;
    }
    return k;
}

// Programs are translated in parallel, each into its own counted range of
// the code: a tree gives one core instruction per lowered instruction plus
// the end (and one for each operand that lies in LDS); a register program as linear_records counts.  The code holds the
// programs one after another in the order given (null: their own order), each
// ending with the length of the one after it; progs[p] says where program p
// lies.  With `rows`, functions of a feature that have a row push it, and the
// programs that compute the rows follow the others, a share for every wave of a
// block: two records each, three if the feature is loaded first.
static gp_status translate_with(const ProgData& pd, int vi, const VariantMap& m, const uint32_t* order, RowPlan* rows,
                                RawWords& code, std::vector<DevProg>& progs) {
    const int32_t P = pd.n_prog;
    progs = pd.progs;
    RowPlan features;
    // (other kernels have no place for a feature beyond their slots: its offset is written as it comes, and an
    // evaluation never takes such a kernel)
    const CoreVariantDesc& v = kCoreVariants[vi];
    const bool in_lds = v.cap > v.nf && pd.n_load > v.nf;
    if (in_lds && pd.n_load > v.cap)
        return fail(GP_E_INVAL, "variant %d takes %d features, the programs read %d", vi, v.cap, pd.n_load);
    if (in_lds && !rows) {
        no_rows(pd, vi, features);
        rows = &features;
    }
    std::vector<int64_t> start((size_t)P + 1, 0);
    auto at = [&](int32_t i) { return order ? (int32_t)order[i] : i; };
    auto records = [&](int32_t p) {
        const DevProg& src = pd.progs[p];
        if ((src.meta & 1u) == FORM_TREE)
            return (int64_t)src.len + 1 +
                   (in_lds ? pushes_of_features(pd.code.data() + src.code_off, src.len, v, *rows) : 0);
        return linear_records(pd.code.data() + src.code_off, src.len, src.live);
    };
    for (int32_t i = 0; i < P; i++) start[i + 1] = start[i] + records(at(i));
    const int32_t R = rows ? rows->n() : 0;
    if ((start[P] + 3 * R) * 16 > 0xFFFFFFF0ll) return fail(GP_E_INVAL, "programs exceed 4 GiB of core code");
    // the core reads records two or four at a time, ahead of the one it runs: up
    // to seven past a program's last one, so the code ends with padding
    code.resize((size_t)(start[P] + 3 * R) * 4 + kCodePadding);
    std::fill(code.begin() + 4 * start[P], code.end(), 0u);
    if (rows) {
        // wave w computes rows w, w + W, ...
        auto length = [&](int32_t r) { return rows->op[r] != OP_PUSH && rows->feat[r] >= v.nf ? 3 : 2; };
        int64_t at_rec = start[P];
        char err[256];
        rows->rec.clear();
        for (int32_t w = 0; w < v.waves; w++) {
            rows->rec.push_back((uint32_t)at_rec);
            for (int32_t r = w; r < R; r += v.waves) {
                const int n = length(r), f = rows->feat[r], next = r + v.waves < R ? length(r + v.waves) : 0;
                Emitter e{v, m, code.data() + 4 * at_rec, n, err};
                if (f >= v.nf) e.load(f);
                if (rows->op[r] != OP_PUSH)
                    e.exit(rows->op[r], f >= v.nf ? 0 : (core_reg_levels(vi) + f) * v.t, 0, 0, false, false, 0);
                e.end((uint32_t)r, (uint32_t)next);
                if (!e.ok || e.n != n) return fail(GP_E_INVAL, "row %d: %s", r, e.ok ? "length" : err);
                at_rec += n;
            }
        }
        rows->rec.push_back((uint32_t)at_rec);
    }
    std::vector<int32_t> rc((size_t)P, GP_OK);
    auto translate = [&](int32_t i, uint32_t* out, int64_t cap, int64_t* n, char* err) {
        const int32_t p = at(i);
        const DevProg& src = pd.progs[p];
        const uint32_t next = i + 1 < P ? (uint32_t)(start[i + 2] - start[i + 1]) : 0u;
        const uint32_t* w = pd.code.data() + src.code_off;
        if ((src.meta & 1u) == FORM_TREE)
            return translate_tree(w, src.len, vi, m, rows, (uint32_t)src.row, next, out, cap, n, err);
        return translate_linear(w, src.len, src.live, w + src.len, pd.n_reg, pd.n_feat, vi, m, (uint32_t)src.row, next, out, cap,
                                n, err);
    };
    parallel_for(P, [&](int64_t i0, int64_t i1) {
        char err[256];
        for (int64_t i = i0; i < i1; i++) {
            const int64_t cap = start[i + 1] - start[i];
            int64_t n = 0;
            rc[i] = translate((int32_t)i, code.data() + 4 * start[i], cap, &n, err);
            if (rc[i] == GP_OK && n != cap) rc[i] = GP_E_INVAL;
        }
    });
    for (int32_t i = 0; i < P; i++) {
        const int32_t p = at(i);
        if (rc[i] != GP_OK) {
            // translate the first failing program again on this thread for its message
            std::vector<uint32_t> tmp(4 * (size_t)(start[i + 1] - start[i] + 8));
            char err[256] = "internal: core code length differs from its count";
            int64_t n = 0;
            translate(i, tmp.data(), (int64_t)tmp.size() / 4, &n, err);
            return fail((gp_status)rc[i], "program %d: %s", p, err);
        }
        progs[p].code_off = (uint32_t)(4 * start[i]);   // words
        progs[p].len = (uint32_t)(start[i + 1] - start[i]);
    }
    return GP_OK;
}

// The rows worth computing: those used by at least one and a half programs
// for each block that computes them (over the fewest groups the programs are
// cut into), the most used first, as many as the LDS beside the resident
// blocks holds.  Whether a launch then uses them is another question
// (runtime.cpp, translation_for).  A row costs a block one evaluation a tile, by one of its
// waves; a use then reads 16 bytes a lane instead of evaluating the function
// again (about 90 vector instructions at T = 4).
static constexpr uint32_t kRowSaving = 33;   // of the cost of one use (runtime.cpp, op_cost)

void no_rows(const ProgData& pd, int vi, RowPlan& plan) {
    plan = RowPlan();
    plan.cost = pd.cost;
    plan.sum();
    const CoreVariantDesc& v = kCoreVariants[vi];
    if (pd.n_load <= v.nf) return;
    plan.row.assign(4 * GP_MAX_FEAT, -1);
    plan.first_lds = v.nf;
    for (int f = v.nf; f < pd.n_load; f++) {
        plan.op.push_back(OP_PUSH);
        plan.feat.push_back(f);
    }
}

void plan_rows(const ProgData& pd, int vi, int64_t blocks, RowPlan& plan) {
    no_rows(pd, vi, plan);
    const CoreVariantDesc& v = kCoreVariants[vi];
    if (v.rows_base == 0 || pd.form != FORM_TREE || pd.n_transc == 0 || pd.n_load > GP_MAX_FEAT) return;
    if (2 * pd.n_transc < 3 * blocks) return;
    std::vector<int64_t> uses(4 * GP_MAX_FEAT, 0);
    auto each = [&](const DevProg& p, auto&& fn) {
        const uint32_t* w = pd.code.data() + p.code_off;
        for (uint32_t i = 0; i < p.len; i++) {
            const uint32_t op = w[2 * i] & 15u, mode = (w[2 * i] >> 4) & 15u;
            if (mode == M_X && op >= GP_SIN && op <= GP_PLOG) fn(row_key(op, (int)((w[2 * i] >> 8) & 255u)));
        }
    };
    // (a short walk takes less time than waking the host threads)
    auto walk = [&](const std::function<void(int64_t, int64_t)>& fn) {
        if (pd.n_instr < (int64_t)1 << 15) fn(0, (int64_t)pd.progs.size());
        else parallel_for((int64_t)pd.progs.size(), fn);
    };
    std::mutex mu;
    walk([&](int64_t i0, int64_t i1) {
        std::vector<int32_t> part(uses.size(), 0);
        for (int64_t i = i0; i < i1; i++) each(pd.progs[i], [&](int k) { part[k]++; });
        std::lock_guard<std::mutex> g(mu);
        for (size_t k = 0; k < uses.size(); k++) uses[k] += part[k];
    });
    const int per_cu = std::max(1, 4 * core_variant_simd(vi) / v.waves);
    // (a block's LDS is given in parts of 1280 bytes, 128 a CU: a third of all the bytes does not fit three times, and
    // 1148 programs over 21 features then took 2.24 ms x 383000 cases, not 1.72)
    const int have = plan.n(), most = (128 / per_cu * 1280 - v.rows_base) / (256 * v.t) - have;
    std::vector<int> keys;
    for (int k = 0; k < (int)uses.size(); k++)
        if (2 * uses[k] >= 3 * std::max<int64_t>(2, blocks)) keys.push_back(k);
    std::stable_sort(keys.begin(), keys.end(), [&](int a, int b) { return uses[a] > uses[b]; });
    if ((int)keys.size() > most) keys.resize(std::max(0, most));
    if (keys.empty()) return;
    plan.row.assign(uses.size(), -1);
    for (size_t r = 0; r < keys.size(); r++) {
        plan.row[keys[r]] = have + (int32_t)r;
        plan.op.push_back(GP_SIN + (uint32_t)(keys[r] / GP_MAX_FEAT));
        plan.feat.push_back(keys[r] % GP_MAX_FEAT);
    }
    walk([&](int64_t i0, int64_t i1) {
        for (int64_t i = i0; i < i1; i++)
            each(pd.progs[i], [&](int k) { if (plan.row[k] >= 0) plan.cost[i] -= std::min(plan.cost[i] - 1, kRowSaving); });
    });
    plan.sum();
}

gp_status core_translate(const ProgData& pd, int vi, const uint32_t* order, RowPlan* rows, RawWords& code,
                         std::vector<DevProg>& progs) {
    std::shared_ptr<const VariantMap> m;
    {
        std::lock_guard<std::mutex> g(g_mu);
        if ((int)g_maps.size() > vi) m = g_maps[vi];
    }
    if (!m) return fail(GP_E_DEVICE, "core variant %d not probed", vi);
    return translate_with(pd, vi, *m, order, rows, code, progs);
}

gp_status core_translate_at(const ProgData& pd, int vi, uint64_t base, RawWords& code,
                            std::vector<DevProg>& progs) {
    if (vi < 0 || vi >= core_variants()) return fail(GP_E_INVAL, "variant %d does not exist", vi);
    if (base & (GPX_SLOT - 1)) return fail(GP_E_INVAL, "table base must be %d-byte aligned", GPX_SLOT);
    return translate_with(pd, vi, map_at(vi, base), nullptr, nullptr, code, progs);
}

int core_variant_waves(int vi) { return kCoreVariants[vi].waves; }
int core_variant_simd(int vi) {
    const CoreVariantDesc& v = kCoreVariants[vi];
    return std::max(1, 512 / ((v.ncv + (core_reg_levels(vi) + v.nf) * v.t + 7) / 8 * 8));
}
int core_variant_t(int vi) { return kCoreVariants[vi].t; }
int core_variant_ncv(int vi) { return kCoreVariants[vi].ncv; }
int core_variant_d(int vi) { return kCoreVariants[vi].d; }
int core_variant_nf(int vi) { return kCoreVariants[vi].nf; }
int core_variant_cap(int vi) { return kCoreVariants[vi].cap; }
bool core_variant_fits(int vi, const ProgData& pd) {
    const CoreVariantDesc& v = kCoreVariants[vi];
    // (an operand that is pushed takes the level above)
    return v.cap >= pd.n_load && v.d >= pd.max_depth + (pd.n_load > v.nf) && !(mode_no_transc(v.arith) && pd.n_transc > 0) &&
           (v.arith == 2) == (pd.opset == OPSET_BOOL) && !(v.arith >= 2 && pd.form != FORM_TREE);
}
std::string core_variant_name(int vi) {
    const CoreVariantDesc& v = kCoreVariants[vi];
    static const char* const suffix[] = {"", "_a", "_b", "_at", "_t"};
    char s[64];
    snprintf(s, sizeof s, "k_core_%d_%d_%d_%d%s", v.t, v.d, v.nf, v.ncv, suffix[v.arith]);
    return s;
}
int core_variant_named(const std::string& name) {
    for (int i = 0; i < core_variants(); i++)
        if (core_variant_name(i) == name) return i;
    return -1;
}
int core_variant_arith(int vi) { return mode_no_transc(kCoreVariants[vi].arith); }
bool core_variant_bool(int vi) { return kCoreVariants[vi].arith == 2; }
bool core_variant_trees_only(int vi) { return kCoreVariants[vi].arith >= 2; }

}  // namespace gpx
