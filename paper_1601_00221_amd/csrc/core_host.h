// Host side of the interpreter core (core_host.cpp).
#pragma once

#include <hip/hip_runtime_api.h>
#include <stdint.h>

#include <string>
#include <vector>

#include "../../include/gp.h"
#include "gp_internal.h"
#include "runtime.h"

namespace gpx {

int core_variants();
int core_variant_t(int vi);        // case slots per lane
int core_variant_d(int vi);        // stack levels
int core_variant_nf(int vi);       // features in registers
int core_variant_cap(int vi);      // features it takes: more than nf where the others lie in LDS (eval_core only)
bool core_variant_fits(int vi, const ProgData& pd);   // features, depth, functions and form
int core_variant_arith(int vi);    // 1: no sin/cos/exp/log code
bool core_variant_bool(int vi);    // the Boolean function set (32-bit word slots)
bool core_variant_trees_only(int vi);   // no linear handlers (Boolean and trees-only arithmetic kernels)
int core_variant_ncv(int vi);      // VGPRs left to the compiled code
std::string core_variant_name(int vi);            // of its kernel
int core_variant_named(const std::string& name);  // -1: none
int core_reg_levels(int vi);       // register/stack levels before the features
// Variant for programs reading n_load features, needing `depth` stack levels,
// with a fraction transc_frac of sin/cos/exp/log instructions (has_transc:
// any at all), of the Boolean function set if `boolean`, and trees only if
// `trees_only` (then a kernel without linear handlers may be taken); -1 if
// none fits.
int pick_core_variant(int n_load, int depth, double transc_frac, bool has_transc, bool boolean = false,
                      bool trees_only = false, bool wide = false);
// Locate the variant's handler table on the current device (one probe launch
// on stream s the first time).
gp_status core_ready(int vi, hipStream_t s);
// True if core_ready has found variant vi's handler table on the current device.
bool core_is_ready(int vi);
int core_variant_waves(int vi);     // of a block
int core_variant_simd(int vi);      // waves that a SIMD holds
// No function has a row: the features that variant vi holds in LDS alone, and the programs' costs as they are.
void no_rows(const ProgData& pd, int vi, RowPlan& plan);
// Which functions of a feature a launch computes once a tile into LDS, for variant vi, where `blocks` blocks share a
// tile's programs; and the programs' costs without them.
void plan_rows(const ProgData& pd, int vi, int64_t blocks, RowPlan& plan);
// Core instructions of lowered programs, one program after another in the
// given order (null: their own), and where each one lies.  rows (may be null)
// is read, and told where the rows' programs lie.
gp_status core_translate(const ProgData& pd, int vi, const uint32_t* order, RowPlan* rows, RawWords& code,
                         std::vector<DevProg>& progs);
// The same with the handler table taken to start at `base` (no device needed).
gp_status core_translate_at(const ProgData& pd, int vi, uint64_t base, RawWords& code,
                            std::vector<DevProg>& progs);

}  // namespace gpx
