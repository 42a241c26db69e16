// The register-resident solver of the small levels (resident.hip).
#pragma once

#include "common.h"

namespace mls {

// true when the launch shape of level l is the library's own choice there,
// h = 1/8 .. 1/64 at V(1,1): nothing set by the caller, or the general
// solver's default block named and everything else left to the library
bool resident_level(const mls2mc_ctx* ctx, int l);
// that default block: the autotuner's name for the resident solver
int resident_token(const mls2mc_ctx* ctx, int l);
// one batch on one level; the caller has checked resident_level
int launch_resident(mls2mc_ctx* ctx, const SolveArgs& a, hipStream_t s);
// the particles of several work items of one level l (items_dev: bases set,
// total = the sum of their N)
int launch_resident_list(mls2mc_ctx* ctx, int l, const SolveItem* items_dev, int n_items, int64_t total, bool mixed,
                         hipStream_t s);

}  // namespace mls
