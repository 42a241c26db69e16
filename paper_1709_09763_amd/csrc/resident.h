// The register-resident solvers of the small levels (resident.hip) and of
// h = 1/128 (resident7.hip).
#pragma once

#include "common.h"

namespace mls {

// true when the launch shape of level l is the library's own choice there,
// h = 1/8 .. 1/64, and h = 1/128 where resident7_runs, at V(1,1): nothing set
// by the caller, or the general solver's default block named and everything
// else left to the library
bool resident_level(const mls2mc_ctx* ctx, int l);
// what a launch over `total` particles of level l takes of ctx->ws_solver
size_t resident_workspace(const mls2mc_ctx* ctx, int l, int64_t total);
// that default block: the autotuner's name for the resident solver
int resident_token(const mls2mc_ctx* ctx, int l);
// one batch on one level; the caller has checked resident_level
int launch_resident(mls2mc_ctx* ctx, const SolveArgs& a, hipStream_t s);
// the particles of several work items of one level l (items_dev: bases set,
// total = the sum of their N)
int launch_resident_list(mls2mc_ctx* ctx, int l, const SolveItem* items_dev, int n_items, int64_t total, bool mixed,
                         hipStream_t s);

// h = 1/128: the FP64 Dirichlet problem with up to 128 observations
bool resident7_runs(const mls2mc_ctx* ctx);
size_t resident7_workspace(const mls2mc_ctx* ctx, int64_t total);
int launch_resident7(mls2mc_ctx* ctx, const SolveArgs& a, int32_t* iters, hipStream_t s);
int launch_resident7_list(mls2mc_ctx* ctx, const SolveItem* items_dev, int n_items, int64_t total, hipStream_t s);

}  // namespace mls
