// Register-resident multigrid-PCG at h = 1/128, FP64 Dirichlet problem.  The
// method is solver.hip's (same cycle, the finest level's V-cycle weights
// rounded to FP32 as there); resident.hip explains strips and colours.
//
// What bounds the level: 16384 unknowns are four times what resident.hip's
// layout holds next to its weights, and in the general solver every pass of
// an iteration reads its vectors through the caches.  Here a workgroup of
// 512 threads holds a particle: each thread sixteen rows of two neighbouring
// columns (a wave: sixteen whole rows), with r and the search direction in
// registers throughout and z in registers from the up-leg to the stencil
// pass.  What is left to read are weights, and they are streamed: the FP32
// edges (kLdsRows rows of each strip from the LDS) and FP64 inverse diagonals
// of the V-cycle and the h = 1/64 level's weights from a slot of the
// workgroup's own, the FP64 edges of the stencil pass formed from the
// coefficients themselves - 1.1 MB an iteration, which 256 workgroups draw
// from the memory-side cache.
//
// Measured (us for 1 / 256 / 1000 particles, 13.7 iterations): general solver
// 1833 / 2739 / 10338, here 345 / 633 / 2311: 22 us an iteration where one
// particle runs alone (its instructions and barriers), 40 where the weights
// of 256 are streamed.  Otherwise: 1024 threads of eight rows 482 / 869 / 3313
// (128 registers: 45 values a thread and iteration spilled, against 14 at 512
// threads); nine rows of edges in the LDS instead of ten 350 / 641 / 2350;
// nontemporal loads of the coefficients 356 / 726 / 2698; the h = 1/64 weights
// held through the visit of h = 1/32 362 / 697 / 2523.
//
// The V-cycle is cycle7 of strips7.h, which explains the layout.
//
// The solution is not kept: the thread that owns an observation's node adds
// alpha p there (so launches that ask for the field, and those with more
// observations than the LDS list holds, stay with the general solver).
#include <algorithm>

#include "resident.h"
#include "strips7.h"

namespace mls {

namespace {

constexpr int kN = 128, kNT = 512, kR = kRows7<kNT>;  // nodes per side, threads, rows per thread
constexpr int kObs = 128;                             // observations that the LDS list holds
constexpr int kLdsRows = 10;                          // rows of each strip whose FP32 edges stay in the LDS

struct Mem7 {
    Exchange7<double, kNT> x;
    float4 e[kLdsRows][kNT];  // set-up: the h = 1/64 coefficients
    Levels5<double> low;
    double red[2][16];
    double obsx[3 * kObs];          // the solution at the observations' nodes
    unsigned short node[3 * kObs];  // where an observation's node is in obsx (0xffff: on the boundary)
    int64_t draw;
};
static_assert(sizeof(float4) * kLdsRows * kNT >= sizeof(double) * 2 * 64 * 64, "the h = 1/64 coefficients fit in e");

// The workgroup's slot: a part per wave, so that a lane reaches all of its
// values with immediate offsets.  In doubles: edges [row][lane], 16 bytes each;
// inverse diagonals [row pair][colour][lane], two rows each; h = 1/64 weights
constexpr int kWaveInv = (kR - kLdsRows) * 64 * 2;
constexpr int kWaveC6 = kWaveInv + 2 * kR * 64;
constexpr int kWave = kWaveC6 + kW * (kR / 4) * 64;
constexpr int64_t kSlot = (int64_t)kWave * (kNT / 64);

struct Params7 {
    int64_t N;
    const int64_t* N_dev;
    const double* kappa;
    double* ws;
    double* G;
    int8_t* status;
    int32_t* iters;
    const double* y;
    double* phi;
    const SolveItem* items;  // null: one batch; else the particles of several items
    int n_items;
    const int32_t* obs_idx;
    const double* obs_w;
    int nobs;
    double inv_sigma, tol2;
    int max_iters;
    unsigned long long* queue;
};

__global__ __launch_bounds__(kNT) __attribute__((amdgpu_waves_per_eu(2))) void resident7_kernel(Params7 A)
{
    __shared__ __align__(16) Mem7 m;
    const int t0 = threadIdx.x;
    const int wv = __builtin_amdgcn_readfirstlane(t0 >> 6);
    constexpr int n = kN;
    double* a0 = m.x.rs6 + kNT;
    double* a3 = m.x.rs6;
    double* slot = A.ws + blockIdx.x * kSlot + wv * kWave;
    float4* eg = reinterpret_cast<float4*>(slot);
    double* w6 = slot + kWaveC6;

    // the thread's nodes that observations read: a bit per node (row * 2 +
    // column), their first place in obsx; wave_obs: bits of any lane
    unsigned own_obs, wave_obs = 0;
    int obs_at = 0;
    {
        const int t = t0;
        unsigned* bits = reinterpret_cast<unsigned*>(m.x.a1);
        int* at = reinterpret_cast<int*>(m.x.a2);
        int* count = at + kNT;
        bits[t] = 0;
        if (t == 0) *count = 0;
        group_order();
        auto owner = [&](int q, int& u, int& bit) -> bool {
            const int idx = A.obs_idx[q], i = idx % (n + 1), j = idx / (n + 1);
            u = (j / kR) * 64 + (i >> 1);
            bit = (j % kR) << 1 | (i & 1);
            return i > 0 && i < n && j > 0 && j < n;
        };
        int u, bit;
        for (int q = t; q < 3 * A.nobs; q += kNT)
            if (owner(q, u, bit)) atomicOr(&bits[u], 1u << bit);
        group_order();
        own_obs = bits[t];
        if (own_obs) at[t] = obs_at = atomicAdd(count, __popc(own_obs));
        group_order();
        for (int q = t; q < 3 * A.nobs; q += kNT)
            m.node[q] = owner(q, u, bit) ? at[u] + __popc(bits[u] & ((1u << bit) - 1)) : 0xffff;
#pragma unroll
        for (int k = 0; k < 2 * kR; ++k)
            if (__any(own_obs >> k & 1)) wave_obs |= 1u << k;
        group_order();
    }

    const int64_t NN = A.N_dev ? min(A.N, *A.N_dev) : A.N;
    auto draw = [&]() -> int64_t {
        if (threadIdx.x == 0) m.draw = (int64_t)atomicAdd(A.queue, 1ull);
        group_order();
        const int64_t v = m.draw;
        group_order();
        return v;
    };
    for (int64_t q = draw(); q < NN; q = draw()) {
        const int t = again(t0), lane = t & 63;
        const double* kappa = A.kappa;
        double *Gq = A.G, *phi = A.phi;
        const double* y = A.y;
        int8_t* status = A.status;
        int32_t* iters = A.iters;
        int64_t qi = q;
        if (A.items) {
            int lo = 0, hi = A.n_items - 1;  // last item with base <= q
            while (lo < hi) {
                const int mid = (lo + hi + 1) >> 1;
                if (A.items[mid].base <= q) lo = mid; else hi = mid - 1;
            }
            const SolveItem& it = A.items[lo];
            qi -= it.base;
            kappa = (const double*)it.kappa; Gq = it.G; phi = it.phi; y = it.y; status = it.status; iters = it.iters;
        }
        const double* kap = kappa + qi * (int64_t)(2 * n * n);
        Gq += qi * A.nobs;
        const double* kw = kap + (int64_t)(kR * wv) * (2 * n);  // the wave's first row; four values per lane and row

        // ---- set-up
        auto fine_cell = [&](int ci, int cj, double& lo, double& up) {
            const double* c = kap + 2 * (cj * n + ci);
            lo = c[0];
            up = c[1];
        };
        double* k6 = reinterpret_cast<double*>(m.e);
        double* k5 = m.x.rs6;
        coarsen<double, 6, kNT>(k6, t, fine_cell);
        auto clear = [&](double* a, int c) { for (int k = t; k < c; k += kNT) a[k] = 0.0; };
        clear(m.obsx, 3 * A.nobs);
        group_order();
        weights6<double, kNT>(w6, k6, t);
        coarsen<double, 5, kNT>(k5, t, [&](int ci, int cj, double& lo, double& up) {
            lo = k6[2 * (cj * 64 + ci)];
            up = k6[2 * (cj * 64 + ci) + 1];
        });
        group_order();
        build_levels5(m.low, k5, t);
        // the finest level's V-cycle weights: FP32 edges x (a - b), y (b - east
        // a), z (a, to the row above), w (b, to the row above); FP64 inverse
        // diagonals of rows k, k + 1 in one pair: [k / 2][colour]
        {
            double ua0 = 0.0, ub0 = 0.0;  // upper triangles of the row below
            float va0 = 0.f, vb0 = 0.f;   // vertical edges from the row below
            if (wv > 0) {
                const double* c = kw - 2 * n + 4 * lane;
                ua0 = c[1];
                ub0 = c[3];
                va0 = (float)(0.5 * (ua0 + west(c[2])));
                vb0 = (float)(0.5 * (ub0 + c[0]));
            }
            double ir0 = 0.0, ib0 = 0.0;
#pragma unroll
            for (int k = 0; k < kR; ++k) {
                const double* c = kw + k * (2 * n) + 4 * lane;
                const double la = c[0], ua = c[1], lb = c[2], ub = c[3];
                float4 w;
                w.x = (float)(0.5 * (la + ua0));
                w.y = (float)(0.5 * (lb + ub0));
                w.z = (float)(0.5 * (ua + west(lb)));
                w.w = (float)(0.5 * (ub + la));
                const double da = (double)west(w.y) + (double)w.x + (double)w.z + (double)va0;
                const double db = (double)w.x + (double)w.y + (double)w.w + (double)vb0;
                const bool in = wv > 0 || k > 0;
                const double ia = in && lane > 0 ? 1.0 / da : 0.0, ib = in ? 1.0 / db : 0.0;
                if (k < kLdsRows) {
                    // over the h = 1/64 coefficients, dead since the barrier above
                    m.e[k < kLdsRows ? k : 0][t] = w;
                } else {
                    eg[(k - kLdsRows) * 64 + lane] = w;
                }
                const double ir = k & 1 ? ib : ia, ibk = k & 1 ? ia : ib;
                if (k & 1) {
                    double* d = slot + kWaveInv + (k >> 1) * 256 + 2 * lane;
                    d[0] = ir0; d[1] = ir;
                    d[128] = ib0; d[129] = ibk;
                }
                ir0 = ir;
                ib0 = ibk;
                ua0 = ua; ub0 = ub; va0 = w.z; vb0 = w.w;
            }
        }
        group_order();
        // also the exchange, out of the coefficients' use
        clear(m.x.pad, sizeof(m.x) / 8);
        clear_levels5<double, kNT>(m.low, t);
        group_order();

        auto edge = [&](int k, int u) -> float4 {
            return k < kLdsRows ? m.e[k < kLdsRows ? k : 0][u] : eg[(k - kLdsRows) * 64 + (u & 63)];
        };
        auto inv = [&](int k, int c, int u) -> double {
            return slot[kWaveInv + (k >> 1) * 256 + c * 128 + (k & 1) + 2 * (u & 63)];
        };
        auto total = [&](double v, int which) -> double {
            v = lane63_sum(v);
            if ((t0 & 63) == 63) m.red[which][wv] = v;
            group_order();
            double s = 0.0;
#pragma unroll
            for (int k = 0; k < kNT / 64; ++k) s += m.red[which][k];
            return read_lane(s, 0);
        };
        // ---- state
        double rr[kR], rb[kR], pr[kR], pb[kR], zr[kR], zb[kR];
        const double h2 = 1.0 / (double)(n * n);
#pragma unroll
        for (int k = 0; k < kR; ++k) {
            const bool in = wv > 0 || k > 0;
            const double va = in && lane > 0 ? h2 : 0.0, vb = in ? h2 : 0.0;
            rr[k] = k & 1 ? vb : va;
            rb[k] = k & 1 ? va : vb;
            pr[k] = pb[k] = 0.0;
        }

        auto vcycle = [&]() -> double {
            cycle7<double, kNT>(rr, rb, zr, zb, edge, inv, w6, m.x, m.low, t0, wv);
            double d = 0.0;
#pragma unroll
            for (int k = 0; k < kR; ++k) d += rr[k] * zr[k] + rb[k] * zb[k];
            return total(d, 1);
        };

        // ---- PCG; one copy of the cycle serves the first direction too
        double rz = 0.0, rz0 = 0.0, beta = 0.0;
        int it = 0;
        int8_t st = 1;
        bool first = true;
        while (true) {
            const double v = vcycle();
            if (first) {
                rz0 = v;
                if (!(v > 0.0) || !isfinite(v)) { st = 2; break; }
            } else {
                ++it;
                if (!isfinite(v)) { st = 2; break; }
                if (v <= A.tol2 * rz0) { st = 0; break; }
                beta = v / rz;
            }
            rz = v;
            first = false;
            if (it >= A.max_iters) break;
            // p = z + beta p, and q = A p in z's registers: the sum of the
            // edges' fluxes w (p_c - p_nb), edges from the coefficients
#pragma unroll
            for (int k = 0; k < kR; ++k) {
                pr[k] = zr[k] + beta * pr[k];
                pb[k] = zb[k] + beta * pb[k];
            }
            // the last row's column b is red, row 0's column a
            const int t = again(t0), lane = t & 63;
            a0[t] = pr[kR - 1];
            m.x.a2[t] = pb[kR - 1];
            m.x.a1[t] = pr[0];
            a3[t] = pb[0];
            group_order();
            double pq = 0.0;
            {
                double ua0 = 0.0, ub0 = 0.0, fa = 0.0, fb = 0.0;
                if (wv > 0) {
                    const double* c = kw - 2 * n + 4 * lane;
                    ua0 = c[1];
                    ub0 = c[3];
                    fa = 0.5 * (ua0 + west(c[2])) * (m.x.a2[t - 64] - pr[0]);
                    fb = 0.5 * (ub0 + c[0]) * (a0[t - 64] - pb[0]);
                }
                const double upa = wv < kNT / 64 - 1 ? m.x.a1[t + 64] : 0.0, upb = wv < kNT / 64 - 1 ? a3[t + 64] : 0.0;
                double cell[kR][4];
                auto load = [&](int k) {
                    const double* c = kw + k * (2 * n) + 4 * lane;
#pragma unroll
                    for (int h = 0; h < 4; ++h) cell[k][h] = c[h];
                };
#pragma unroll
                for (int k = 0; k < kAhead; ++k) load(k);
#pragma unroll
                for (int k = 0; k < kR; ++k) {
                    if (k + kAhead < kR) load(k + kAhead);
                    const double la = cell[k][0], ua = cell[k][1], lb = cell[k][2], ub = cell[k][3];
                    const double pa = k & 1 ? pb[k] : pr[k], pc = k & 1 ? pr[k] : pb[k];
                    const int k1 = k + 1 < kR ? k + 1 : 0;
                    const double na = k + 1 < kR ? (k1 & 1 ? pb[k1] : pr[k1]) : upa;
                    const double nc = k + 1 < kR ? (k1 & 1 ? pr[k1] : pb[k1]) : upb;
                    const double fx = 0.5 * (la + ua0) * (pa - pc);
                    const double fe = 0.5 * (lb + ub0) * (pc - east(pa));
                    const double ga = 0.5 * (ua + west(lb)) * (pa - na);
                    const double gb = 0.5 * (ub + la) * (pc - nc);
                    const double qa = (fx - west(fe)) + (ga - fa), qc = (fe - fx) + (gb - fb);
                    zr[k] = k & 1 ? qc : qa;
                    zb[k] = k & 1 ? qa : qc;
                    pq += pa * qa + pc * qc;
                    ua0 = ua; ub0 = ub; fa = ga; fb = gb;
                }
            }
            pq = total(pq, 0);
            const double alpha = rz / pq;
#pragma unroll
            for (int k = 0; k < kR; ++k) {
                rr[k] -= alpha * zr[k];
                rb[k] -= alpha * zb[k];
            }
            if (wave_obs) {
                const unsigned mine = again(own_obs);
#pragma unroll
                for (int k = 0; k < 2 * kR; ++k)
                    if (wave_obs >> k & 1) {
                        const int r = k >> 1;
                        const double p = (k ^ r) & 1 ? pb[r] : pr[r];
                        if (mine >> k & 1) m.obsx[obs_at + __popc(mine & ((1u << k) - 1))] += alpha * p;
                    }
            }
        }

        // ---- observations, potential
        group_order();
        double ph = 0.0;
        for (int o = t; o < A.nobs; o += kNT) {
            double g = 0.0;
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const int at = m.node[3 * o + k];
                g += A.obs_w[3 * o + k] * (at != 0xffff ? m.obsx[at] : 0.0);
            }
            Gq[o] = g;
            if (y) {
                const double r = (y[o] - g) * A.inv_sigma;
                ph += r * r;
            }
        }
        if (y) ph = total(ph, 0);
        if (t == 0) {
            if (status) status[qi] = st;
            if (iters) iters[qi] = it;
            if (phi) phi[qi] = 0.5 * ph;
        }
        group_order();
    }
    // every workgroup has drawn past the end; the last one to finish resets
    // the counter for the next launch on this context
    if (t0 == 0) {
        __threadfence();
        if (atomicAdd(A.queue + 1, 1ull) == (unsigned long long)(gridDim.x - 1)) {
            atomicExch(A.queue, 0ull);
            atomicExch(A.queue + 1, 0ull);
        }
    }
}

int64_t grid7(const mls2mc_ctx* ctx, int64_t total) { return std::min<int64_t>(total, ctx->n_cu); }

int launch_params7(mls2mc_ctx* ctx, Params7& A, hipStream_t s)
{
    const int64_t grid = grid7(ctx, A.N);
    MLS_TRY(ctx->ws_solver.ensure(resident7_workspace(ctx, A.N)));
    A.ws = ctx->ws_solver.as<double>();
    A.queue = ctx->d_queue;
    A.obs_idx = ctx->obs[7].idx;
    A.obs_w = ctx->obs[7].w;
    A.nobs = ctx->nobs;
    A.inv_sigma = 1.0 / ctx->prob.sigma_n;
    A.tol2 = ctx->rtol * ctx->rtol;
    A.max_iters = ctx->max_iters;
    resident7_kernel<<<(unsigned)grid, kNT, 0, s>>>(A);
    MLS_CHECK_HIP(hipGetLastError());
    return MLS2MC_OK;
}

}  // namespace

bool resident7_runs(const mls2mc_ctx* ctx)
{
    return ctx->prob.bc != MLS2MC_BC_FLOW_CELL && ctx->prob.precision != MLS2MC_MIXED && ctx->nobs <= kObs &&
           ctx->max_lds + 1024 >= (int)sizeof(Mem7);
}

size_t resident7_workspace(const mls2mc_ctx* ctx, int64_t total)
{
    return (size_t)grid7(ctx, total) * kSlot * sizeof(double);
}

int launch_resident7(mls2mc_ctx* ctx, const SolveArgs& a, int32_t* iters, hipStream_t s)
{
    Params7 A = {};
    A.N = a.N; A.N_dev = a.N_dev; A.kappa = (const double*)a.kappa; A.G = a.G;
    A.status = a.status; A.iters = iters; A.y = a.y; A.phi = a.phi;
    return launch_params7(ctx, A, s);
}

int launch_resident7_list(mls2mc_ctx* ctx, const SolveItem* items_dev, int n_items, int64_t total, hipStream_t s)
{
    Params7 A = {};
    A.N = total;
    A.items = items_dev;
    A.n_items = n_items;
    return launch_params7(ctx, A, s);
}

}  // namespace mls
