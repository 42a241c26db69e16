// Register-resident multigrid-PCG for the small levels, h = 1/8 .. 1/64, of
// the Dirichlet problem and of the flow cell (Sec. 5; Example 5.3), FP64 and
// mixed.  The discretisation, the V(1,1) cycle, the stopping rule and the
// observations are those of solver.hip and flowcell.hip; what differs is
// where a particle lives.
//
// What bounds these levels: not memory (a particle's coefficients are 4 KB at
// h = 1/16 and 64 KB at h = 1/64, read once) but the serial chain of passes
// of a PCG iteration, each ending in a workgroup barrier.  With the arrays in
// LDS or in a global slot every pass reads five values and four weights per
// node through the LDS or the caches.  Here one thread owns a strip of 2 P
// nodes of one column and keeps their r, z, p, x and edge weights in
// registers for the whole solve:
//
//  * horizontal neighbours are the adjacent lanes (a wave holds whole rows of
//    strips), so their values come by a one-lane DPP shift;
//  * vertical neighbours are the thread's own registers, except one value per
//    thread and pass from the strip above or below, through one LDS row;
//  * nodes are held by colour: with e = i mod 2, R[k] is row 2k + e and B[k]
//    row 2k + 1 - e of the strip's row pairs.  Every lane then has one red
//    and one black node per pair, so no lane idles in a colour sweep; the
//    horizontal neighbours of R[k] are B[k] of the adjacent lanes, its
//    vertical ones the own B[k] and B[k-1] (even lanes) or B[k+1] (odd).
//
// Column 0 is the boundary and takes a lane of its own: its values are zero,
// which also gives the last column of the strip before it its zero right
// neighbour.  Nodes outside the problem have inverse diagonal 0, so their z
// and p stay zero.
//
// The coarse level h = 1/32 of an h = 1/64 solve is spread over the whole
// workgroup (one row pair per thread); the levels from h = 1/16 down run in
// the first wave alone, without barriers, and h = 1/4 is solved with its
// inverse (the flow cell: visited by one matrix).  The workgroup is the
// particle: the grid has one per particle, no global workspace, and the
// hardware's dispatch evens out the iteration counts.
//
// Identities used (all exact in exact arithmetic): after the first red sweep
// from z = 0 the red equations hold, so after the black sweep the red
// residual is the sum of w z_black alone; A p is formed as the sum of
// w (p_c - p_nb).
#include <algorithm>
#include <type_traits>

#include "resident.h"
#include "strips.h"

namespace mls {

namespace {

// ------------------------------------------------------------- memory --
// The finest level's split.  Row pairs per thread against threads, measured
// (us per 200 / 4000 particles, FP64): h = 1/32 four pairs, 128 threads
// 53 / 255, two pairs, 256 threads 55 / 285; h = 1/64 four pairs, 512 threads
// 83 / 1218, two pairs, 1024 threads 117 / 1732.  The flow cell's 65 rows at
// h = 1/64: five pairs, 448 threads (seven waves, two per SIMD) 118 / 1697;
// four pairs, 576 threads (nine waves, three on one SIMD: 168 registers and
// spills) 201 / 3194.
template <int LG, bool FLOW>
struct Fine;
template <> struct Fine<3, false> { static constexpr int P = 1, NT = 64; };
template <> struct Fine<4, false> { static constexpr int P = 2, NT = 64; };
template <> struct Fine<5, false> { static constexpr int P = 4, NT = 128; };
template <> struct Fine<6, false> { static constexpr int P = 4, NT = 512; };
template <> struct Fine<3, true> { static constexpr int P = 1, NT = 64; };
template <> struct Fine<4, true> { static constexpr int P = 3, NT = 64; };
template <> struct Fine<5, true> { static constexpr int P = 3, NT = 192; };
template <> struct Fine<6, true> { static constexpr int P = 5, NT = 448; };

template <typename T, int LG, bool FLOW>
struct Mem {
    using F = Fine<LG, FLOW>;
    using GF = Geo<LG, F::P, F::NT, FLOW>;
    static constexpr int P4 = FLOW ? 3 : 2, P5 = FLOW ? 2 : 1;
    using GC = std::conditional_t<LG == 6, Geo<5, P5, LG == 6 ? F::NT : 576, FLOW>,
                                  std::conditional_t<LG == 5, Geo<4, P4, 64, FLOW>, Geo<3, 1, 64, FLOW>>>;
    // the exchange of one value per thread, shared by all levels (a level's
    // neighbouring strip is n threads away), between zeros for the strips
    // outside; FP64 values where the mixed form replaces its residual
    static constexpr int pad = GF::n;
    double ex[2][F::NT + 2 * pad];
    double red[2][16];
    double cinv[FLOW ? 225 : 81];
    // the finest level's red residuals; the next level's solution takes the
    // end of their place (dead by then), with the zeros behind it beyond
    static constexpr int sol_len = grid_rows<GF, GC> * (GF::n / 2), sol_off = GF::rs - sol_len;
    static_assert(sol_off >= GF::n, "the residuals' leading zero row stays");
    T rs[GF::rs + GF::n / 2 + 1];
    // coarse levels below the finest: 5 by the workgroup, 4 and 3 by one wave
    struct None {};
    template <bool HAS, int L, int P, int NT>
    using Level = std::conditional_t<HAS, CoarseMem<T, L, P, NT, FLOW>, None>;
    Level<LG >= 6, 5, P5, LG >= 6 ? F::NT : 576> c5;
    Level<LG >= 5, 4, P4, 64> c4;
    Level<LG >= 4, 3, 1, 64> c3;
    using G5 = Geo<5, P5, LG >= 6 ? F::NT : 576, FLOW>;
    using G4 = Geo<4, P4, 64, FLOW>;
    using G3 = Geo<3, 1, 64, FLOW>;
    T e4[LG >= 6 ? (grid_rows<G5, G4> + 1) * 16 + 1 : 1];
    T e3[LG >= 5 ? (grid_rows<G4, G3> + 1) * 8 + 1 : 1];
    T e2[(G3::pairs + 1) * 4 + 1];
};

// ------------------------------------------------------------- kernel --
struct ResParams {
    int64_t N, first;  // particles, and the first one of this launch
    const int64_t* N_dev;
    const void* kappa;
    double* G;
    double* p_out;
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
};

constexpr double kDrift2 = 1e-6;  // mixed: replace r after (r, z) fell by this factor (as in solver.hip)

// Waves per SIMD the registers are budgeted for.  A second workgroup per CU
// at h = 1/64 (four waves, 128 registers) would overlap one particle's
// barriers with the other's arithmetic, but the state and weights alone take
// 120: the spills made it 2 times slower.  At h = 1/32 two waves (up to 256
// registers) keep everything; one wave took 1.6 times as long at 4000
// particles, three spilled.
template <int LG>
constexpr int kWaves = LG == 4 ? 3 : LG == 3 ? 4 : 2;

template <typename T, int LG, bool FLOW>
__global__ __launch_bounds__((Fine<LG, FLOW>::NT)) __attribute__((amdgpu_waves_per_eu(kWaves<LG>))) void
resident_kernel(ResParams A)
{
    using F = Fine<LG, FLOW>;
    using M = Mem<T, LG, FLOW>;
    using G = typename M::GF;
    constexpr int P = F::P, NT = F::NT, n = G::n, NW = NT / 64;
    constexpr bool MIXED = sizeof(T) == 4;
    constexpr bool REDO = LG == 6 && FLOW;
    constexpr int rows = G::rows;
    // the solution's grid for the observations takes the place of the rest
    __shared__ __align__(16) union {
        M m;
        double x[(n + 2) * (n + 1)];
    } sm;
    M& m = sm.m;

    int64_t q = A.first + blockIdx.x;
    const void* kappa = A.kappa;
    double *Gq = A.G, *phi = A.phi;
    const double* y = A.y;
    int8_t* status = A.status;
    int32_t* iters = A.iters;
    if (A.items) {
        int lo = 0, hi = A.n_items - 1;  // last item with base <= q
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (A.items[mid].base <= q) lo = mid; else hi = mid - 1;
        }
        const SolveItem& it = A.items[lo];
        q -= it.base;
        kappa = it.kappa; Gq = it.G; phi = it.phi; y = it.y; status = it.status; iters = it.iters;
    } else if (A.N_dev && q >= *A.N_dev) {
        return;
    }
    const T* kap = (const T*)kappa + q * (int64_t)(2 * n * n);
    Gq += q * A.nobs;

    const int t = threadIdx.x, i = t & (n - 1), e = i & 1, m0 = (t / n) * P, row0 = 2 * m0;

    // ---- set-up: weights of every level
    Weights<T, P> W;
    auto fine_cell = [&](int ci, int cj, double& lo, double& up) {
        const T* c = kap + 2 * (cj * n + ci);
        lo = (double)c[0];
        up = (double)c[1];
    };
    make_weights<false, G>(W, t, fine_cell);
    constexpr int pad = M::pad;
    for (int k = t; k < NT + 2 * pad; k += NT) m.ex[0][k] = m.ex[1][k] = 0.0;
    auto clear = [&](T* a, int c) { for (int k = t; k < c; k += NT) a[k] = T(0); };
    clear(m.e2, sizeof(m.e2) / sizeof(T));
    clear(m.e3, sizeof(m.e3) / sizeof(T));
    clear(m.e4, sizeof(m.e4) / sizeof(T));
#define MLS_LDS_CELL(K, w)                                  \
    [&](int ci, int cj, double& lo, double& up) {           \
        lo = (double)(K)[2 * (cj * (w) + ci)];              \
        up = (double)(K)[2 * (cj * (w) + ci) + 1];          \
    }
    if constexpr (LG == 6) {
        coarsen<T, 5, NT>(m.rs, t, fine_cell);
        order<NT>();
        coarse_weights(m.c5, m.rs);
    }
    if (t < 64) {
        if constexpr (LG == 3) coarsen<T, 2, 64>(m.rs, t, fine_cell);
        if constexpr (LG == 4) coarsen<T, 3, 64>(m.rs, t, fine_cell);
        if constexpr (LG == 5) coarsen<T, 4, 64>(m.rs, t, fine_cell);
        if constexpr (LG == 6) coarsen<T, 4, 64>(m.c5.rs, t, MLS_LDS_CELL(m.rs, 32));
        wave_order();
        if constexpr (LG >= 5) {
            const T* k4;
            if constexpr (LG == 6) k4 = m.c5.rs;
            else k4 = m.rs;
            coarse_weights(m.c4, k4);
            coarsen<T, 3, 64>(m.c4.rs, t, MLS_LDS_CELL(k4, 16));
            wave_order();
        }
        const T* k2;
        if constexpr (LG >= 4) {
            const T* k3;
            if constexpr (LG == 4) k3 = m.rs;
            else k3 = m.c4.rs;
            coarse_weights(m.c3, k3);
            coarsen<T, 2, 64>(m.c3.rs, t, MLS_LDS_CELL(k3, 8));
            k2 = m.c3.rs;
        } else {
            k2 = m.rs;
        }
        wave_order();
        if constexpr (FLOW) visit2_build(k2, m.cinv);
        else exact_build(k2, m.cinv);
    }
#undef MLS_LDS_CELL
    order<NT>();
    clear(m.rs, sizeof(m.rs) / sizeof(T));
    if constexpr (LG == 6) clear(m.c5.rs, sizeof(m.c5.rs) / sizeof(T));
    if constexpr (LG >= 5) clear(m.c4.rs, sizeof(m.c4.rs) / sizeof(T));
    if constexpr (LG >= 4) clear(m.c3.rs, sizeof(m.c3.rs) / sizeof(T));
    order<NT>();

    // ---- state
    T rr[P], rb[P], zr[P], zb[P], pr[P], pb[P], xr[P], xb[P], O[P];
    double x64[MIXED ? 2 : 1][MIXED ? P : 1];  // mixed: the FP64 iterate
    auto valid_row = [&](int c, int k) { return G::valid(i, row0 + 2 * k + ((c == 0) == (e != 0) ? 1 : 0)); };
    const double h2 = 1.0 / (double)(n * n);
    auto rhs = [&](int c, int k) -> double {
        if (!valid_row(c, k)) return 0.0;
        if (FLOW) return i == n - 1 ? (double)W.wr[c][k] : 0.0;  // the lifted boundary value 1
        return h2;
    };
#pragma unroll
    for (int k = 0; k < P; ++k) {
        rr[k] = T(rhs(0, k));
        rb[k] = T(rhs(1, k));
        pr[k] = pb[k] = xr[k] = xb[k] = T(0);
        if constexpr (MIXED) x64[0][k] = x64[1][k] = 0.0;
    }

    T* ex0 = reinterpret_cast<T*>(m.ex[0]) + pad;
    T* ex1 = reinterpret_cast<T*>(m.ex[1]) + pad;
    T* sol_next = m.rs + M::sol_off;
    auto total = [&](double v, int which) -> double {
        v = lane63_sum(v);
        if constexpr (NW == 1) {
            return read_lane(v, 63);
        } else {
            if ((t & 63) == 63) m.red[which][t >> 6] = v;
            order<NT>();
            double s = 0.0;
#pragma unroll
            for (int k = 0; k < NW; ++k) s += m.red[which][k];
            return wave_uniform(s);
        }
    };
    // z = V r from the residual in registers; (r, z)
    auto vcycle = [&]() -> double {
        const At<G, P, REDO> at;
#pragma unroll
        for (int k = 0; k < P; ++k) zr[k] = rr[k] * W.inv[0][k];
        down_leg<G, NT>(W, at, rb, zr, zb, ex0, ex1, m.rs);
        order<NT>();
        const T* ec;
        if constexpr (LG == 3) {
            exact_solve<FLOW>(m.rs, m.cinv, m.e2);
            ec = m.e2;
        } else {
            auto visit2 = [&]() { exact_solve<FLOW>(m.c3.rs, m.cinv, m.e2); };
            ec = sol_next;
            if constexpr (LG == 4) {
                coarse_visit<3, 1, 64, FLOW, REDO>(m.rs, m.c3, sol_next, m.e2, ex0, ex1, visit2);
            } else {
                auto visit3 = [&]() {
                    coarse_visit<3, 1, 64, FLOW, REDO>(m.c4.rs, m.c3, m.e3, m.e2, ex0, ex1, visit2);
                };
                if constexpr (LG == 5) {
                    if (t < 64) coarse_visit<4, M::P4, 64, FLOW, REDO>(m.rs, m.c4, sol_next, m.e3, ex0, ex1, visit3);
                } else {
                    coarse_visit<5, M::P5, NT, FLOW, REDO>(m.rs, m.c5, sol_next, m.e4, ex0, ex1, [&]() {
                        if (t < 64) coarse_visit<4, M::P4, 64, FLOW, REDO>(m.c5.rs, m.c4, m.e4, m.e3, ex0, ex1, visit3);
                    });
                }
            }
        }
        order<NT>();
        const At<G, P, REDO> at2;
        up_leg<G, NT>(W, at2, rr, rb, zr, zb, ex0, ex1, ec);
        double d = 0.0;
#pragma unroll
        for (int k = 0; k < P; ++k) d += (double)rr[k] * (double)zr[k] + (double)rb[k] * (double)zb[k];
        return total(d, 1);
    };
    // (A x) at the thread's pair k from the edges' fluxes w (x_c - x_nb): a
    // node's east flux, with the other sign, is its east neighbour's west one
    auto flux = [&](auto r, auto b, auto o_r, auto o_b, int k, auto& ar, auto& ab) {
        using V = decltype(r);
        T wr0 = W.wr[0][k], wr1 = W.wr[1][k], w0 = W.o[0][k], w1 = W.o[1][k], ws = W.s[k];
        // mixed: keep the promoted weights out of the iterations' registers
        if constexpr (sizeof(V) != sizeof(T)) asm volatile("" : "+v"(wr0), "+v"(wr1), "+v"(w0), "+v"(w1), "+v"(ws));
        const V fr = V(wr0) * (r - east(b)), fb = V(wr1) * (b - east(r)), fs = V(ws) * (r - b);
        ar = (fr - west(fb)) + (fs + V(w0) * (r - o_r));
        ab = (fb - west(fr)) + (V(w1) * (b - o_b) - fs);
    };
    // mixed: x64 += x, x = 0, r = b - A x64 in FP64 (rounded)
    auto replace_residual = [&]() {
        if constexpr (MIXED) {
#pragma unroll
            for (int k = 0; k < P; ++k) {
                x64[0][k] += (double)xr[k];
                x64[1][k] += (double)xb[k];
                xr[k] = xb[k] = T(0);
            }
            double* exd0 = m.ex[0] + pad;
            double* exd1 = m.ex[1] + pad;
            order<NT>();  // the exchange is read as T until here
            publish<G, 1>(x64[0], exd0, t);
            publish<G, 0>(x64[1], exd1, t);
            if (t < pad)  // its outer zeros, at their FP64 places
                exd0[t - pad] = exd1[t - pad] = exd0[t + NT] = exd1[t + NT] = 0.0;
            order<NT>();
            const At<G, P, REDO> at;
            double Or[P], Ob[P];
            outer<G, 0>(x64[1], exd1, at, Or);
            outer<G, 1>(x64[0], exd0, at, Ob);
#pragma unroll
            for (int k = 0; k < P; ++k) {
                double ar, ab;
                flux(x64[0][k], x64[1][k], Or[k], Ob[k], k, ar, ab);
                T ir = W.inv[0][k], ib = W.inv[1][k];
                asm volatile("" : "+v"(ir), "+v"(ib));
                rr[k] = T((ir != T(0) ? h2 : 0.0) - ar);
                rb[k] = T((ib != T(0) ? h2 : 0.0) - ab);
            }
            order<NT>();
            if (t < pad)  // and back to T
                ex0[t - pad] = ex1[t - pad] = ex0[t + NT] = ex1[t + NT] = T(0);
            order<NT>();
        }
    };

    // PCG.  One copy of the cycle serves the first direction, the iterations
    // and the mixed form's confirmation on a replaced residual.
    double rz = 0.0, rz0 = 0.0, rz_upd = 0.0;
    T beta = T(0);
    int it = 0;
    int8_t st = 1;
    enum { FIRST, STEP, CONFIRM } phase = FIRST;
    bool bad_alpha = false;
    while (true) {
        const double v = vcycle();
        bool again = false;  // mixed: confirm on the replaced residual first
        if (phase == FIRST) {
            rz = rz0 = rz_upd = v;
            if (!(v > 0.0) || !isfinite(v)) { st = FLOW && isfinite(v) ? 0 : 2; break; }
        } else if (phase == CONFIRM) {
            if (!isfinite(v)) { st = 2; break; }
            if (v <= A.tol2 * rz0) { st = 0; break; }
            rz = rz_upd = v;  // not there yet: go on from the true residual, directions restarted
            beta = T(0);
        } else {
            ++it;
            if (!isfinite(v) || (FLOW && bad_alpha)) { st = 2; break; }
            const bool conv = v <= A.tol2 * rz0;
            if constexpr (MIXED) {
                if (conv || v <= kDrift2 * rz_upd) {
                    replace_residual();
                    rz_upd = v;
                    again = conv;
                }
            } else {
                if (conv) { st = 0; break; }
            }
            beta = T(v / rz);
            rz = v;
        }
        phase = again ? CONFIRM : STEP;
        if (again) continue;
        if (it >= A.max_iters) break;
        // p = z + beta p and q = A p (kept in z's registers)
#pragma unroll
        for (int k = 0; k < P; ++k) {
            pr[k] = zr[k] + beta * pr[k];
            pb[k] = zb[k] + beta * pb[k];
        }
        publish<G, 1>(pr, ex0, t);
        publish<G, 0>(pb, ex1, t);
        order<NT>();
        double pq = 0.0;
        const At<G, P, REDO> at;
        T O2[P];
        outer<G, 0>(pb, ex1, at, O);
        outer<G, 1>(pr, ex0, at, O2);
#pragma unroll
        for (int k = 0; k < P; ++k) {
            flux(pr[k], pb[k], O[k], O2[k], k, zr[k], zb[k]);
            pq += (double)pr[k] * (double)zr[k] + (double)pb[k] * (double)zb[k];
        }
        pq = total(pq, 0);
        const double alpha_d = rz / pq;
        const T alpha = T(alpha_d);
        bad_alpha = !isfinite(alpha_d);
#pragma unroll
        for (int k = 0; k < P; ++k) {
            xr[k] += alpha * pr[k];
            xb[k] += alpha * pb[k];
            rr[k] -= alpha * zr[k];
            rb[k] -= alpha * zb[k];
        }
    }

    // ---- observations, field, potential
    auto sol = [&](int c, int k) -> double {
        if constexpr (MIXED) return x64[c][k] + (st != 0 ? (double)(c ? xb[k] : xr[k]) : 0.0);
        else return c ? xb[k] : xr[k];
    };
    order<NT>();  // the level arrays are dead: their memory takes the grid
    {
        constexpr int s = n + 1;
        // rows of the observation table: offset by the ghost row on the flow cell
        for (int k = t; k < n + 2; k += NT) {
            sm.x[k * s + n] = FLOW ? 1.0 : 0.0;  // column n: the boundary value
            if (!FLOW && k <= n) sm.x[n * s + k] = 0.0;
        }
#pragma unroll
        for (int k = 0; k < P; ++k)
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const int j = row0 + 2 * k + ((c == 0) == (e != 0) ? 1 : 0);
                if (j >= rows) continue;
                const double v = sol(c, k);
                sm.x[j * s + i] = v;
                if (A.p_out && G::valid(i, j))
                    A.p_out[q * (int64_t)((n - 1) * (FLOW ? n + 1 : n - 1)) + (j - (FLOW ? 0 : 1)) * (n - 1) + i - 1] = v;
            }
    }
    order<NT>();
    double ph = 0.0;
    for (int o = t; o < A.nobs; o += NT) {
        double g = 0.0;
#pragma unroll
        for (int k = 0; k < 3; ++k) g += A.obs_w[3 * o + k] * sm.x[A.obs_idx[3 * o + k] - (FLOW ? n + 1 : 0)];
        Gq[o] = g;
        if (y) {
            const double r = (y[o] - g) * A.inv_sigma;
            ph += r * r;
        }
    }
    if (y) {
        order<NT>();
        ph = total(ph, 0);
    }
    if (t == 0) {
        if (status) status[q] = st;
        if (iters) iters[q] = it;
        if (phi) phi[q] = 0.5 * ph;
    }
}

template <typename T, bool FLOW>
int launch_level(int l, unsigned grid, const ResParams& A, hipStream_t s)
{
    switch (l) {
    case 3: resident_kernel<T, 3, FLOW><<<grid, Fine<3, FLOW>::NT, 0, s>>>(A); break;
    case 4: resident_kernel<T, 4, FLOW><<<grid, Fine<4, FLOW>::NT, 0, s>>>(A); break;
    case 5: resident_kernel<T, 5, FLOW><<<grid, Fine<5, FLOW>::NT, 0, s>>>(A); break;
    case 6: resident_kernel<T, 6, FLOW><<<grid, Fine<6, FLOW>::NT, 0, s>>>(A); break;
    default: MLS_REQUIRE(false, "resident solver: level outside h = 1/8 .. 1/64");
    }
    MLS_CHECK_HIP(hipGetLastError());
    return MLS2MC_OK;
}

int launch_params(mls2mc_ctx* ctx, int l, int64_t total, bool mixed, ResParams& A, hipStream_t s)
{
    A.obs_idx = ctx->obs[l].idx;
    A.obs_w = ctx->obs[l].w;
    A.nobs = ctx->nobs;
    A.inv_sigma = 1.0 / ctx->prob.sigma_n;
    A.tol2 = ctx->rtol * ctx->rtol;
    A.max_iters = ctx->max_iters;
    for (A.first = 0; A.first < total; A.first += kLaunchParticles) {
        const unsigned grid = (unsigned)std::min(kLaunchParticles, total - A.first);
        if (ctx->prob.bc == MLS2MC_BC_FLOW_CELL) MLS_TRY((launch_level<double, true>(l, grid, A, s)));
        else if (mixed) MLS_TRY((launch_level<float, false>(l, grid, A, s)));
        else MLS_TRY((launch_level<double, false>(l, grid, A, s)));
    }
    return MLS2MC_OK;
}

}  // namespace

int resident_token(const mls2mc_ctx* ctx, int l)
{
    if (ctx->prob.bc == MLS2MC_BC_FLOW_CELL) return l <= 5 ? 256 : 512;
    return l <= 4 ? 64 : l == 5 ? 128 : l == 6 ? 256 : 1024;
}

bool resident_level(const mls2mc_ctx* ctx, int l)
{
    if (l < 3 || l > 7 || (l == 7 && !resident7_runs(ctx))) return false;
    if (ctx->solver_grid[l] != 0 || ctx->solver_lds[l] != 0) return false;
    return ctx->solver_block[l] == 0 ? ctx->solver_nu[l] <= 1
                                     : ctx->solver_block[l] == resident_token(ctx, l) && ctx->solver_nu[l] == 0;
}

size_t resident_workspace(const mls2mc_ctx* ctx, int l, int64_t total)
{
    return l == 7 ? resident7_workspace(ctx, total) : 0;
}

int launch_resident(mls2mc_ctx* ctx, const SolveArgs& a, hipStream_t s)
{
    if (a.N == 0) return MLS2MC_OK;
    ResParams A = {};
    A.N = a.N; A.N_dev = a.N_dev; A.kappa = a.kappa; A.G = a.G; A.p_out = a.p_out;
    A.status = a.status; A.iters = a.iters; A.y = a.y; A.phi = a.phi;
    ProfRec rec;
    if (ctx->prof_on) {
        if (!A.iters) {  // the iteration totals need per-particle counts
            MLS_TRY(ctx->ws_prof.ensure(sizeof(int32_t) * (size_t)a.N));
            A.iters = ctx->ws_prof.as<int32_t>();
        }
        MLS_TRY(prof_begin(ctx, MLS2MC_PROF_SOLVE, a.l, a.N, s, &rec));
    }
    if (a.l == 7) MLS_TRY(launch_resident7(ctx, a, A.iters, s));
    else MLS_TRY(launch_params(ctx, a.l, a.N, a.kappa_f32, A, s));
    if (ctx->prof_on) {
        MLS_TRY(prof_end(ctx, MLS2MC_PROF_SOLVE, a.l, rec, s));
        MLS_TRY(launch_reduce_i32(a.N, A.iters, nullptr, ctx->d_prof_iters + 2 * a.l, s));
    }
    return MLS2MC_OK;
}

int launch_resident_list(mls2mc_ctx* ctx, int l, const SolveItem* items_dev, int n_items, int64_t total, bool mixed,
                         hipStream_t s)
{
    if (total == 0 || n_items == 0) return MLS2MC_OK;
    if (l == 7) return launch_resident7_list(ctx, items_dev, n_items, total, s);
    ResParams A = {};
    A.N = total;
    A.items = items_dev;
    A.n_items = n_items;
    return launch_params(ctx, l, total, mixed, A, s);
}

}  // namespace mls
