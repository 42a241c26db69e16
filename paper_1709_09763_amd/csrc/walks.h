// Fused row walks of the multigrid V(1,1) legs on the large levels, for the
// Dirichlet solver (solver.hip) and the flow cell's (flowcell.hip).
#pragma once

#include <type_traits>

#include "common.h"

namespace mls {

// ------------------------------------------------------- fused row walks --
// On a large level (n >= 256) the down-leg (optional residual update r -= a q,
// red sweep from a zero start, black sweep, restriction of the residual)
// and the up-leg (black sweep with the coarse correction, red sweep, the
// dot (b, z)) each run as one pass over the rows instead of three and two.
// Thread t of a band owns the column pair (2t, 2t+1) of every row of the
// band, so each row step gives every thread one red and one black node.
// Going up row j, the down walk updates the residual of row j and its red
// node, the black node of row j-1 (its red neighbours are final), the red
// residual of row j-2 (its black neighbours are final) and, one step later
// (the residuals of a row come from neighbouring threads), the coarse
// right-hand side of coarse row (j-4)/2.  A node's own column lives in the
// thread's registers, the neighbouring threads' values pass through a ring
// of LDS rows, with one barrier per row step.  Every node evaluates the
// same expression as the separate sweeps, so the iterates are bitwise
// theirs; only the order of the terms of (b, z) differs.
//
// The m = BS / (n/2) bands walk their row ranges [j0, j1) in lock step.  A
// band first recomputes, without storing, the three rows below j0 from the
// residual update's inputs, which the band below overwrites only at the end
// of its walk; above j1 it recomputes the red and black values from the
// updated residual, which the band above stored in its first steps.  The up
// walk reads only values that no band writes during it (the right-hand side,
// the weights, the coarse correction), so its bands need no ordering at all.
template <int BS>
__device__ __forceinline__ bool walk_level(int n, int nu)
{
    return nu == 1 && n >= 256 && BS % (n >> 1) == 0;
}

// LDS elements of the walks on a level of width n: per band four rows of
// the node values and four rows of red residuals (down) or of the down-leg's
// red values (up), one per thread between two zeros
__host__ __device__ inline int64_t walk_ring_elems_level(int bs, int n)
{
    const int64_t m = bs / (n >> 1);
    return m * (4 * (int64_t)(n + 1) + 4 * (int64_t)((n >> 1) + 2));
}
// the most any walked level of a hierarchy with finest level l needs
__host__ __device__ inline int64_t walk_ring_elems(int bs, int l)
{
    int64_t e = 0;
    for (int L = l; L >= 8; --L) {
        const int n = 1 << L;
        if (bs % (n >> 1) == 0) {
            const int64_t v = walk_ring_elems_level(bs, n);
            if (v > e) e = v;
        }
    }
    return e;
}

// One band's rows: [j0, j1), the ring offset of the band, this thread's
// pair.  A band has n / m rows, an even number (the last one up to the last
// row of unknowns), so every band starts on a row of the parity of the first
// and the walks can unroll two row steps of fixed parity.
struct WalkRows {
    int t, j0, j1;
    int64_t ring_off;
};
template <int BS>
__device__ __forceinline__ WalkRows walk_rows(int n, int lo, int hi)
{
    const int P = n >> 1, m = BS / P;
    const int band = threadIdx.x / P;
    WalkRows w;
    w.t = threadIdx.x - band * P;
    const int rows = n / m;
    w.j0 = lo + band * rows;
    w.j1 = band == m - 1 ? hi + 1 : w.j0 + rows;
    w.ring_off = (int64_t)band * (4 * (n + 1) + 4 * (P + 2));
    return w;
}

template <int K>
using Par = std::integral_constant<int, K>;

// FLOW: the flow cell's rows.  Its unknowns are the rows 0 .. n, between ghost
// rows -1 and n + 1 whose edges weigh zero, and an array's row j is at
// (j + 1) s: the walks address it from one row further on.  The Dirichlet
// problem's unknowns are the rows 1 .. n - 1.
template <bool FLOW>
struct WalkSpan {
    int lo, hi;  // first and last row of unknowns
    __device__ __forceinline__ explicit WalkSpan(int n) : lo(FLOW ? 0 : 1), hi(FLOW ? n : n - 1) {}
};

// The walked levels never sit in LDS (a row of 257 values already exceeds
// the residency budgets), so the walks address their arrays as global
// memory and their rows as LDS: global and LDS instructions instead of flat
// ones, which also lets the compiler keep them apart.
template <typename T>
using gmem = T __attribute__((address_space(1)))*;
template <typename T>
using lmem = T __attribute__((address_space(3)))*;

// The barrier between row steps: it orders the LDS ring only, so the
// global loads and stores of a step stay in flight across it (a full
// barrier would wait for every store to be acknowledged).
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Down-leg of a V(1,1) cycle on level L into the coarser level's right-hand
// side C.b.  With Q: b -= alpha Q first (the CG residual update; b is
// updated in place) and, with X and Pn, also X += alpha Pn (the mixed
// solver's iterate).  Without Q, b is only read.  x receives z.  In a step
// on row j every phase works on the thread's column of parity j: the red
// node of row j, the black node of row j-1 and the red node of row j-2 all
// sit in it.  The node values of the last four rows are kept in the LDS
// ring (the thread's own ones too); the weights come from registers on the
// finest level and from memory on a walked coarse level (see below).  z is
// not stored: the up-leg overwrites its black values without reading them,
// and forms its red ones, b / d, again (16 B less per unknown than storing
// and reading z back).
// coarse_red (flow cell): C.x gets the coarse level's first red sweep from
// zero too, for a coarser level with separate sweeps.
template <int BS, bool FINE, bool FLOW, typename T, typename LEVEL, typename COARSE>
__device__ __forceinline__ void walk_down_here(const LEVEL& L, const COARSE& C, T* __restrict__ b, const T* __restrict__ Q, T alpha,
                          T* __restrict__ X, const T* __restrict__ Pn, T* __restrict__ ring, bool coarse_red = false)
{
    using W = std::remove_const_t<std::remove_reference_t<decltype(*L.wx)>>;
    const int n = L.n, s = L.s, P = n >> 1, sc = C.s, nc = C.n;
    const WalkSpan<FLOW> span(n), cspan(nc);
    const int lo = span.lo, hi = span.hi, first = FLOW ? s : 0, firstc = FLOW ? sc : 0;  // of row 0
    const WalkRows w = walk_rows<BS>(n, lo, hi);
    const int t = w.t, j0 = w.j0, j1 = w.j1, ca = 2 * t;
    const lmem<T> lring = (lmem<T>)ring;
    const lmem<T> zr = lring + w.ring_off;  // node values, 4 rows of s
    const lmem<T> rr = zr + 4 * s;          // red residuals, 4 rows of P + 2
    // columns 0 and n of the rows are never written: they read as the zero boundary
    for (int k = threadIdx.x; k < walk_ring_elems_level(BS, n); k += BS) lring[k] = T(0);
    __syncthreads();
    const gmem<const W> wx = (gmem<const W>)(L.wx + first);
    const gmem<const W> wy = (gmem<const W>)(L.wy + first);
    const gmem<T> gb = (gmem<T>)(b + first);
    const gmem<const T> gQ = (gmem<const T>)(Q + first);
    const gmem<T> gX = (gmem<T>)(X + first);
    const gmem<const T> gPn = (gmem<const T>)(Pn + first);
    const gmem<T> gCb = (gmem<T>)(C.b + firstc);
    T r0[2] = {T(0), T(0)}, r1[2] = {T(0), T(0)}, r2[2] = {T(0), T(0)};  // updated residual, rows j .. j-2
    // On the finest level (FINE; FP32 weights in both solvers) the weights
    // of the thread's columns are read from global memory once per row and
    // carried through the three steps that use them: wx of columns
    // ca-1 .. ca+1 for rows j .. j-2, wy of columns ca, ca+1 for rows
    // j .. j-3.  Read again from memory, those rows fall out of the L2 when
    // every CU of an XCD walks its own particle.  On the walked coarse level
    // (FP64 weights in the FP64 solver) the registers are dearer than the
    // re-reads, and the weights are read where they are used.
    constexpr bool win = FINE;
    W x0[3], x1[3], x2[3], y0[2], y1[2], y2[2], y3[2];
    // wx of row j - r, column ca - 1 + u; wy of row j - r, column ca + u
    auto WX = [&](int j, int r, int u) -> T {
        if constexpr (win) return T(r == 0 ? x0[u] : r == 1 ? x1[u] : x2[u]);
        else return T(wx[(j - r) * s + ca - 1 + u]);
    };
    auto WY = [&](int j, int r, int u) -> T {
        if constexpr (win) return T(r == 0 ? y0[u] : r == 1 ? y1[u] : r == 2 ? y2[u] : y3[u]);
        else return T(wy[(j - r) * s + ca + u]);
    };
    auto load_w = [&](int jj, W* xr, W* yr) {
        const bool in = jj >= lo - 1 && jj <= (FLOW ? n : n - 1);
        const int c = jj * s + ca;
        xr[0] = in && ca > 0 ? wx[c - 1] : W(0);
        xr[1] = in ? wx[c] : W(0);
        xr[2] = in ? wx[c + 1] : W(0);
        yr[0] = in ? wy[c] : W(0);
        yr[1] = in ? wy[c + 1] : W(0);
    };
    if constexpr (win) {
        load_w(j0 - 4, x0, y0);
#pragma unroll
        for (int u = 0; u < 3; ++u) x1[u] = x2[u] = W(0);
        y1[0] = y1[1] = y2[0] = y2[1] = y3[0] = y3[1] = W(0);
    }
    auto body = [&](auto par, int j) {
        constexpr int k = decltype(par)::value;  // the active column: ca + k
        r2[0] = r1[0]; r2[1] = r1[1]; r1[0] = r0[0]; r1[1] = r0[1]; r0[0] = T(0); r0[1] = T(0);
        if constexpr (win) {
#pragma unroll
            for (int u = 0; u < 3; ++u) { x2[u] = x1[u]; x1[u] = x0[u]; }
            y3[0] = y2[0]; y3[1] = y2[1]; y2[0] = y1[0]; y2[1] = y1[1]; y1[0] = y0[0]; y1[1] = y0[1];
            load_w(j, x0, y0);
        }
        const bool active = ca + k > 0;  // column 0 is the boundary
        auto Z = [&](int jj, int i) -> T __attribute__((address_space(3)))& { return zr[(jj & 3) * s + i]; };
        if (j == hi + 1) {  // the row above the unknowns, read by the black sweep and the residuals below it
            Z(hi + 1, ca) = T(0);
            Z(hi + 1, ca + 1) = T(0);
        }
        // ---- row j: residual update and the red node
        if (j >= lo && j <= hi && j <= j1 + 2) {
            const int c = j * s + ca;
            if (Q && j < j1) {
                r0[0] = gb[c] - alpha * gQ[c];
                r0[1] = gb[c + 1] - alpha * gQ[c + 1];
                if (j >= j0) {
                    if (ca > 0) gb[c] = r0[0];
                    gb[c + 1] = r0[1];
                    if (X) {
                        gX[c] += alpha * gPn[c];
                        gX[c + 1] += alpha * gPn[c + 1];
                    }
                }
            } else {  // no update, or rows above the band (updated there already)
                r0[0] = gb[c];
                r0[1] = gb[c + 1];
            }
            if (active)
                Z(j, ca + k) = r0[k] / (WX(j, 0, k) + WX(j, 0, k + 1) + WY(j, 1, k) + WY(j, 0, k));
        }
        // ---- row j-1: the black node (red neighbours final)
        const int jb = j - 1;
        if (jb >= lo && jb <= hi && jb >= j0 - 2 && jb <= j1 + 1) {
            const int i = ca + k;
            if (active) {
                const T nb = WX(j, 1, k) * Z(jb, i - 1) + WX(j, 1, k + 1) * Z(jb, i + 1) + WY(j, 2, k) * Z(jb - 1, i)
                           + WY(j, 1, k) * Z(j, i);
                Z(jb, i) = (r1[k] + nb) / (WX(j, 1, k) + WX(j, 1, k + 1) + WY(j, 2, k) + WY(j, 1, k));
            }
        }
        // ---- row j-2: the red residual (black neighbours final)
        const int jc = j - 2;
        if (jc >= lo && jc <= hi && jc >= j0 - 1 && jc <= j1 && active) {
            const int i = ca + k;
            const T d = WX(j, 2, k) + WX(j, 2, k + 1) + WY(j, 3, k) + WY(j, 2, k);
            const T lnb = WX(j, 2, k) * Z(jc, i - 1) + WX(j, 2, k + 1) * Z(jc, i + 1) + WY(j, 3, k) * Z(jc - 1, i)
                        + WY(j, 2, k) * Z(jc + 1, i);
            rr[(jc & 3) * (P + 2) + t] = r2[k] - (d * Z(jc, i) - lnb);
        }
        // ---- coarse row (j-4)/2: restriction of the red residuals
        if (k == 0) {
            const int J = (j - 4) >> 1;
            if (J >= cspan.lo && J <= cspan.hi && 2 * J >= j0 && 2 * J < j1 && t >= 1 && t <= nc - 1) {
                const T a0 = rr[((2 * J) & 3) * (P + 2) + t];
                const T ap = FLOW && 2 * J == hi ? T(0) : rr[((2 * J + 1) & 3) * (P + 2) + t];
                const T am = rr[((2 * J - 1) & 3) * (P + 2) + t - 1];
                const T v = a0 + T(0.5) * (ap + am);
                gCb[J * sc + t] = v;
                if (FLOW && coarse_red) {
                    const int q = firstc + J * sc + t;
                    C.x[q] = ((J + t) & 1) ? T(0) : v / (C.wx[q - 1] + C.wx[q] + C.wy[q - sc] + C.wy[q]);
                }
            }
        }
        // the band above stored its first three rows (the rows this band's
        // walk ends on) in steps 3 to 5: one full barrier after them makes
        // those stores visible; every other step orders the LDS ring only
        if (j - (j0 - 3) == 6) __syncthreads();
        else lds_barrier();
    };
    // rows j0 - 3 .. j1 + 3
#pragma unroll 1
    for (int j = j0 - 3; j <= j0 + (n / (BS / P)) + 4; j += 2) {
        body(Par<FLOW ? 1 : 0>{}, j);
        body(Par<FLOW ? 0 : 1>{}, j + 1);
    }
    __syncthreads();  // the updated residual and C.b are complete
}

// Up-leg of a V(1,1) cycle on level L after the coarser level was solved
// (its correction e, row stride sc): the black sweep with the correction
// interpolated at the red neighbours, then the red sweep, writing z to x.
// Returns (b, z) over the interior nodes when want_dot.  In a step on row j
// the phases work on the thread's column of parity j + 1: the down-leg's red
// value b / d of row j + 1 (formed again here, bitwise: the down-leg started
// from zero), the black node of row j and the red node of row j - 1.  Values
// pass through the LDS ring as in walk_down.  The walk reads only what no
// band writes during it (the right-hand side, the weights, the correction).
template <int BS, bool FINE, bool FLOW, typename T, typename LEVEL>
__device__ __forceinline__ double walk_up_here(const LEVEL& L, const T* __restrict__ e, int sc, const T* __restrict__ b,
                          T* __restrict__ x, bool want_dot, T* __restrict__ ring, double* red)
{
    using W = std::remove_const_t<std::remove_reference_t<decltype(*L.wx)>>;
    const int n = L.n, s = L.s, P = n >> 1;
    const WalkSpan<FLOW> span(n);
    const int lo = span.lo, hi = span.hi, first = FLOW ? s : 0;
    const WalkRows w = walk_rows<BS>(n, lo, hi);
    const int t = w.t, j0 = w.j0, j1 = w.j1, ca = 2 * t;
    const lmem<T> lring = (lmem<T>)ring;
    const lmem<T> zb = lring + w.ring_off;  // new values, 4 rows of s
    const lmem<T> zd = zb + 4 * s + 1;      // the down-leg's red values, 4 rows of P + 2 from -1
    for (int k = threadIdx.x; k < walk_ring_elems_level(BS, n); k += BS) lring[k] = T(0);
    __syncthreads();
    const gmem<const W> wx = (gmem<const W>)(L.wx + first);
    const gmem<const W> wy = (gmem<const W>)(L.wy + first);
    const gmem<const T> ge = (gmem<const T>)(e + (FLOW ? sc : 0));
    const gmem<const T> gbv = (gmem<const T>)(b + first);
    const gmem<T> gx = (gmem<T>)(x + first);
    auto pe = [&](int ii, int jj) -> T {
        const int q = (jj >> 1) * sc + (ii >> 1);
        return (ii & 1) ? T(0.5) * (ge[q] + ge[q + sc + 1]) : ge[q];
    };
    // As in walk_down, on the finest level each row's weights of the
    // thread's columns (wx of columns ca-1 .. ca+1 for rows j+1 .. j-1; wy of
    // columns ca, ca+1 for rows j+1 .. j-2) are read from global memory once
    // and carried in registers.
    constexpr bool win = FINE;
    W x0[3], x1[3], x2[3], y0[2], y1[2], y2[2], y3[2];
    auto WX = [&](int j, int r, int u) -> T {  // wx of row j + 1 - r, column ca - 1 + u
        if constexpr (win) return T(r == 0 ? x0[u] : r == 1 ? x1[u] : x2[u]);
        else return T(wx[(j + 1 - r) * s + ca - 1 + u]);
    };
    auto WY = [&](int j, int r, int u) -> T {  // wy of row j + 1 - r, column ca + u
        if constexpr (win) return T(r == 0 ? y0[u] : r == 1 ? y1[u] : r == 2 ? y2[u] : y3[u]);
        else return T(wy[(j + 1 - r) * s + ca + u]);
    };
    auto load_w = [&](int jj, W* xr, W* yr) {
        const bool in = jj >= lo - 1 && jj <= (FLOW ? n : n - 1);
        const int c = jj * s + ca;
        xr[0] = in && ca > 0 ? wx[c - 1] : W(0);
        xr[1] = in ? wx[c] : W(0);
        xr[2] = in ? wx[c + 1] : W(0);
        yr[0] = in ? wy[c] : W(0);
        yr[1] = in ? wy[c + 1] : W(0);
    };
    T bn[2] = {T(0), T(0)}, b0[2] = {T(0), T(0)}, b1[2] = {T(0), T(0)};  // right-hand side of rows j+1 .. j-1
    T dn = T(0), d0 = T(0), d1 = T(0);  // the thread's red value of the down-leg, rows j+1 .. j-1
    if constexpr (win) {
        load_w(j0 - 3, x0, y0);
#pragma unroll
        for (int u = 0; u < 3; ++u) x1[u] = x2[u] = W(0);
        y1[0] = y1[1] = y2[0] = y2[1] = W(0);
    }
    double dot = 0.0;
    // k: the active column, ca + k, which holds the red nodes of rows j + 1
    // and j - 1 and the black node of row j.  ahead: only the red value of
    // row j + 1 (the steps before the band's first black row)
    auto body = [&](auto par, int j, auto ahead) {
        constexpr int k = 1 - decltype(par)::value;
        b1[0] = b0[0]; b1[1] = b0[1]; b0[0] = bn[0]; b0[1] = bn[1];
        d1 = d0; d0 = dn;
        if constexpr (win) {
#pragma unroll
            for (int u = 0; u < 3; ++u) { x2[u] = x1[u]; x1[u] = x0[u]; }
            y3[0] = y2[0]; y3[1] = y2[1]; y2[0] = y1[0]; y2[1] = y1[1]; y1[0] = y0[0]; y1[1] = y0[1];
            load_w(j + 1, x0, y0);
        }
        auto Z = [&](int jj, int i) -> T __attribute__((address_space(3)))& { return zb[(jj & 3) * s + i]; };
        const int i = ca + k;
        // ---- row j+1: its right-hand side and the down-leg's red value
        const int jn = j + 1;
        bn[0] = bn[1] = dn = T(0);
        if (jn >= lo && jn <= hi && jn <= j1 + 1) {
            bn[0] = gbv[jn * s + ca];
            bn[1] = gbv[jn * s + ca + 1];
            if (i > 0) dn = bn[k] / (WX(j, 0, k) + WX(j, 0, k + 1) + WY(j, 1, k) + WY(j, 0, k));
        }
        zd[(jn & 3) * (P + 2) + t] = dn;
        if constexpr (!decltype(ahead)::value) {
            if (j == hi + 1) {  // the row above the unknowns, read by the red sweep below it
                Z(hi + 1, ca) = T(0);
                Z(hi + 1, ca + 1) = T(0);
            }
            // ---- row j: the black node, corrected.  Its neighbours of row j:
            // the thread's own red node and the neighbouring thread's
            if (j >= lo && j <= hi && j <= j1 && i > 0) {
                const T out = zd[(j & 3) * (P + 2) + (k == 0 ? t - 1 : t + 1)];
                const T xw = k == 0 ? out : d0;
                const T xe = k == 0 ? d0 : out;
                const T nb = WX(j, 1, k) * (xw + pe(i - 1, j)) + WX(j, 1, k + 1) * (xe + pe(i + 1, j))
                           + WY(j, 2, k) * (d1 + pe(i, j - 1)) + WY(j, 1, k) * (dn + pe(i, j + 1));
                Z(j, i) = (b0[k] + nb) / (WX(j, 1, k) + WX(j, 1, k + 1) + WY(j, 2, k) + WY(j, 1, k));
            }
            // ---- row j-1: the red node (black neighbours new); the row is then final
            const int jr = j - 1;
            if (jr >= j0 && jr < j1) {
                if (i > 0) {
                    const T lnb = WX(j, 2, k) * Z(jr, i - 1) + WX(j, 2, k + 1) * Z(jr, i + 1)
                                + WY(j, 3, k) * Z(jr - 1, i) + WY(j, 2, k) * Z(j, i);
                    Z(jr, i) = (b1[k] + lnb) / (WX(j, 2, k) + WX(j, 2, k + 1) + WY(j, 3, k) + WY(j, 2, k));
                }
                const T za = Z(jr, ca), zbb = Z(jr, ca + 1);
                if (ca > 0) __builtin_nontemporal_store(za, &gx[jr * s + ca]);
                __builtin_nontemporal_store(zbb, &gx[jr * s + ca + 1]);
                // column 0 is the boundary: its right-hand side entry is never
                // written and may hold a stale word of another level's layout
                // (any bit pattern, NaN included), so it stays out of the dot
                if (want_dot) dot += (ca > 0 ? (double)b1[0] * (double)za : 0.0) + (double)b1[1] * (double)zbb;
            }
        }
        lds_barrier();  // the walk reads no global value another thread writes
    };
    // rows j0 - 1 .. j1, after the red values of rows j0 - 2 and j0 - 1 (the
    // flow cell's last band has one row more)
    using First = Par<FLOW ? 1 : 0>;
    using Second = Par<FLOW ? 0 : 1>;
    body(First{}, j0 - 3, std::true_type{});
    body(Second{}, j0 - 2, std::true_type{});
#pragma unroll 1
    for (int j = j0 - 1; j <= j0 + (n / (BS / (n >> 1))) + (FLOW ? 1 : 0); j += 2) {
        body(First{}, j, std::false_type{});
        body(Second{}, j + 1, std::false_type{});
    }
    __syncthreads();  // the new z is complete
    return want_dot ? block_sum<BS>(dot, red) : 0.0;
}

// The compiler's choice of a call or not (the ..._here forms are always inlined:
// the 1024-thread solver needs that, forced everywhere it cost the 512-thread
// mixed form 482 -> 616 ms per 4096 particles at h = 1/512).
template <int BS, bool FINE, bool FLOW, typename T, typename LEVEL, typename COARSE>
__device__ void walk_down(const LEVEL& L, const COARSE& C, T* __restrict__ b, const T* __restrict__ Q, T alpha,
                          T* __restrict__ X, const T* __restrict__ Pn, T* __restrict__ ring, bool coarse_red = false)
{
    walk_down_here<BS, FINE, FLOW>(L, C, b, Q, alpha, X, Pn, ring, coarse_red);
}
template <int BS, bool FINE, bool FLOW, typename T, typename LEVEL>
__device__ double walk_up(const LEVEL& L, const T* __restrict__ e, int sc, const T* __restrict__ b,
                          T* __restrict__ x, bool want_dot, T* __restrict__ ring, double* red)
{
    return walk_up_here<BS, FINE, FLOW>(L, e, sc, b, x, want_dot, ring, red);
}

}  // namespace mls
