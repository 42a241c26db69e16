// Strips of a multigrid level in registers: what the register-resident
// solvers (resident.hip, resident7.hip) share.  A thread owns a strip of one
// column, held by colour (resident.hip explains the layout); here are its
// weights, the exchange with the neighbouring strips, a coarse level's V(1,1)
// visit and the exact h = 1/4 solve.
#pragma once

#include "common.h"
#include "lanes.h"

namespace mls {

namespace {


// c ? a : b of two values in registers (by value: a select of their addresses
// would put the arrays they come from into scratch memory)
template <typename T>
__device__ __forceinline__ T pick(bool c, T a, T b) { return c ? a : b; }

// LDS accesses of one wave complete in order; the fences keep the compiler's
// order, without a wait
__device__ __forceinline__ void wave_order()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}
// workgroup barrier that orders the LDS only
__device__ __forceinline__ void group_order()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}
template <int NT>
__device__ __forceinline__ void order()
{
    if constexpr (NT > 64) group_order();
    else wave_order();
}

// ------------------------------------------------------------ strips --
// A level of width n = 2^LG spread over NT threads, P row pairs each: strips
// of 2P rows, NT / n of them (those past the problem's rows hold no valid
// node).
template <int LG, int P, int NT, bool FLOW>
struct Geo {
    static constexpr int n = 1 << LG;
    static constexpr int rows = FLOW ? n + 1 : n;           // rows 0 .. rows - 1 hold the unknowns
    static constexpr int strips = NT / n;
    static constexpr int pairs = strips * P;                // row pairs held
    // red residuals, [pair][column], after a zero row; at least as many rows
    // as the coarser level's threads read
    static constexpr int need = n == 8 ? 5 : n == 16 ? 16 : n == 32 ? (FLOW ? 24 : 16) : (FLOW ? 64 : 32);
    static constexpr int rs = ((pairs > need ? pairs : need) + 1) * n;
    static_assert(NT % n == 0 && 2 * pairs >= rows, "whole strips that cover the rows");
    static __device__ __forceinline__ bool valid(int i, int j) { return i > 0 && j < rows && (FLOW || j > 0); }
};

template <typename T, int P>
struct Weights {
    T wr[2][P], o[2][P], inv[2][P];  // [colour][pair]: east edge, the vertical edge out of the pair, 1 / diagonal
    T s[P];                          // the edge inside the pair
};
constexpr int kW = 7;  // values of T per pair in Weights

// Weights of the thread's nodes.  cell(i, j, lo, up) gives the coefficients
// of the lower and upper triangle of cell (i, j), j >= 0.  Column 0 keeps its
// east edges (the operator's flux into column 1).  On the coarse levels,
// where only neighbour sums are formed, the vertical edges to the boundary
// are dropped once they are in the diagonal.
template <bool COARSE, typename G, typename T, int P, typename CELL>
__device__ __forceinline__ void make_weights(Weights<T, P>& W, int t, CELL cell)
{
    constexpr int n = G::n;
    const int i = t & (n - 1), row0 = (t / n) * 2 * P;
    const bool e = i & 1;
    double up0 = 0.0;   // upper triangle of the cell row below
    double wy0 = 0.0;   // vertical edge from the row below
    if (row0 > 0) {
        double lo = 0.0;
        if (row0 - 1 < n) cell(i, row0 - 1, lo, up0);
        wy0 = 0.5 * (up0 + west(lo));
    } else {
        (void)west(up0);
    }
    double wx[2 * P], wy[2 * P];
#pragma unroll
    for (int a = 0; a < 2 * P; ++a) {
        double lo = 0.0, up = 0.0;
        if (row0 + a < n) cell(i, row0 + a, lo, up);
        wx[a] = 0.5 * (lo + up0);
        wy[a] = 0.5 * (up + west(lo));
        up0 = up;
    }
#pragma unroll
    for (int k = 0; k < P; ++k) {
        const double below = k ? wy[2 * k - 1] : wy0, in = wy[2 * k], above = wy[2 * k + 1];
        const double x0 = wx[2 * k], x1 = wx[2 * k + 1], l0 = west(x0), l1 = west(x1);
        const int j0 = row0 + 2 * k;
        const bool v0 = G::valid(i, j0), v1 = G::valid(i, j0 + 1);
#pragma unroll
        for (int c = 0; c < 2; ++c) {  // c = 0: red
            const bool hi = (c == 0) == e;  // the colour's node is the pair's upper row
            const bool v = hi ? v1 : v0;
            const T l = T(hi ? l1 : l0), r = T(hi ? x1 : x0), o = T(hi ? above : below), si = T(in);
            const int j = j0 + (hi ? 1 : 0);
            W.wr[c][k] = G::valid(1, j) ? r : T(0);
            W.o[c][k] = v && !(COARSE && !G::valid(i, j + (hi ? 1 : -1))) ? o : T(0);
            W.inv[c][k] = v ? T(1) / (l + r + si + o) : T(0);
        }
        W.s[k] = (v0 || v1) ? T(in) : T(0);
    }
}

template <typename T, int P, int NT>
__device__ __forceinline__ void store_weights(const Weights<T, P>& W, T* m, int t)
{
#pragma unroll
    for (int k = 0; k < P; ++k) {
        T* q = m + k * kW * NT + t;
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            q[(3 * c + 0) * NT] = W.wr[c][k];
            q[(3 * c + 1) * NT] = W.o[c][k];
            q[(3 * c + 2) * NT] = W.inv[c][k];
        }
        q[6 * NT] = W.s[k];
    }
}

template <typename T, int P, int NT>
__device__ __forceinline__ void load_weights(Weights<T, P>& W, const T* m, int t)
{
#pragma unroll
    for (int k = 0; k < P; ++k) {
        const T* q = m + k * kW * NT + t;
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            W.wr[c][k] = q[(3 * c + 0) * NT];
            W.o[c][k] = q[(3 * c + 1) * NT];
            W.inv[c][k] = q[(3 * c + 2) * NT];
        }
        W.s[k] = q[6 * NT];
    }
}

// LDS offsets of a thread on a level, and of its red nodes' corrections on
// the coarser level's grid (row stride n / 2): the coarse node itself in
// even columns, the middle of its diagonal edge in odd ones
template <typename G, int P, bool REDO>
struct At {
    int t, ex[2], rs, pe0, pe1;
    __device__ __forceinline__ At()
    {
        constexpr int n = G::n, sc = n / 2;
        t = threadIdx.x;
        // REDO: formed again at each use; held through the iterations, the
        // offsets of all levels cost registers that the kernel has not got
        if constexpr (REDO) asm volatile("" : "+v"(t));
        const int i = t & (n - 1), m0 = (t / n) * P, e = i & 1;
        ex[0] = t + (e ? n : -n);  // the strip that the red nodes look into
        ex[1] = t + (e ? -n : n);
        rs = (m0 + 1) * n + i;
        pe0 = m0 * sc + (i >> 1);
        pe1 = pe0 + (e ? sc + 1 : 0);
    }
};

// O[k]: the vertical neighbour outside the pair of this thread's colour-C
// node k, X holding the other colour.  Red nodes of even columns and black
// nodes of odd ones look down, the others up; the neighbouring strip's thread
// of the same column looks the same way, so each publishes one value.
template <typename G, int C, typename T, int P>
__device__ __forceinline__ void publish(const T (&X)[P], T* ex, int t)
{
    const bool up = ((t & 1) != 0) == (C == 0);
    ex[t] = pick(up, X[0], X[P - 1]);
}
template <typename G, int C, typename T, int P, bool REDO>
__device__ __forceinline__ void outer(const T (&X)[P], const T* ex, const At<G, P, REDO>& at, T (&O)[P])
{
    const bool up = ((at.t & 1) != 0) == (C == 0);
    const T edge = ex[at.ex[C]];
#pragma unroll
    for (int k = 0; k < P; ++k) {
        const T a = k + 1 < P ? X[k + 1 < P ? k + 1 : 0] : edge;
        const T b = k > 0 ? X[k > 0 ? k - 1 : 0] : edge;
        O[k] = pick(up, a, b);
    }
}

// sum of w X over the neighbours of the colour-C node k.  The west edge's
// weight belongs to the west neighbour, which sends the product.
template <int C, typename T, int P>
__device__ __forceinline__ T nb(const Weights<T, P>& W, const T (&X)[P], const T (&O)[P], int k)
{
    return west(W.wr[1 - C][k] * X[k]) + W.wr[C][k] * east(X[k]) + (W.s[k] * X[k] + W.o[C][k] * O[k]);
}

// Restriction: the red residual of the coarse node and of its two neighbours
// along the triangle diagonal.  q points at the coarse node's own entry.
template <int NF, typename T>
__device__ __forceinline__ T restricted(const T* q)
{
    return q[0] + T(0.5) * (q[1] + q[-NF - 1]);
}

// ----------------------------------------------------- coarse memory --
// A coarse level's LDS: weights, red residuals, its solution on the node
// grid.  During the set-up the residuals' memory of a level holds the
// coefficients of the next coarser one.
template <typename T, int LG, int P, int NT, bool FLOW>
struct CoarseMem {
    using G = Geo<LG, P, NT, FLOW>;
    T w[kW * P * NT];
    T rs[G::rs];
};

// Rows of a level's solution grid (stride n: column n of a row is column 0 of
// the next, both boundary and zero) under a finer level GF: those that its
// threads write and those that the finer level's read; one zero row and one
// zero entry follow.
template <typename GF, typename G>
constexpr int grid_rows = GF::pairs > 2 * G::pairs ? GF::pairs : 2 * G::pairs;

// ----------------------------------------------------- h = 1/4, exact --
// Unknowns (i, j), 1 <= i <= 3; rows 1 .. 3, or 0 .. 4 on the flow cell
template <bool FLOW>
struct Exact {
    static constexpr int rows = FLOW ? 5 : 3, j0 = FLOW ? 0 : 1, N = 3 * rows;
};

// inverse of the h = 1/4 operator by Gauss-Jordan sweeps in place (an
// M-matrix: no pivoting); one wave, lane u < N holds row u in registers and
// stores it as column u of A (the inverse is symmetric).  Dirichlet problem.
template <typename T>
__device__ __forceinline__ void exact_build(const T* kap, double* A, int t = threadIdx.x)
{
    using E = Exact<false>;
    constexpr int N = E::N;
    const int u = t < N ? t : N - 1;
    const int i = u % 3 + 1, j = u / 3 + E::j0;
    auto lo = [&](int ii, int jj) { return (jj >= 0 && jj < 4) ? (double)kap[2 * (4 * jj + ii)] : 0.0; };
    auto up = [&](int ii, int jj) { return (jj >= 0 && jj < 4) ? (double)kap[2 * (4 * jj + ii) + 1] : 0.0; };
    const double we = (double)T(0.5 * (lo(i, j) + up(i, j - 1))), ww = (double)T(0.5 * (lo(i - 1, j) + up(i - 1, j - 1)));
    const double wn = (double)T(0.5 * (up(i, j) + lo(i - 1, j))), ws = (double)T(0.5 * (up(i, j - 1) + lo(i - 1, j - 1)));
    const double d = ww + we + ws + wn;
    double a[N];
#pragma unroll
    for (int v = 0; v < N; ++v) {
        double x = 0.0;
        if (v == u) x = d;
        else if (v == u - 1 && i > 1) x = -ww;
        else if (v == u + 1 && i < 3) x = -we;
        else if (v == u - 3) x = -ws;
        else if (v == u + 3) x = -wn;
        a[v] = x;
    }
#pragma unroll
    for (int p = 0; p < N; ++p) {
        double row[N];  // the pivot row, in every lane
#pragma unroll
        for (int v = 0; v < N; ++v) row[v] = read_lane(a[v], p);
        const double r = 1.0 / row[p];
        const bool own = u == p;
        const double f = own ? 0.0 : a[p] * r;
#pragma unroll
        for (int v = 0; v < N; ++v) {
            if (v == p) a[v] = own ? r : -f;
            else a[v] = own ? a[v] * r : a[v] - f * row[v];
        }
    }
    if (t < N)
#pragma unroll
        for (int v = 0; v < N; ++v) A[N * v + u] = a[v];
}

// The flow cell's h = 1/4 visit as a matrix: V(1,1) there and the exact
// tridiagonal solve of h = 1/2, as the general solver ends its cycle, so that
// both need the same iterations and stop equally close to the solution (with
// the exact inverse in its place the cycle was a little stronger, and stopped
// with up to 1.5 times the error).  One wave; lane u < 15 holds row u, every
// column's value at unknown u, through the sweeps (neighbours by moves within
// the row of 16 lanes), and stores it as column u of A (the visit is
// symmetric).  kap: the coefficients of h = 1/4.
template <typename T>
__device__ __forceinline__ void visit2_build(const T* kap, double* A, int t = threadIdx.x)
{
    const int u = t < 15 ? t : 14;
    const int i = u % 3 + 1, j = u / 3;
    auto lo = [&](int ii, int jj) { return (jj >= 0 && jj < 4) ? (double)kap[2 * (4 * jj + ii)] : 0.0; };
    auto up = [&](int ii, int jj) { return (jj >= 0 && jj < 4) ? (double)kap[2 * (4 * jj + ii) + 1] : 0.0; };
    double we = 0.5 * (lo(i, j) + up(i, j - 1)), ww = 0.5 * (lo(i - 1, j) + up(i - 1, j - 1));
    const double wn = 0.5 * (up(i, j) + lo(i - 1, j)), ws = 0.5 * (up(i, j - 1) + lo(i - 1, j - 1));
    const double inv = 1.0 / (ww + we + ws + wn);
    if (i == 1) ww = 0.0;  // into the boundary columns
    if (i == 3) we = 0.0;
    const bool red = !((i + j) & 1);
    auto nb = [&](double x) {
        return (ww * dpp<0x111>(x) + we * dpp<0x101>(x)) + (ws * dpp<0x113>(x) + wn * dpp<0x103>(x));
    };
    // h = 1/2: unknowns (1, 0), (1, 1), (1, 2), in every lane
    auto clo = [&](int ii, int jj) {
        return 0.25 * (lo(2 * ii, 2 * jj) + lo(2 * ii + 1, 2 * jj) + lo(2 * ii + 1, 2 * jj + 1) + up(2 * ii + 1, 2 * jj));
    };
    auto cup = [&](int ii, int jj) {
        return 0.25 * (up(2 * ii, 2 * jj) + up(2 * ii, 2 * jj + 1) + up(2 * ii + 1, 2 * jj + 1) + lo(2 * ii, 2 * jj + 1));
    };
    const double e0 = 0.5 * (clo(0, 0) + cup(1, 0)), e1 = 0.5 * (clo(0, 1) + cup(1, 1));
    const double d0 = 0.5 * (clo(0, 0) + clo(1, 0)) + e0;
    const double d1 = 0.5 * (clo(0, 1) + cup(0, 0) + clo(1, 1) + cup(1, 0)) + e0 + e1;
    const double d2 = 0.5 * (cup(0, 1) + cup(1, 1)) + e1;
    const double r0 = 1.0 / d0, r1 = 1.0 / (d1 - e0 * e0 * r0), r2 = 1.0 / (d2 - e1 * e1 * r1);
    // a red node's correction: that of its own h = 1/2 node (column 2), or half
    // of the one at the other end of its diagonal edge (the boundary's is zero)
    const int J = i == 3 ? (j - 1) / 2 : i == 1 ? (j + 1) / 2 : j / 2;
    const double share = !red ? 0.0 : i == 2 ? 1.0 : 0.5;
    // (three columns at a time hide each other's latency; all fifteen would take
    // more registers than the rest of the kernel)
#pragma unroll 3
    for (int v = 0; v < 15; ++v) {
        const double b = u == v ? 1.0 : 0.0;
        double z = red ? b * inv : 0.0;
        double s = nb(z);
        z = red ? z : (b + s) * inv;
        // the red residual, restricted to (2, 2J) along the diagonal
        s = nb(z);
        s = red ? s : 0.0;
        const double c = s + 0.5 * (dpp<0x104>(s) + dpp<0x114>(s));
        const double c0 = read_lane(c, 1), c1 = read_lane(c, 7), c2 = read_lane(c, 13);
        const double y1 = c1 + e0 * r0 * c0;
        const double x2 = (c2 + e1 * r1 * y1) * r2;
        const double x1 = (y1 + e1 * x2) * r1, x0 = (c0 + e0 * x1) * r0;
        z += share * (J == 0 ? x0 : J == 1 ? x1 : x2);
        s = nb(z);
        z = red ? z : (b + s) * inv;
        s = nb(z);
        if (t < 15) A[15 * v + u] = red ? (b + s) * inv : z;
    }
}

// e2 = A (restriction of the level h = 1/8's red residuals), A from exact_build
// or visit2_build; one wave
template <bool FLOW, typename T>
__device__ __forceinline__ void exact_solve(const T* rs3, const double* A, T* e2, int t = threadIdx.x)
{
    using E = Exact<FLOW>;
    const int u = t < E::N ? t : E::N - 1;
    const int i = u % 3 + 1, j = u / 3 + E::j0;
    const double b = (double)restricted<8>(rs3 + 8 * (j + 1) + 2 * i);
    double v = 0.0, w = 0.0;
#pragma unroll
    for (int q = 0; q < E::N; ++q) (q & 1 ? w : v) += A[E::N * q + u] * read_lane(b, q);
    if (t < E::N) e2[j * 4 + i] = T(v + w);
}

// ------------------------------------------------------ coarse levels --

// the down-leg after the first red sweep (zr = b / d): black sweep, red
// residual into rs
template <typename G, int NT, typename T, int P, bool REDO>
__device__ __forceinline__ void down_leg(const Weights<T, P>& W, const At<G, P, REDO>& at, const T (&bb)[P], T (&zr)[P],
                                         T (&zb)[P], T* ex0, T* ex1, T* rs)
{
    T O[P];
    publish<G, 1>(zr, ex0, at.t);
    order<NT>();
    outer<G, 1>(zr, ex0, at, O);
#pragma unroll
    for (int k = 0; k < P; ++k) zb[k] = (bb[k] + nb<1>(W, zr, O, k)) * W.inv[1][k];
    publish<G, 0>(zb, ex1, at.t);
    order<NT>();
    outer<G, 0>(zb, ex1, at, O);
#pragma unroll
    for (int k = 0; k < P; ++k) rs[at.rs + k * G::n] = nb<0>(W, zb, O, k);
}

// the up-leg: coarse correction at the red nodes, black sweep, red sweep.
// Surplus and boundary nodes read grid entries that are zero or feed only
// zero weights.
template <typename G, int NT, typename T, int P, bool REDO>
__device__ __forceinline__ void up_leg(const Weights<T, P>& W, const At<G, P, REDO>& at, const T (&br)[P], const T (&bb)[P],
                                       T (&zr)[P], T (&zb)[P], T* ex0, T* ex1, const T* ec)
{
    constexpr int sc = G::n / 2;
    T O[P];
#pragma unroll
    for (int k = 0; k < P; ++k) zr[k] += T(0.5) * (ec[at.pe0 + k * sc] + ec[at.pe1 + k * sc]);
    publish<G, 1>(zr, ex0, at.t);
    order<NT>();
    outer<G, 1>(zr, ex0, at, O);
#pragma unroll
    for (int k = 0; k < P; ++k) zb[k] = (bb[k] + nb<1>(W, zr, O, k)) * W.inv[1][k];
    publish<G, 0>(zb, ex1, at.t);
    order<NT>();
    outer<G, 0>(zb, ex1, at, O);
#pragma unroll
    for (int k = 0; k < P; ++k) zr[k] = (br[k] + nb<0>(W, zb, O, k)) * W.inv[0][k];
}

// One V(1,1) visit of a coarse level held by NT threads: right-hand side from
// the finer level's red residuals, down-leg, the levels below, up-leg; the
// level's solution goes to sol.  Nodes outside the problem take whatever
// right-hand side lies there: their inverse diagonal and weights are zero.
template <int LG, int P, int NT, bool FLOW, bool REDO, typename T, typename BELOW>
__device__ __forceinline__ void coarse_visit(const T* rsf, CoarseMem<T, LG, P, NT, FLOW>& m, T* sol, const T* ec,
                                             T* ex0, T* ex1, BELOW below)
{
    using G = Geo<LG, P, NT, FLOW>;
    constexpr int n = G::n, nf = 2 * n;
    T br[P], bb[P], zr[P], zb[P];
    {
        const At<G, P, REDO> at;
        const int i = at.t & (n - 1), e = i & 1, m0 = (at.t / n) * P;
        Weights<T, P> W;
        load_weights<T, P, NT>(W, m.w, at.t);
        const T* qr = rsf + (2 * m0 + e + 1) * nf + 2 * i;
        const T* qb = rsf + (2 * m0 + 2 - e) * nf + 2 * i;
#pragma unroll
        for (int k = 0; k < P; ++k) {
            br[k] = restricted<nf>(qr + 2 * nf * k);
            bb[k] = restricted<nf>(qb + 2 * nf * k);
            zr[k] = br[k] * W.inv[0][k];
        }
        down_leg<G, NT>(W, at, bb, zr, zb, ex0, ex1, m.rs);
    }
    order<NT>();
    below();
    order<NT>();
    {
        // offsets and weights again: kept, they would hold registers through
        // the levels below
        const At<G, P, REDO> at;
        const int i = at.t & (n - 1), e = i & 1, m0 = (at.t / n) * P;
        Weights<T, P> W;
        load_weights<T, P, NT>(W, m.w, at.t);
        up_leg<G, NT>(W, at, br, bb, zr, zb, ex0, ex1, ec);
        T* gr = sol + (2 * m0 + e) * n + i;
        T* gb = sol + (2 * m0 + 1 - e) * n + i;
#pragma unroll
        for (int k = 0; k < P; ++k) {
            gr[2 * n * k] = zr[k];
            gb[2 * n * k] = zb[k];
        }
    }
}

// coarse triangle coefficients from the four children of each
template <typename T, int LC, int NT, typename CELL>
__device__ __forceinline__ void coarsen(T* kc, int t, CELL cell)
{
    constexpr int nc = 1 << LC;
    for (int q = t; q < nc * nc; q += NT) {
        const int i = 2 * (q & (nc - 1)), j = 2 * (q >> LC);
        double l00, u00, l10, u10, l01, u01, l11, u11;
        cell(i, j, l00, u00);
        cell(i + 1, j, l10, u10);
        cell(i, j + 1, l01, u01);
        cell(i + 1, j + 1, l11, u11);
        kc[2 * q] = T(0.25 * (l00 + l10 + l11 + u10));
        kc[2 * q + 1] = T(0.25 * (u00 + u11 + u01 + l01));
    }
}

template <typename T, int LG, int P, int NT, bool FLOW>
__device__ __forceinline__ void coarse_weights(CoarseMem<T, LG, P, NT, FLOW>& m, const T* kap, int t = threadIdx.x)
{
    using G = Geo<LG, P, NT, FLOW>;
    Weights<T, P> W;
    make_weights<true, G>(W, t, [&](int i, int j, double& lo, double& up) {
        lo = (double)kap[2 * (j * G::n + i)];
        up = (double)kap[2 * (j * G::n + i) + 1];
    });
    store_weights<T, P, NT>(W, m.w, t);
}

}  // namespace

}  // namespace mls
