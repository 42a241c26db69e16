// A V(1,1) cycle at h = 1/128 (Dirichlet rows) with the level's nodes in
// registers, for the resident solver of that level (resident7.hip) and for the
// row-walking solvers of the finer levels, whose h = 1/128 visit it is.
//
//  * Two columns per thread: with a = 2 lane and b = a + 1, row k of the
//    thread's strip has one node of each colour, red in column a where k is
//    even.  No lane is idle and no select depends on the lane.  A node's
//    horizontal neighbours are the thread's own other column and one adjacent
//    lane.
//  * A strip exchanges its first and last row's values of one colour with
//    the strips above and below (the edge's weight is the lower strip's, which
//    sends the product).
//  * After the down-leg nothing of z is kept: the up-leg forms the red values
//    again from r, and the black ones are swept anyway.
//  * The level h = 1/64 has column I = lane in the same threads, half as many
//    rows each, so restriction and prolongation stay in registers but for one
//    value per thread.  The levels from h = 1/32 down are those of
//    resident.hip.
#pragma once

#include <type_traits>

#include "strips.h"

namespace mls {

namespace {

template <int NT>
constexpr int kRows7 = 8192 / NT;  // rows per thread: two columns each, 128 x 128 nodes
template <int NT>
using Geo6 = Geo<6, kRows7<NT> / 4, NT, false>;
using G5 = Geo<5, 1, 512, false>;
using G4 = Geo<4, 2, 64, false>;
using G3 = Geo<3, 1, 64, false>;
constexpr int kAhead = 2;                             // rows whose weights are asked for ahead of their use
constexpr int kSol5 = grid_rows<Geo6<512>, G5> * 32;  // the h = 1/32 level's solution grid

// Exchange between strips, one value per thread: a1, a2 and in rs6 also a3 and
// a0, which are not in use between the restriction onto h = 1/32 and the h =
// 1/32 level's solution, whose place rs6 is.  The coarse levels' exchange reads
// up to one strip outside a1 and a2, with zero weight.  Between cycles the
// memory may hold any finite values.
template <typename T, int NT>
struct Exchange7 {
    T pad[64];
    T a1[NT], a2[NT];
    T rs6[Geo6<NT>::rs + 33];
    static constexpr int sol_off = Geo6<NT>::rs - kSol5;
    static_assert(Geo6<NT>::rs >= 2 * NT, "a3 and a0 fit in rs6, before its trailing zeros");
};

// the levels from h = 1/32 down
template <typename T>
struct Levels5 {
    CoarseMem<T, 5, 1, 512, false> c5;
    CoarseMem<T, 4, 2, 64, false> c4;
    CoarseMem<T, 3, 1, 64, false> c3;
    T e4[(grid_rows<G5, G4> + 1) * 16 + 1];
    T e3[(grid_rows<G4, G3> + 1) * 8 + 1];
    T e2[(G3::pairs + 1) * 4 + 1];
    double cinv[81];
};

// a value that the compiler forms again at each use instead of holding what
// follows from it (addresses) through the loops
__device__ __forceinline__ int again(int v)
{
    asm volatile("" : "+v"(v));
    return v;
}

// the h = 1/64 level's weights of a thread, from that level's coefficients
template <typename T, int NT>
__device__ __forceinline__ void weights6(T* w6, const T* k6, int t)
{
    Weights<T, kRows7<NT> / 4> W;
    make_weights<true, Geo6<NT>>(W, t, [&](int i, int j, double& lo, double& up) {
        lo = (double)k6[2 * (j * 64 + i)];
        up = (double)k6[2 * (j * 64 + i) + 1];
    });
    store_weights<T, kRows7<NT> / 4, 64>(W, w6, t & 63);
}

// weights of the levels from h = 1/32 (coefficients k5) down; a barrier before
// and after it
template <typename T>
__device__ __forceinline__ void build_levels5(Levels5<T>& m, const T* k5, int t)
{
    if (t < 512) coarse_weights(m.c5, k5, t);
    if (t < 64) {
        auto cell = [](const T* kc, int w) {
            return [=](int i, int j, double& lo, double& up) {
                lo = (double)kc[2 * (j * w + i)];
                up = (double)kc[2 * (j * w + i) + 1];
            };
        };
        coarsen<T, 4, 64>(m.c5.rs, t, cell(k5, 32));
        wave_order();
        coarse_weights(m.c4, m.c5.rs, t);
        coarsen<T, 3, 64>(m.c4.rs, t, cell(m.c5.rs, 16));
        wave_order();
        coarse_weights(m.c3, m.c4.rs, t);
        coarsen<T, 2, 64>(m.c3.rs, t, cell(m.c4.rs, 8));
        wave_order();
        exact_build(m.c3.rs, m.cinv, t);
    }
}
template <typename T, int NT>
__device__ __forceinline__ void clear_levels5(Levels5<T>& m, int t)
{
    auto clear = [&](T* a, int c) { for (int k = t; k < c; k += NT) a[k] = T(0); };
    clear(m.c5.rs, sizeof(m.c5.rs) / sizeof(T));
    clear(m.c4.rs, sizeof(m.c4.rs) / sizeof(T));
    clear(m.c3.rs, sizeof(m.c3.rs) / sizeof(T));
    clear(m.e4, sizeof(m.e4) / sizeof(T));
    clear(m.e3, sizeof(m.e3) / sizeof(T));
    clear(m.e2, sizeof(m.e2) / sizeof(T));
}

// z = V r (zr, zb from rr, rb: [row], the red and the black node).  edge(k, t):
// row k's edges x (a - b), y (b - east a), z (a, to the row above), w (b, to the
// row above); inv(k, colour, t): inverse diagonals, zero outside the problem.
// w6: the thread's wave's h = 1/64 weights.
template <typename T, int NT, typename EDGE, typename INV>
__device__ __forceinline__ void cycle7(const T (&rr)[kRows7<NT>], const T (&rb)[kRows7<NT>], T (&zr)[kRows7<NT>],
                                       T (&zb)[kRows7<NT>], EDGE edge, INV inv, const T* w6, Exchange7<T, NT>& x,
                                       Levels5<T>& m, int t0, int wv)
{
    constexpr int R = kRows7<NT>, top = NT / 64 - 1;
    T* a0 = x.rs6 + NT;
    T* a3 = x.rs6;
    using Red = std::integral_constant<int, 0>;
    using Black = std::integral_constant<int, 1>;
    // neighbour sums of colour C (0: red) from the other colour's X; dn:
    // the product from the strip below, up: the value of the one above
    auto sums = [&](auto C, const T (&X)[R], T dn, T up, auto use) {
        constexpr int c = decltype(C)::value;
        const int u = again(t0);
        decltype(edge(0, 0)) w[R];
        T d[R];
        T below = dn;
#pragma unroll
        for (int k = 0; k < kAhead; ++k) { w[k] = edge(k, u); d[k] = inv(k, c, u); }
#pragma unroll
        for (int k = 0; k < R; ++k) {
            if (k + kAhead < R) {
                w[k + kAhead < R ? k + kAhead : 0] = edge(k + kAhead, u);
                d[k + kAhead < R ? k + kAhead : 0] = inv(k + kAhead, c, u);
            }
            const bool col_b = (k & 1) == (c == 0);  // this colour's column in row k
            const T v = (T)(col_b ? w[k].w : w[k].z);
            const T hw = (T)w[k].y;
            const T far = col_b ? hw * east(X[k]) : west(hw * X[k]);
            const T nxt = k + 1 < R ? X[k + 1 < R ? k + 1 : 0] : up;
            use(k, ((T)w[k].x * X[k] + far) + (v * nxt + below), d[k]);
            below = (T)(col_b ? w[k].z : w[k].w) * X[k];  // X's node: the other column
        }
    };
    {
        const int t = again(t0);
        const auto e7 = edge(R - 1, t);
#pragma unroll
        for (int k = 0; k < R; ++k) zr[k] = rr[k] * inv(k, 0, t);
        a0[t] = (T)e7.w * zr[R - 1];
        x.a1[t] = zr[0];
        if (t < 33) x.rs6[Geo6<NT>::rs + t] = T(0);
    }
    group_order();
    int t = again(t0), lane = t & 63;
    sums(Black(), zr, wv > 0 ? a0[t - 64] : T(0), wv < top ? x.a1[t + 64] : T(0),
         [&](int k, T s, T d) { zb[k] = (rb[k] + s) * d; });
    x.a2[t] = (T)edge(R - 1, t).z * zb[R - 1];
    a3[t] = zb[0];
    group_order();
    // the red residual
    sums(Red(), zb, wv > 0 ? x.a2[t - 64] : T(0), wv < top ? a3[t + 64] : T(0), [&](int k, T s, T) { zr[k] = s; });
    a0[t] = zr[R - 1];
    group_order();
    T E[R / 2 + 1];
    {
        constexpr int P6 = R / 4;
        const bool e = lane & 1;
        T br[P6], bb[P6], yr[P6], yb[P6];
        {
            // the diagonal's lower end, column 2 lane - 1: of the adjacent
            // lane (lane 0 is the boundary column)
            const T q0 = wv > 0 ? a0[t - 65] : T(0);
            T b[R / 2];
#pragma unroll
            for (int J = 0; J < R / 2; ++J)
                b[J] = zr[2 * J] + T(0.5) * (zr[2 * J + 1] + (J ? west(zr[J ? 2 * J - 1 : 0]) : q0));
            const At<Geo6<NT>, P6, true> at;
            Weights<T, P6> W;
            load_weights<T, P6, 64>(W, w6, again(t0) & 63);
#pragma unroll
            for (int k = 0; k < P6; ++k) {
                br[k] = pick(e, b[2 * k + 1], b[2 * k]);
                bb[k] = pick(e, b[2 * k], b[2 * k + 1]);
                yr[k] = br[k] * W.inv[0][k];
            }
            down_leg<Geo6<NT>, NT>(W, at, bb, yr, yb, x.a1, x.a2, x.rs6);
        }
        group_order();
        T* sol5 = x.rs6 + Exchange7<T, NT>::sol_off;
        auto visit5 = [&]() {
            coarse_visit<5, 1, 512, false, true>(x.rs6, m.c5, sol5, m.e4, x.a1, x.a2, [&]() {
                if (wv == 0)
                    coarse_visit<4, 2, 64, false, true>(m.c5.rs, m.c4, m.e4, m.e3, x.a1, x.a2, [&]() {
                        coarse_visit<3, 1, 64, false, true>(m.c4.rs, m.c3, m.e3, m.e2, x.a1, x.a2, [&]() {
                            exact_solve<false>(m.c3.rs, m.cinv, m.e2, again(t0));
                        });
                    });
            });
        };
        if constexpr (NT == 512) {
            visit5();
        } else if (wv < 8) {  // by whole waves: the others meet its barriers
            visit5();
        } else {
#pragma unroll
            for (int k = 0; k < 6; ++k) group_order();
        }
        group_order();
        {
            const At<Geo6<NT>, P6, true> at;
            Weights<T, P6> W;
            load_weights<T, P6, 64>(W, w6, again(t0) & 63);
            up_leg<Geo6<NT>, NT>(W, at, br, bb, yr, yb, x.a1, x.a2, sol5);
        }
#pragma unroll
        for (int k = 0; k < P6; ++k) {
            E[2 * k] = pick(e, yb[k], yr[k]);
            E[2 * k + 1] = pick(e, yr[k], yb[k]);
        }
        a3[t] = E[0];
    }
    t = again(t0);
    lane = t & 63;
    const auto e7 = edge(R - 1, t);
    group_order();
    E[R / 2] = wv < top && lane < 63 ? a3[t + 65] : T(0);  // of the strip above, next column
#pragma unroll
    for (int J = 0; J < R / 2; ++J) {
        zr[2 * J] = rr[2 * J] * inv(2 * J, 0, t) + E[J];
        zr[2 * J + 1] = rr[2 * J + 1] * inv(2 * J + 1, 0, t) +
                        T(0.5) * (E[J] + (J + 1 < R / 2 ? east(E[J + 1]) : E[R / 2]));
    }
    a0[t] = (T)e7.w * zr[R - 1];
    x.a1[t] = zr[0];
    group_order();
    sums(Black(), zr, wv > 0 ? a0[t - 64] : T(0), wv < top ? x.a1[t + 64] : T(0),
         [&](int k, T s, T d) { zb[k] = (rb[k] + s) * d; });
    x.a2[t] = (T)edge(R - 1, t).z * zb[R - 1];
    a3[t] = zb[0];
    group_order();
    sums(Red(), zb, wv > 0 ? x.a2[t - 64] : T(0), wv < top ? a3[t + 64] : T(0),
         [&](int k, T s, T d) { zr[k] = (rr[k] + s) * d; });
}

}  // namespace

}  // namespace mls
