// Sampler kernels of MLS^2MC: the Gaussian potential (Sec. 2.1), the
// ESS-adaptive step for tempering and bridging (Secs. 3.1, 3.2, 3.4, 4.1),
// multinomial resampling (Sec. 2.4), and the pCN Markov move.
#include <algorithm>
#include <cmath>

#include "common.h"
#include "lanes.h"
#include "sampler.h"

namespace mls {

// ------------------------------------------------------------ potential --
// W lanes per particle, so that its row is read by neighbouring lanes.  (The
// grid is bounded, and the lanes go on to further particles.)  A wave per
// particle is the fastest from about 16 observations on, but wastes its lanes
// on shorter rows when there are many (us at 10^6 particles with 1 / 4 / 16 /
// 64 lanes: one observation 3.6 / 8.0 / 26 / 108, four 7.3 / 11 / 33 / 107,
// nine 33 / 20 / 33 / 107, 25 349 / 46 / 46 / 109; at 1000 particles and 25
// 4.3 / 3.0 / 2.8 / 2.9).
constexpr int64_t kRowBlocks = int64_t(1) << 22;
static unsigned row_blocks(int64_t N, int W)
{
    return (unsigned)std::min<int64_t>((N + 256 / W - 1) / (256 / W), kRowBlocks);
}

// sum over groups of W lanes, in every lane of the group
template <int W>
__device__ __forceinline__ double group_sum(double v)
{
#pragma unroll
    for (int off = W / 2; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

template <int W>
__global__ __launch_bounds__(256) void loglik_kernel(int64_t N, int nobs, const double* __restrict__ G,
                                                     const double* __restrict__ y, double inv_sigma,
                                                     double* __restrict__ phi)
{
    constexpr int64_t P = 256 / W;
    const int lane = threadIdx.x & (W - 1);
    for (int64_t q = blockIdx.x * P + threadIdx.x / W; q < N; q += gridDim.x * P) {
        double s = 0.0;
        for (int o = lane; o < nobs; o += W) {
            const double r = (y[o] - G[q * nobs + o]) * inv_sigma;
            s += r * r;
        }
        if constexpr (W == 64) s = lane63_sum(s);
        else s = group_sum<W>(s);
        if (lane == W - 1) phi[q] = 0.5 * s;
    }
}

int launch_loglik(mls2mc_ctx* ctx, int64_t N, const double* G, const double* y, double* phi,
                  hipStream_t s)
{
    if (N == 0) return MLS2MC_OK;
    const int nobs = ctx->nobs;
    const double inv_sigma = 1.0 / ctx->prob.sigma_n;
    if (nobs <= 4) loglik_kernel<1><<<row_blocks(N, 1), 256, 0, s>>>(N, nobs, G, y, inv_sigma, phi);
    else if (nobs <= 16) loglik_kernel<4><<<row_blocks(N, 4), 256, 0, s>>>(N, nobs, G, y, inv_sigma, phi);
    else loglik_kernel<64><<<row_blocks(N, 64), 256, 0, s>>>(N, nobs, G, y, inv_sigma, phi);
    MLS_CHECK_HIP(hipGetLastError());
    return MLS2MC_OK;
}

// ------------------------------------------------------------ next step --
// lw_j(t) = (-t*scale) d_j; its maximum is attained at min_j d_j (the factor
// is <= 0 and rounding is monotone), so one minimum serves every bisection
// step.  ESS(t) = (sum e^{lw-m})^2 / sum e^{2(lw-m)}.  The 64 bisection steps
// are a serial chain of evaluations, so what bounds the step is the latency
// of one evaluation, not its arithmetic:
//  * up to kStepSmall particles one workgroup keeps d in registers and an
//    evaluation is one exponential per element and one barrier (both sums
//    reduced by DPP together; 130 us -> 27 us at N = 200, where four barriers
//    and shuffles took 2 us per evaluation).  From 2049 particles on, where an
//    evaluation takes one CU 2.6 us and more, it first brackets the root in
//    about a dozen evaluations, and the bisection then evaluates only the
//    midpoints inside the bracket (ESS does not grow with t);
//  * beyond, a launch evaluates all midpoints of the next L bisection levels
//    (2^L - 1, every one by its own workgroups) and the next launch walks
//    down them: 64 / L launches instead of 64 passes of one workgroup
//    (474 us -> 76 us at N = 16384: 11 launches of 6.2 us).
// Both take the midpoints and the comparisons of plain bisection.  Where the
// line lies (us a call with its launches, inside / at an end; one workgroup
// with plain bisection in global memory, launches, one workgroup with the
// bracket): 2049 particles 150 / 13, 54 / 41-46, 52 / 13; 4096 196 / 13-16,
// 60 / 43-46, 59 / 13; 8192 283 / 18-22, 67 / 43-46, 80 / 13; 16384 460 /
// 28-34, 76 / 45-50, about 150 / 19.  Up to 4096 one workgroup loses neither;
// beyond, the steps inside, most of a run's, decide for the launches, and an
// end costs up to 30 us more than in one workgroup (until about 30000).
constexpr int kNS = 1024;
constexpr int64_t kStepSmall = 4096;

struct StepIn {
    int64_t N;
    const double* d;
    double scale, cur, tau, eps;
    double *out3, *logw, *w;
};

// {sum a, sum b} over the workgroup in every thread; red: two buffers of one
// entry per wave, used in turn so that one barrier serves
template <int BS>
__device__ __forceinline__ double2 pair_sum(double a, double b, double2 (*red)[BS / 64], int& turn)
{
    a = lane63_sum(a);
    b = lane63_sum(b);
    double2* r = red[turn];
    turn ^= 1;
    if ((threadIdx.x & 63) == 63) r[threadIdx.x >> 6] = make_double2(a, b);
    __syncthreads();
    double2 s = r[0];
#pragma unroll
    for (int k = 1; k < BS / 64; ++k) {
        s.x += r[k].x;
        s.y += r[k].y;
    }
    return make_double2(wave_uniform(s.x), wave_uniform(s.y));
}

template <int BS, int PER>
__global__ __launch_bounds__(BS) void next_step_small_kernel(StepIn A)
{
    __shared__ double red1[BS / 64];
    __shared__ double2 red[2][BS / 64];
    double d[PER];
    double dmin = INFINITY;
    int bad = 0;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int64_t j = threadIdx.x + k * BS;
        d[k] = j < A.N ? A.d[j] : INFINITY;  // an infinite difference weighs nothing below
        if (j < A.N && !isfinite(d[k])) bad = 1;
        dmin = fmin(dmin, d[k]);
    }
    dmin = -block_max<BS>(-dmin, red1);
    if (__syncthreads_or(bad)) {
        if (threadIdx.x == 0) A.out3[0] = A.out3[1] = A.out3[2] = NAN;
        return;
    }
    int turn = 0;
    double2 s;
    auto ess = [&](double t) {
        const double a = -t * A.scale;
        const double m = a * dmin;
        double s1 = 0.0, s2 = 0.0;
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            const double v = threadIdx.x + k * BS < A.N ? exp(a * d[k] - m) : 0.0;
            s1 += v;
            s2 += v * v;
        }
        s = pair_sum<BS>(s1, s2, red, turn);
        return s.x * s.x / s.y;
    };
    const double tmax = 1.0 - A.cur;
    const double tmin = A.eps < tmax ? A.eps : tmax;
    double t, e;
    bool at_end = false;
    const double e_end = ess(tmax);
    if ((e = e_end) >= A.tau) {
        t = tmax;
        at_end = true;
    } else if ((e = ess(tmin)) <= A.tau) {
        t = tmin;
        at_end = (tmin == tmax);
    } else if constexpr (PER <= 2) {
        double lo = tmin, hi = tmax, elo = e;
        double2 slo = s;
        for (int it = 0; it < 64; ++it) {
            const double mid = 0.5 * (lo + hi);
            if (mid == lo || mid == hi) break;  // adjacent: the remaining steps change nothing
            const double em = ess(mid);
            if (em >= A.tau) {
                lo = mid;
                elo = em;
                slo = s;
            } else {
                hi = mid;
            }
        }
        t = lo;
        e = elo;
        s = slo;
    } else {
        double known = tmin, out = tmax, elo = e;  // ESS(known) = elo >= tau > ESS(out)
        double2 slo = s;
        auto in = [&](double tt, double et) -> bool {
            if (!(et >= A.tau)) {
                out = tt;
                return false;
            }
            known = tt;
            elo = et;
            slo = s;
            return true;
        };
        // the root of log(ESS / tau) over log t by Chandrupatla's method (inverse
        // quadratic interpolation where it is safe, else the bracket's middle)
        double x1 = log(tmax), f1 = log(e_end / A.tau), x2 = log(tmin), f2 = log(e / A.tau), x3 = x1, f3 = f1;
        double at = 0.5;
        for (int it = 0; it < 48 && isfinite(f1) && isfinite(f2); ++it) {
            const double x = x1 + at * (x2 - x1), tt = exp(x);
            if (!(tt > known && tt < out)) break;
            const double et = ess(tt), f = log(et / A.tau);
            in(tt, et);
            if ((f >= 0.0) == (f1 >= 0.0)) {
                x3 = x1;
                f3 = f1;
            } else {
                x3 = x2;
                f3 = f2;
                x2 = x1;
                f2 = f1;
            }
            x1 = x;
            f1 = f;
            const double edge = 0x1p-50 / fabs(x2 - x1);  // a bracket of a few adjacent numbers ends it
            if (!(edge < 0.5)) break;
            const double xi = (x1 - x2) / (x3 - x2), phi = (f1 - f2) / (f3 - f2);
            at = 0.5;
            if (phi * phi < xi && (1.0 - phi) * (1.0 - phi) < 1.0 - xi)
                at = f1 / (f2 - f1) * (f3 / (f2 - f3)) + (x3 - x1) / (x2 - x1) * (f1 / (f3 - f1)) * (f2 / (f3 - f2));
            at = fmin(fmax(at, edge), 1.0 - edge);
        }
        // the bisection, whose midpoints outside the bracket are decided
        double lo = tmin, hi = tmax;
        for (int it = 0; it < 64; ++it) {
            const double mid = 0.5 * (lo + hi);
            if (mid == lo || mid == hi) break;
            if (mid <= known || (mid < out && in(mid, ess(mid)))) lo = mid;
            else hi = mid;
        }
        if (known != lo) {
            elo = ess(lo);
            slo = s;
        }
        t = lo;
        e = elo;
        s = slo;
    }
    const double a = -t * A.scale;
    const double lse = a * dmin + log(s.x);
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int64_t j = threadIdx.x + k * BS;
        if (j >= A.N) break;
        const double lw = a * d[k];
        if (A.logw) A.logw[j] = lw;
        if (A.w) A.w[j] = exp(lw - lse);
    }
    if (threadIdx.x == 0) {
        A.out3[0] = at_end ? 1.0 : A.cur + t;
        A.out3[1] = lse - log((double)A.N);
        A.out3[2] = e;
    }
}

// Scratch of the many-workgroup step, kept by the context: per-block minima,
// the state of the search before each round, and two buffers of partial sums
// [candidate][chunk].
enum { SS_LO, SS_HI, SS_S1, SS_S2, SS_DMIN, SS_MODE, SS_LEN = 8 };
enum { STEP_SEARCH = 0, STEP_DONE = 1, STEP_END = 2, STEP_BAD = 3 };
constexpr int kStepMin = 256;        // blocks of the minimum
constexpr int kStepParts = 576;      // most partial sums of a round
constexpr int kStepCand = 129;       // most candidates of a round
struct StepScratch {
    double minima[kStepMin];
    double state[68][SS_LEN];
    double2 part[2][kStepParts];
};
static_assert(sizeof(StepScratch) <= kStepScratchBytes, "the context's step scratch");

__global__ __launch_bounds__(256) void step_min_kernel(int64_t N, const double* __restrict__ d, StepScratch* S)
{
    __shared__ double red[4];
    double dmin = INFINITY;
    int bad = 0;
    for (int64_t j = blockIdx.x * 256 + threadIdx.x; j < N; j += gridDim.x * 256) {
        const double v = d[j];
        if (!isfinite(v)) bad = 1;
        dmin = fmin(dmin, v);
    }
    dmin = -block_max<256>(-dmin, red);
    bad = __syncthreads_or(bad);
    if (threadIdx.x == 0) S->minima[blockIdx.x] = bad ? NAN : dmin;
}

struct StepState {
    double lo, hi, s1, s2, dmin;
    int mode;
};

// The search's state before round r (each of L levels): the state before
// round r - 1 advanced by that round's sums.  Every workgroup forms it for
// itself; e, s1 and s2 are LDS arrays of kStepCand entries.  nmin: blocks of
// the minimum; levels: bisection levels of round r - 1.
template <int BS>
__device__ StepState step_state(const StepIn& A, const StepScratch* S, int r, int nmin, int L, int levels, int chunks,
                                double* e, double* s1, double* s2)
{
    __shared__ double red[BS / 64];
    StepState st;
    const double tmax = 1.0 - A.cur;
    const double tmin = A.eps < tmax ? A.eps : tmax;
    if (r == 0) {
        double m = INFINITY;
        int bad = 0;
        for (int k = threadIdx.x; k < nmin; k += BS) {
            const double v = S->minima[k];
            if (isnan(v)) bad = 1;
            m = fmin(m, v);
        }
        st.dmin = -block_max<BS>(-m, red);
        st.mode = __syncthreads_or(bad) ? STEP_BAD : STEP_SEARCH;
        st.lo = tmin;
        st.hi = tmax;
        st.s1 = st.s2 = 0.0;
        return st;
    }
    const double* p = S->state[r - 1];
    st.lo = p[SS_LO]; st.hi = p[SS_HI]; st.s1 = p[SS_S1]; st.s2 = p[SS_S2]; st.dmin = p[SS_DMIN];
    st.mode = (int)p[SS_MODE];
    if (st.mode != STEP_SEARCH) return st;
    const int n = r == 1 ? (1 << L) + 1 : 1 << levels;
    const double2* part = S->part[(r - 1) & 1];
    for (int c = threadIdx.x; c < n; c += BS) {
        double a = 0.0, b = 0.0;
        for (int k = 0; k < chunks; ++k) {
            a += part[c * chunks + k].x;
            b += part[c * chunks + k].y;
        }
        s1[c] = a;
        s2[c] = b;
        e[c] = a * a / b;
    }
    __syncthreads();
    auto take = [&](int c) { st.s1 = s1[c]; st.s2 = s2[c]; };
    if (r == 1) {  // the first round also took both ends: 0 is tmax, 1 << L is tmin
        if (e[0] >= A.tau) {
            st.lo = tmax;
            take(0);
            st.mode = STEP_END;
            return st;
        }
        take(1 << L);
        if (e[1 << L] <= A.tau) {
            st.mode = tmin == tmax ? STEP_END : STEP_DONE;
            return st;
        }
    }
    int node = 1;
    for (int k = 0; k < levels; ++k) {
        const double mid = 0.5 * (st.lo + st.hi);
        if (e[node] >= A.tau) {
            st.lo = mid;
            take(node);
            node = 2 * node + 1;
        } else {
            st.hi = mid;
            node = 2 * node;
        }
    }
    return st;
}

// Round r: candidate blockIdx.x (the heap index of a midpoint; in the first
// round also the two ends), chunk blockIdx.y of the particles.
__global__ __launch_bounds__(256) void step_round_kernel(StepIn A, StepScratch* S, int r, int nmin, int L, int prev,
                                                         int levels, int64_t chunk)
{
    __shared__ double e[kStepCand], s1[kStepCand], s2[kStepCand];
    __shared__ double2 red[2][4];
    const StepState st = step_state<256>(A, S, r, nmin, L, prev, gridDim.y, e, s1, s2);
    if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) {
        double* p = S->state[r];
        p[SS_LO] = st.lo; p[SS_HI] = st.hi; p[SS_S1] = st.s1; p[SS_S2] = st.s2; p[SS_DMIN] = st.dmin;
        p[SS_MODE] = (double)st.mode;
    }
    if (st.mode != STEP_SEARCH) return;
    const int c = r == 0 ? blockIdx.x : blockIdx.x + 1;
    double t;
    if (r == 0 && c == 0) {
        t = st.hi;
    } else if (r == 0 && c == 1 << L) {
        t = st.lo;
    } else {
        double lo = st.lo, hi = st.hi;
        for (int bit = 30 - __builtin_clz(c); bit >= 0; --bit) {
            const double mid = 0.5 * (lo + hi);
            if ((c >> bit) & 1) lo = mid;
            else hi = mid;
        }
        t = 0.5 * (lo + hi);
    }
    const double a = -t * A.scale;
    const double m = a * st.dmin;
    double v1 = 0.0, v2 = 0.0;
    const int64_t j0 = blockIdx.y * chunk, j1 = j0 + chunk < A.N ? j0 + chunk : A.N;
    for (int64_t j = j0 + threadIdx.x; j < j1; j += 256) {
        const double v = exp(a * A.d[j] - m);
        v1 += v;
        v2 += v * v;
    }
    int turn = 0;
    const double2 s = pair_sum<256>(v1, v2, red, turn);
    if (threadIdx.x == 0) S->part[r & 1][c * gridDim.y + blockIdx.y] = s;
}

__global__ __launch_bounds__(256) void step_out_kernel(StepIn A, const StepScratch* S, int r, int L, int prev,
                                                       int chunks)
{
    __shared__ double e[kStepCand], s1[kStepCand], s2[kStepCand];
    const StepState st = step_state<256>(A, S, r, 0, L, prev, chunks, e, s1, s2);
    const bool first = blockIdx.x == 0 && threadIdx.x == 0;
    if (st.mode == STEP_BAD) {
        if (first) A.out3[0] = A.out3[1] = A.out3[2] = NAN;
        return;
    }
    const double t = st.lo;
    const double a = -t * A.scale;
    const double lse = a * st.dmin + log(st.s1);
    for (int64_t j = blockIdx.x * (int64_t)256 + threadIdx.x; j < A.N; j += gridDim.x * (int64_t)256) {
        const double lw = a * A.d[j];
        if (A.logw) A.logw[j] = lw;
        if (A.w) A.w[j] = exp(lw - lse);
    }
    if (first) {
        A.out3[0] = st.mode == STEP_END ? 1.0 : A.cur + t;
        A.out3[1] = lse - log((double)A.N);
        A.out3[2] = st.s1 * st.s1 / st.s2;
    }
}

int launch_next_step(mls2mc_ctx* ctx, int64_t N, const double* d, double scale, double cur, double tau,
                     double eps, double* out3, double* logw, double* w, hipStream_t s)
{
    const StepIn A{N, d, scale, cur, tau, eps, out3, logw, w};
    if (N <= kStepSmall) {
        if (N <= 256) next_step_small_kernel<256, 1><<<1, 256, 0, s>>>(A);
        else if (N <= 512) next_step_small_kernel<512, 1><<<1, 512, 0, s>>>(A);
        else if (N <= 1024) next_step_small_kernel<512, 2><<<1, 512, 0, s>>>(A);
        else if (N <= 2048) next_step_small_kernel<1024, 2><<<1, 1024, 0, s>>>(A);
        else next_step_small_kernel<1024, 4><<<1, 1024, 0, s>>>(A);
        MLS_CHECK_HIP(hipGetLastError());
        return MLS2MC_OK;
    }
    // Levels per round: a round costs its launch (about 4 us) plus 2^L N
    // exponentials; the more particles, the fewer midpoints pay.  About 512
    // workgroups per round.
    const int L = N <= 8192 ? 7 : N <= 65536 ? 6 : N <= (1 << 18) ? 5 : N <= (1 << 20) ? 4 : 3;
    const int chunks = 512 >> L;
    const int64_t chunk = (N + chunks - 1) / chunks;
    const int nmin = (int)std::min<int64_t>(kStepMin, (N + 1023) / 1024);
    StepScratch* S = step_scratch(ctx);
    step_min_kernel<<<nmin, 256, 0, s>>>(N, d, S);
    int r = 0, prev = 0;
    for (int done = 0; done < 64; ++r) {
        const int levels = std::min(L, 64 - done);
        const unsigned cand = r == 0 ? (1u << L) + 1 : (1u << levels) - 1;
        step_round_kernel<<<dim3(cand, chunks), 256, 0, s>>>(A, S, r, nmin, L, prev, levels, chunk);
        prev = levels;
        done += levels;
    }
    step_out_kernel<<<(unsigned)std::min<int64_t>(1024, (N + 255) / 256), 256, 0, s>>>(A, S, r, L, prev, chunks);
    MLS_CHECK_HIP(hipGetLastError());
    return MLS2MC_OK;
}

// ESS at t = 1 of the weights exp(-scale d), d = dhi - dlo (dlo may be null:
// d = dhi); out[0] = ESS, out[1] = N / ESS - 1 = (cv^LU)^2 of the level-update
// test of Sec. 4.4 (population variance, so ESS = N / (1 + cv^2)).
__global__ __launch_bounds__(kNS) void ess_diff_kernel(int64_t N, const double* __restrict__ dlo,
                                                       const double* __restrict__ dhi,
                                                       double scale, double* __restrict__ out)
{
    __shared__ double red[kNS / 64];
    const double a = -1.0 * scale;
    double mx = -INFINITY;
    int bad = 0;
    for (int64_t j = threadIdx.x; j < N; j += kNS) {
        const double v = dlo ? dhi[j] - dlo[j] : dhi[j];
        if (!isfinite(v)) bad = 1;
        mx = fmax(mx, a * v);
    }
    mx = block_max<kNS>(mx, red);
    if (__syncthreads_or(bad)) {
        if (threadIdx.x == 0) out[0] = out[1] = NAN;
        return;
    }
    __shared__ double2 red2[2][kNS / 64];
    double s1 = 0.0, s2 = 0.0;
    for (int64_t j = threadIdx.x; j < N; j += kNS) {
        const double v = exp(a * (dlo ? dhi[j] - dlo[j] : dhi[j]) - mx);
        s1 += v;
        s2 += v * v;
    }
    int turn = 0;
    const double2 s = pair_sum<kNS>(s1, s2, red2, turn);
    if (threadIdx.x == 0) {
        const double e = s.x * s.x / s.y;
        out[0] = e;
        out[1] = (double)N / e - 1.0;
    }
}

int launch_ess_cv(int64_t N, const double* dlo, const double* dhi, double scale, double* out,
                  hipStream_t s)
{
    ess_diff_kernel<<<1, kNS, 0, s>>>(N, dlo, dhi, scale, out);
    MLS_CHECK_HIP(hipGetLastError());
    return MLS2MC_OK;
}

// ------------------------------------------------ linear test model --
// G_l(theta) = (A + 2^{-2l} E) theta (A, E: N_obs x K, row-major), with the
// fused potential when y is given: a stand-in forward map for which the
// tempered and bridged posteriors are Gaussian in closed form.  One thread
// per particle; only the first min(N, *N_dev) rows when N_dev is given.
__global__ void linear_forward_kernel(int64_t N, const int64_t* __restrict__ N_dev, int K, int nobs,
                                      double sc, const double* __restrict__ A,
                                      const double* __restrict__ E, const double* __restrict__ th,
                                      double* __restrict__ G, const double* __restrict__ y,
                                      double inv_sigma, double* __restrict__ phi,
                                      int8_t* __restrict__ status, int32_t* __restrict__ iters)
{
    const int64_t q = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    const int64_t n = N_dev ? (*N_dev < N ? *N_dev : N) : N;
    if (q >= n) return;
    double ph = 0.0;
    for (int o = 0; o < nobs; ++o) {
        double g = 0.0;
        for (int k = 0; k < K; ++k) g += (A[o * K + k] + sc * E[o * K + k]) * th[q * K + k];
        G[q * nobs + o] = g;
        if (y) {
            const double r = (y[o] - g) * inv_sigma;
            ph += r * r;
        }
    }
    if (y && phi) phi[q] = 0.5 * ph;
    if (status) status[q] = 0;
    if (iters) iters[q] = 0;
}

int launch_linear_forward(mls2mc_ctx* ctx, int l, int64_t N, const double* theta, double* G,
                          int8_t* status, int32_t* iters, const double* y, double* phi,
                          hipStream_t s, const int64_t* N_dev)
{
    if (N == 0) return MLS2MC_OK;
    linear_forward_kernel<<<(unsigned)((N + 127) / 128), 128, 0, s>>>(
        N, N_dev, ctx->prob.K, ctx->nobs, std::ldexp(1.0, -2 * l), ctx->d_lin_A, ctx->d_lin_E, theta, G, y,
        1.0 / ctx->prob.sigma_n, phi, status, iters);
    MLS_CHECK_HIP(hipGetLastError());
    return MLS2MC_OK;
}

// G = S theta for N rows (the linear surrogate; S is N_obs x K)
int launch_linear_map(int64_t N, int K, int nobs, const double* S, const double* theta, double* G, hipStream_t s)
{
    if (N == 0) return MLS2MC_OK;
    linear_forward_kernel<<<(unsigned)((N + 127) / 128), 128, 0, s>>>(N, nullptr, K, nobs, 0.0, S, S, theta, G,
                                                                      nullptr, 0.0, nullptr, nullptr, nullptr);
    MLS_CHECK_HIP(hipGetLastError());
    return MLS2MC_OK;
}

// ------------------------------------------------------------- resample --
// Exact integer CDF (see mls2mc.h): every sum is of integers, so any split
// gives the same ancestors.  Up to kResSmall particles one workgroup does it
// all with the prefix sums in LDS; beyond, blocks of kResBlock particles form
// their maxima, their quantised totals, the prefix sums and the searches in
// four launches.  (us, one workgroup with a serial scan of its 1024 chunk
// totals and searches in global memory -> now: N = 200 17 -> 4, N = 16384
// 146 -> 22.)
constexpr int64_t kResSmall = 4096;
constexpr int kResBlock = 4096;

__device__ __forceinline__ bool bad_weight(double v) { return !(v >= 0.0) || isinf(v); }
__device__ __forceinline__ bool bad_uniform(double v) { return !(v >= 0.0 && v < 1.0); }
// q_j = floor(w_j 2^(62 - c) / 2^ex): ex brings max w into [1/2, 1), c = ceil(log2 N)
__device__ __forceinline__ uint64_t quantised(double w, int ex, int c)
{
    return (uint64_t)floor(ldexp(ldexp(w, -ex), 62 - c));
}
__device__ __forceinline__ int ceil_log2(int64_t N) { return N <= 1 ? 0 : 64 - __builtin_clzll((uint64_t)(N - 1)); }
// floor(u 2^53 T / 2^53)
__device__ __forceinline__ uint64_t target(double u, uint64_t T)
{
    const uint64_t U = (uint64_t)ldexp(u, 53);
    const uint64_t ph = __umul64hi(U, T), pl = U * T;
    return (ph << 11) | (pl >> 53);
}

// inclusive sum of v over the workgroup's threads in order; part: one entry
// per wave.  *total: the sum over all threads.
template <int BS>
__device__ __forceinline__ uint64_t scan_u64(uint64_t v, uint64_t* part, uint64_t* total)
{
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint64_t n = __shfl_up((unsigned long long)v, o, 64);
        if (lane >= o) v += n;
    }
    if (lane == 63) part[wv] = v;
    __syncthreads();
    uint64_t before = 0, all = 0;
#pragma unroll
    for (int k = 0; k < BS / 64; ++k) {
        if (k < wv) before += part[k];
        all += part[k];
    }
    *total = all;
    return v + before;
}

template <int BS, int PER>
__global__ __launch_bounds__(BS) void resample_small_kernel(int N, const double* __restrict__ w,
                                                            const double* __restrict__ u,
                                                            int32_t* __restrict__ anc)
{
    __shared__ double red[BS / 64];
    __shared__ uint64_t part[BS / 64];
    __shared__ uint64_t C[BS * PER];
    double wv[PER], uv[PER], mx = 0.0;
    int bad = 0;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int j = threadIdx.x * PER + k, i = threadIdx.x + k * BS;
        wv[k] = j < N ? w[j] : 0.0;
        uv[k] = i < N ? u[i] : 0.0;
        if (bad_weight(wv[k]) || bad_uniform(uv[k])) bad = 1;
        else mx = fmax(mx, wv[k]);
    }
    mx = block_max<BS>(mx, red);
    if (__syncthreads_or(bad) || !(mx > 0.0)) {
        for (int i = threadIdx.x; i < N; i += BS) anc[i] = -1;
        return;
    }
    int ex;
    frexp(mx, &ex);
    const int c = ceil_log2(N);
    uint64_t run[PER], sum = 0, T;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        sum += quantised(wv[k], ex, c);
        run[k] = sum;
    }
    const uint64_t before = scan_u64<BS>(sum, part, &T) - sum;
#pragma unroll
    for (int k = 0; k < PER; ++k) C[threadIdx.x * PER + k] = before + run[k];  // past N: T, never below a target
    __syncthreads();
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int i = threadIdx.x + k * BS;
        if (i >= N) break;
        const uint64_t ti = target(uv[k], T);
        int a = 0, b = N - 1;
        while (a < b) {
            const int mid = (a + b) >> 1;
            if (C[mid] > ti) b = mid; else a = mid + 1;
        }
        anc[i] = a;
    }
}

// per block: the largest weight, or -1 when a weight or uniform is invalid
__global__ __launch_bounds__(1024) void resample_max_kernel(int64_t N, const double* __restrict__ w,
                                                            const double* __restrict__ u, double* __restrict__ pm)
{
    __shared__ double red[16];
    double mx = 0.0;
    int bad = 0;
    const int64_t j0 = blockIdx.x * (int64_t)kResBlock;
#pragma unroll
    for (int k = 0; k < kResBlock / 1024; ++k) {
        const int64_t j = j0 + threadIdx.x + 1024 * k;
        if (j >= N) break;
        const double v = w[j];
        if (bad_weight(v) || bad_uniform(u[j])) bad = 1;
        else mx = fmax(mx, v);
    }
    mx = block_max<1024>(mx, red);
    bad = __syncthreads_or(bad);
    if (threadIdx.x == 0) pm[blockIdx.x] = bad ? -1.0 : mx;
}

// per block: its quantised total; the first block also notes the largest
// weight (0 when nothing can be drawn) in pm[gridDim.x]
__global__ __launch_bounds__(1024) void resample_total_kernel(int64_t N, const double* __restrict__ w,
                                                              double* __restrict__ pm, uint64_t* __restrict__ ps)
{
    __shared__ double red[16];
    __shared__ uint64_t part[16];
    double mx = 0.0;
    int bad = 0;
    for (unsigned k = threadIdx.x; k < gridDim.x; k += 1024) {
        const double v = pm[k];
        if (v < 0.0) bad = 1;
        mx = fmax(mx, v);
    }
    mx = block_max<1024>(mx, red);
    if (__syncthreads_or(bad)) mx = 0.0;
    if (blockIdx.x == 0 && threadIdx.x == 0) pm[gridDim.x] = mx;
    if (!(mx > 0.0)) return;
    int ex;
    frexp(mx, &ex);
    const int c = ceil_log2(N);
    uint64_t sum = 0, T;
    const int64_t j0 = blockIdx.x * (int64_t)kResBlock;
#pragma unroll
    for (int k = 0; k < kResBlock / 1024; ++k) {
        const int64_t j = j0 + threadIdx.x + 1024 * k;
        if (j < N) sum += quantised(w[j], ex, c);
    }
    (void)scan_u64<1024>(sum, part, &T);
    if (threadIdx.x == 0) ps[blockIdx.x] = T;
}

__global__ __launch_bounds__(1024) void resample_prefix_kernel(int64_t N, const double* __restrict__ w,
                                                               const double* __restrict__ pm,
                                                               const uint64_t* __restrict__ ps,
                                                               uint64_t* __restrict__ C)
{
    __shared__ uint64_t part[2][16];
    const double mx = pm[gridDim.x];
    if (!(mx > 0.0)) return;
    uint64_t sum = 0, T, before;
    for (unsigned k = threadIdx.x; k < blockIdx.x; k += 1024) sum += ps[k];
    (void)scan_u64<1024>(sum, part[0], &before);
    int ex;
    frexp(mx, &ex);
    const int c = ceil_log2(N);
    constexpr int PER = kResBlock / 1024;
    const int64_t j0 = blockIdx.x * (int64_t)kResBlock + threadIdx.x * PER;
    uint64_t run[PER];
    sum = 0;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        if (j0 + k < N) sum += quantised(w[j0 + k], ex, c);
        run[k] = sum;
    }
    before += scan_u64<1024>(sum, part[1], &T) - sum;
#pragma unroll
    for (int k = 0; k < PER; ++k)
        if (j0 + k < N) C[j0 + k] = before + run[k];
}

__global__ __launch_bounds__(256) void resample_search_kernel(int64_t N, const double* __restrict__ u,
                                                              const double* __restrict__ mx,
                                                              const uint64_t* __restrict__ C,
                                                              int32_t* __restrict__ anc)
{
    const int64_t i = blockIdx.x * (int64_t)256 + threadIdx.x;
    if (i >= N) return;
    if (!(*mx > 0.0)) {
        anc[i] = -1;
        return;
    }
    const uint64_t ti = target(u[i], C[N - 1]);
    int64_t a = 0, b = N - 1;
    while (a < b) {
        const int64_t mid = a + (b - a) / 2;
        if (C[mid] > ti) b = mid; else a = mid + 1;
    }
    anc[i] = (int32_t)a;
}

int64_t resample_scratch(int64_t N)
{
    return N <= kResSmall ? 1 : N + 2 * ((N + kResBlock - 1) / kResBlock) + 1;
}

// C: resample_scratch(N) uint64 of scratch (every entry is written before it
// is read, so it needs no clearing)
int launch_resample_into(int64_t N, const double* w, const double* u, uint64_t* C, int32_t* anc,
                         hipStream_t s)
{
    if (N <= kResSmall) {
        if (N <= 256) resample_small_kernel<256, 1><<<1, 256, 0, s>>>((int)N, w, u, anc);
        else if (N <= 1024) resample_small_kernel<1024, 1><<<1, 1024, 0, s>>>((int)N, w, u, anc);
        else resample_small_kernel<1024, 4><<<1, 1024, 0, s>>>((int)N, w, u, anc);
    } else {
        const unsigned nb = (unsigned)((N + kResBlock - 1) / kResBlock);
        uint64_t* ps = C + N;
        double* pm = reinterpret_cast<double*>(ps + nb);
        resample_max_kernel<<<nb, 1024, 0, s>>>(N, w, u, pm);
        resample_total_kernel<<<nb, 1024, 0, s>>>(N, w, pm, ps);
        resample_prefix_kernel<<<nb, 1024, 0, s>>>(N, w, pm, ps, C);
        resample_search_kernel<<<(unsigned)((N + 255) / 256), 256, 0, s>>>(N, u, pm + nb, C, anc);
    }
    MLS_CHECK_HIP(hipGetLastError());
    return MLS2MC_OK;
}

int launch_resample(mls2mc_ctx* ctx, int64_t N, const double* w, const double* u, int32_t* anc,
                    hipStream_t s)
{
    MLS_TRY(ctx->ws_misc.ensure(sizeof(uint64_t) * (size_t)resample_scratch(N)));
    return launch_resample_into(N, w, u, ctx->ws_misc.as<uint64_t>(), anc, s);
}

// --------------------------------------------------------------- gather --
__global__ void gather_kernel(int64_t N, int64_t ncols, const int32_t* __restrict__ anc,
                              int64_t n_src, const double* __restrict__ src,
                              double* __restrict__ dst)
{
    const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (t >= N * ncols) return;
    const int64_t i = t / ncols, c = t - i * ncols;
    const int64_t a = anc[i];
    dst[t] = (a >= 0 && a < n_src) ? src[a * ncols + c] : NAN;
}

int launch_gather(int64_t N, int64_t ncols, const int32_t* anc, int64_t n_src, const double* src,
                  double* dst, hipStream_t s)
{
    if (N * ncols == 0) return MLS2MC_OK;
    gather_kernel<<<(unsigned)((N * ncols + 255) / 256), 256, 0, s>>>(N, ncols, anc, n_src, src,
                                                                     dst);
    MLS_CHECK_HIP(hipGetLastError());
    return MLS2MC_OK;
}

// --------------------------------------------------------------- Philox --
// Philox4x32-10 (Salmon et al., SC'11): counter {idx, sub, stage, stream},
// key {seed lo, seed hi}.
__device__ __forceinline__ void philox10(uint32_t c[4], uint32_t k0, uint32_t k1)
{
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        const uint64_t p0 = (uint64_t)0xD2511F53u * c[0];
        const uint64_t p1 = (uint64_t)0xCD9E8D57u * c[2];
        const uint32_t n0 = (uint32_t)(p1 >> 32) ^ c[1] ^ k0;
        const uint32_t n2 = (uint32_t)(p0 >> 32) ^ c[3] ^ k1;
        c[1] = (uint32_t)p1;
        c[3] = (uint32_t)p0;
        c[0] = n0;
        c[2] = n2;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
}

__device__ __forceinline__ double u53(uint32_t hi, uint32_t lo)
{
    return (double)((((uint64_t)hi << 32) | lo) >> 11) * 0x1.0p-53;
}

__global__ void philox_kernel(uint64_t seed, uint32_t stream_id, uint32_t stage, uint32_t sub,
                              int64_t n, int normal, double* __restrict__ out)
{
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= n) return;
    uint32_t c[4] = {(uint32_t)i, sub, stage, stream_id};
    philox10(c, (uint32_t)seed, (uint32_t)(seed >> 32));
    if (!normal) {
        out[i] = u53(c[0], c[1]);
    } else {
        const double u1 = 1.0 - u53(c[0], c[1]);
        const double u2 = u53(c[2], c[3]);
        out[i] = sqrt(-2.0 * log(u1)) * cos(2.0 * M_PI * u2);
    }
}

int launch_philox(uint64_t seed, uint32_t stream_id, uint32_t stage, uint32_t sub, int64_t n,
                  int normal, double* out, hipStream_t s)
{
    if (n == 0) return MLS2MC_OK;
    philox_kernel<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(seed, stream_id, stage, sub, n,
                                                             normal, out);
    MLS_CHECK_HIP(hipGetLastError());
    return MLS2MC_OK;
}

// ------------------------------------------------------------------ pCN --
__global__ void pcn_propose_kernel(int64_t n, double a, double s, const double* __restrict__ th,
                                   const double* __restrict__ xi, double* __restrict__ out)
{
    const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (t < n) out[t] = a * th[t] + s * xi[t];
}

// pCN: theta' = sqrt(1 - s^2) theta + s xi; random walk: theta' = theta + s xi
int launch_pcn_propose(int64_t N, int K, double s_pcn, int kernel, const double* theta, const double* xi,
                       double* out, hipStream_t s)
{
    const int64_t n = N * K;
    if (n == 0) return MLS2MC_OK;
    const double a = kernel == MLS2MC_KERNEL_RWM ? 1.0 : std::sqrt(1.0 - s_pcn * s_pcn);
    pcn_propose_kernel<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(n, a, s_pcn, theta, xi, out);
    MLS_CHECK_HIP(hipGetLastError());
    return MLS2MC_OK;
}

// mode 0: tempering (Psi = beta Phi_lo); 1: bridging with zeta < 1; 2:
// bridging at zeta = 1 (Psi = beta Phi_hi).  rwm: the random-walk kernel,
// whose ratio also carries the N(0, I) prior term |theta|^2 / 2.
// W lanes per particle, so that its rows are copied by neighbouring lanes; as
// many as its K + nobs values occupy (us with 1 / 4 / 16 / 64 lanes at 10^5
// particles: K = 1, one observation 3.3 / 4.5 / 10 / 34, K = 4, nine 9.7 / 6.2 /
// 11 / 34, K = 20, nine 29 / 13 / 14 / 36, K = 50, 25 110 / 41 / 21 / 37, K = 100,
// 49 210 / 68 / 40 / 44; at 1000 particles the last two 21 / 5.3 / 3.3 / 3.1 and
// 41 / 7.9 / 4.0 / 3.2).  Those accept every particle; lanes that only find it
// rejected cost as much, so many particles take fewer (10^5 particles all
// rejected: 3.1 with one lane, 28 with 64).
template <int W>
__global__ __launch_bounds__(256) void pcn_accept_kernel(
    int64_t N, int K, int nobs, int mode, int rwm, double beta, double zeta, const double* __restrict__ u,
    const double* __restrict__ thn, const double* __restrict__ Gln, const double* __restrict__ Ghn,
    const double* __restrict__ pln, const double* __restrict__ phn, const int8_t* __restrict__ stl,
    const int8_t* __restrict__ sth, double* __restrict__ th, double* __restrict__ Gl, double* __restrict__ Gh,
    double* __restrict__ pl, double* __restrict__ ph, uint8_t* __restrict__ acc)
{
    constexpr int64_t P = 256 / W;
    const int lane = threadIdx.x & (W - 1);
    const bool need_lo = mode != 2, need_hi = mode != 0;
    for (int64_t j = blockIdx.x * P + threadIdx.x / W; j < N; j += gridDim.x * P) {
        double psi_old, psi_new;
        if (mode == 0) {
            psi_old = beta * pl[j];
            psi_new = beta * pln[j];
        } else if (mode == 1) {
            psi_old = beta * ((1.0 - zeta) * pl[j] + zeta * ph[j]);
            psi_new = beta * ((1.0 - zeta) * pln[j] + zeta * phn[j]);
        } else {
            psi_old = beta * ph[j];
            psi_new = beta * phn[j];
        }
        if (rwm) {
            double qo = 0.0, qn = 0.0;
            for (int k = lane; k < K; k += W) {
                qo += th[j * K + k] * th[j * K + k];
                qn += thn[j * K + k] * thn[j * K + k];
            }
            psi_old += 0.5 * group_sum<W>(qo);
            psi_new += 0.5 * group_sum<W>(qn);
        }
        bool ok = true;
        if (need_lo && stl && stl[j] != 0) ok = false;
        if (need_hi && sth && sth[j] != 0) ok = false;
        const bool a = ok && (log(u[j]) < -(psi_new - psi_old));
        if (a) {
            for (int k = lane; k < K; k += W) th[j * K + k] = thn[j * K + k];
            if (need_lo)
                for (int o = lane; o < nobs; o += W) Gl[j * nobs + o] = Gln[j * nobs + o];
            if (need_hi)
                for (int o = lane; o < nobs; o += W) Gh[j * nobs + o] = Ghn[j * nobs + o];
        }
        if (lane == 0) {
            if (a && need_lo) pl[j] = pln[j];
            if (a && need_hi) ph[j] = phn[j];
            if (acc) acc[j] = a ? 1 : 0;
        }
    }
}

int launch_pcn_accept(int64_t N, int K, int nobs, int mode, int rwm, double beta, double zeta,
                      const double* u, const double* th_new, const double* Glo_new,
                      const double* Ghi_new, const double* plo_new, const double* phi_new,
                      const int8_t* st_lo, const int8_t* st_hi, double* theta, double* Glo,
                      double* Ghi, double* plo, double* phi, uint8_t* acc, hipStream_t s)
{
    if (N == 0) return MLS2MC_OK;
#define MLS_ACCEPT(W)                                                                                        \
    pcn_accept_kernel<W><<<row_blocks(N, W), 256, 0, s>>>(N, K, nobs, mode, rwm, beta, zeta, u, th_new, Glo_new, \
                                                          Ghi_new, plo_new, phi_new, st_lo, st_hi, theta, Glo, \
                                                          Ghi, plo, phi, acc)
    const int row = K + nobs;
    if (row <= 4) MLS_ACCEPT(1);
    else if (row <= 16 || (row <= 48 && N > 32768)) MLS_ACCEPT(4);
    else if (row <= 48 || N > 32768) MLS_ACCEPT(16);
    else MLS_ACCEPT(64);
#undef MLS_ACCEPT
    MLS_CHECK_HIP(hipGetLastError());
    return MLS2MC_OK;
}

// ---------------------------------------------------- small reductions --
// out2[0] += sum of iters, out2[1] += count of status != 0 (one workgroup).
__global__ __launch_bounds__(kNS) void reduce_iters_kernel(int64_t N, const int32_t* __restrict__ v,
                                                           const int8_t* __restrict__ st,
                                                           int64_t* __restrict__ out2)
{
    __shared__ double red[kNS / 64];
    double a = 0.0, b = 0.0;
    for (int64_t j = threadIdx.x; j < N; j += kNS) {
        a += (double)v[j];
        if (st) b += st[j] != 0 ? 1.0 : 0.0;
    }
    a = block_sum<kNS>(a, red);
    b = block_sum<kNS>(b, red);
    if (threadIdx.x == 0) {
        out2[0] += (int64_t)a;
        out2[1] += (int64_t)b;
    }
}

int launch_reduce_i32(int64_t N, const int32_t* v, const int8_t* st, int64_t* out2, hipStream_t s)
{
    if (N == 0) return MLS2MC_OK;
    reduce_iters_kernel<<<1, kNS, 0, s>>>(N, v, st, out2);
    MLS_CHECK_HIP(hipGetLastError());
    return MLS2MC_OK;
}

}  // namespace mls
