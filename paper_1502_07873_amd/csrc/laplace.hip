// Laplace KL estimate, quadrature averages and design search, FP64.
//
// D^_KL(theta) = -1/2 log((2 pi)^N |H_1^-1|) - N/2 - h(theta)   (Theorem 4;
// N = 7, or the number of inferred parameters when the prior marks a subset)
// with log det H_1 taken through the scaled Hessian of Section 3.3.3,
// S = sqrt(diag H_1), H~ = S^-1 H_1 S^-1 = L L^T, so that the ~30 decades
// spanned by the raw entries never reach the factorisation;
// I = sum_s w_s D^_KL(theta_s) (Section 3.3.4, Monte Carlo or sparse
// quadrature).  Designs are receiver subsets (Section 4.5); H_1 is additive
// over receivers, so a design's H_1 is the sum of per-receiver Hessians.
#include <type_traits>
#include <utility>

#include "internal.h"
#include "tile.h"

namespace eig {

namespace {

// Matrices are N x N with N (the number of inferred parameters) a template
// argument and every loop unrolled, so that they stay in registers: with a
// runtime n their arrays are indexed in scratch memory, and a greedy step over
// 589 samples and 201 candidates took 105 us in its D^_KL kernel alone.
// Symmetric ones keep the lower triangle, row by row.
template <int N>
constexpr int kTri = N * (N + 1) / 2;
constexpr int tri(int i, int j) { return i * (i + 1) / 2 + j; }

// Offsets of the inferred parameters' lower triangle in a full 7 x 7 matrix.
template <int N>
struct Active {
    int idx[N];
    __device__ __forceinline__ explicit Active(const eig_prior& pr) {
        const int act = N == kNT ? (1 << kNT) - 1 : pr.active;
        int left = act;
#pragma unroll
        for (int a = 0; a < N; ++a) {
            idx[a] = N == kNT ? a : __builtin_ctz(left);
            left &= left - 1;
        }
    }
    __device__ __forceinline__ int at(int i, int j) const { return idx[i] * kNT + idx[j]; }
};

// x / d from r, about 1 / d: the division's value but for the last bit in rare
// cases (exactly its value where r is 1 / d correctly rounded), in 3
// instructions for 12.
__device__ __forceinline__ double div_by(double x, double d, double r) {
    const double q = x * r;
    return __builtin_fma(__builtin_fma(-q, d, x), r, q);
}

// log det of a symmetric positive definite matrix via the scaled Cholesky
// factorisation; false if it is not positive definite or not finite.  a is
// overwritten.  One logarithm is taken, of the product of the factors'
// mantissas; their exponents add up apart.
template <int N>
__device__ __forceinline__ bool scaled_logdet(double (&a)[kTri<N>], double* out) {
    double s[N], rs[N], m = 1.0;
    int e = 0;
    bool ok = true;
    auto factor = [&](double x) {
        m *= __builtin_amdgcn_frexp_mant(x);
        e += __builtin_amdgcn_frexp_exp(x);
    };
    // Rows with a diagonal entry far down the range, the subnormals among them,
    // are brought up by 2^256 each first (exactly): 1 / (s_i s_j) would overflow
    // from s_i s_j = 2^-1024 on.
    // Compared by their high words, whose minimum is an instruction each.
    constexpr double kFarDown = 0x1p-960;
    int low = __double2hiint(a[0]);
#pragma unroll
    for (int j = 1; j < N; ++j) low = min(low, __double2hiint(a[tri(j, j)]));
    if (__builtin_expect(low < __builtin_bit_cast(int64_t, kFarDown) >> 32, 0)) {
        int up[N];
#pragma unroll
        for (int i = 0; i < N; ++i) {
            up[i] = a[tri(i, i)] < kFarDown ? 256 : 0;
            e -= up[i];
        }
#pragma unroll
        for (int i = 0; i < N; ++i)
#pragma unroll
            for (int j = 0; j <= i; ++j) a[tri(i, j)] = ldexp(a[tri(i, j)], up[i] + up[j]);
    }
#pragma unroll
    for (int j = 0; j < N; ++j) {
        const double d = a[tri(j, j)];
        ok = ok && d > 0.0 && isfinite(d);
        s[j] = sqrt(d);
        rs[j] = 1.0 / s[j];
        factor(s[j]);
    }
#pragma unroll
    for (int i = 0; i < N; ++i)
#pragma unroll
        for (int j = 0; j <= i; ++j)
            a[tri(i, j)] = div_by(a[tri(i, j)], s[i] * s[j], rs[i] * rs[j]);
#pragma unroll
    for (int j = 0; j < N; ++j) {
        double v = a[tri(j, j)];
#pragma unroll
        for (int k = 0; k < j; ++k) v -= a[tri(j, k)] * a[tri(j, k)];
        ok = ok && v > 0.0 && isfinite(v);
        const double ljj = sqrt(v), rl = 1.0 / ljj;
        factor(ljj);
#pragma unroll
        for (int i = j + 1; i < N; ++i) {
            double w = a[tri(i, j)];
#pragma unroll
            for (int k = 0; k < j; ++k) w -= a[tri(i, k)] * a[tri(j, k)];
            a[tri(i, j)] = div_by(w, ljj, rl);
        }
    }
    // log 2 in two parts: 14 logarithms' worth of exponents multiplies its rounding
    const double ln2_lo = 2.3190468138462996e-17;
    *out = 2.0 * __builtin_fma((double)e, M_LN2, __builtin_fma((double)e, ln2_lo, log(m)));
    return ok;
}

// Cholesky factor of a symmetric matrix, in place; false if it is not positive
// definite.
template <int N>
__device__ __forceinline__ bool chol(double (&a)[kTri<N>]) {
    bool ok = true;
#pragma unroll
    for (int j = 0; j < N; ++j) {
        double v = a[tri(j, j)];
#pragma unroll
        for (int k = 0; k < j; ++k) v -= a[tri(j, k)] * a[tri(j, k)];
        ok = ok && v > 0.0 && isfinite(v);
        a[tri(j, j)] = sqrt(v);
#pragma unroll
        for (int i = j + 1; i < N; ++i) {
            double w = a[tri(i, j)];
#pragma unroll
            for (int k = 0; k < j; ++k) w -= a[tri(i, k)] * a[tri(j, k)];
            a[tri(i, j)] = w / a[tri(j, j)];
        }
    }
    return ok;
}

// y = L^-1 b.
template <int N>
__device__ __forceinline__ void forward_solve(const double (&L)[kTri<N>], const double (&b)[N],
                                              double (&y)[N]) {
#pragma unroll
    for (int i = 0; i < N; ++i) {
        double v = b[i];
#pragma unroll
        for (int k = 0; k < i; ++k) v -= L[tri(i, k)] * y[k];
        y[i] = v / L[tri(i, i)];
    }
}

// x = A^-1 b from the Cholesky factor of A.
template <int N>
__device__ __forceinline__ void chol_solve(const double (&L)[kTri<N>], const double (&b)[N],
                                           double (&x)[N]) {
    double y[N];
    forward_solve<N>(L, b, y);
#pragma unroll
    for (int i = N - 1; i >= 0; --i) {
        double v = y[i];
#pragma unroll
        for (int k = i + 1; k < N; ++k) v -= L[tri(k, i)] * x[k];
        x[i] = v / L[tri(i, i)];
    }
}

// h(theta) = log p(theta), the prior's marginal over the inferred parameters.
template <int N>
__device__ __forceinline__ double log_prior(const eig_prior& pr, const Active<N>& act,
                                            const double* th) {
    if (pr.kind == EIG_PRIOR_UNIFORM) {
        double v = 0.0;
#pragma unroll
        for (int a = 0; a < N; ++a) v -= log(pr.hi[act.idx[a]] - pr.lo[act.idx[a]]);
        return v;
    }
    // Gaussian: -1/2 r^T C^-1 r - 1/2 (N log 2 pi + log det C), via C = L L^T
    double L[kTri<N>], r[N], y[N];
#pragma unroll
    for (int i = 0; i < N; ++i) {
        r[i] = th[act.idx[i]] - pr.mean[act.idx[i]];
#pragma unroll
        for (int j = 0; j <= i; ++j) L[tri(i, j)] = pr.cov[act.at(i, j)];
    }
    chol<N>(L);
    forward_solve<N>(L, r, y);
    double ld = 0.0, q = 0.0;
#pragma unroll
    for (int i = 0; i < N; ++i) {
        ld += 2.0 * log(L[tri(i, i)]);
        q += y[i] * y[i];
    }
    return -0.5 * q - 0.5 * (N * log(2.0 * M_PI) + ld);
}

__device__ __forceinline__ double quiet_nan() {
    return __longlong_as_double(0x7ff8000000000000ULL);
}

// Theorem 4 on the inferred parameters' block of H_1 (overwritten); lp =
// h(theta).  NaN if the block is not positive definite.
template <int N>
__device__ __forceinline__ double dkl_of(double (&h)[kTri<N>], double lp, double* logdet,
                                         bool* pd) {
    double ld;
    *pd = scaled_logdet<N>(h, &ld);
    *logdet = *pd ? ld : quiet_nan();
    return *pd ? -0.5 * (N * log(2.0 * M_PI) - ld) - 0.5 * N - lp : quiet_nan();
}

// Theorem 3 at theta^: H = H_1 + H_2 - grad grad h on the active parameters,
//   -1/2 log((2 pi)^N |H^-1|) - N/2 - h(theta^) - 1/2 tr(H^-1 grad grad h),
// grad grad h = 0 for the uniform prior and -Gamma^-1 for the Gaussian one.
template <int N>
__global__ void __launch_bounds__(64)
theorem3_kernel(const double* __restrict__ H1, const double* __restrict__ H2, int nsample,
                const eig_prior* __restrict__ prior, const double* __restrict__ theta,
                double* __restrict__ val, int32_t* __restrict__ status) {
    const int s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= nsample) return;
    const eig_prior& pr = *prior;
    const Active<N> act(pr);
    double H[kTri<N>], Gi[kTri<N>];   // Gi: Gamma^-1 (Gaussian prior)
#pragma unroll
    for (int i = 0; i < N; ++i)
#pragma unroll
        for (int j = 0; j <= i; ++j) {
            const size_t o = (size_t)s * kNT * kNT + act.at(i, j);
            H[tri(i, j)] = H1[o] + H2[o];
            Gi[tri(i, j)] = 0.0;
        }
    bool ok = true;
    const bool gauss = pr.kind == EIG_PRIOR_GAUSSIAN;
    double tr = 0.0;   // tr(H^-1 Gamma^-1) = -tr(H^-1 grad grad h)
    if (gauss) {
        double L[kTri<N>];
#pragma unroll
        for (int i = 0; i < N; ++i)
#pragma unroll
            for (int j = 0; j <= i; ++j) L[tri(i, j)] = pr.cov[act.at(i, j)];
        ok = chol<N>(L);
#pragma unroll
        for (int c = 0; c < N; ++c) {
            double e[N] = {}, x[N];
            e[c] = 1.0;
            chol_solve<N>(L, e, x);
#pragma unroll
            for (int a = c; a < N; ++a) {
                Gi[tri(a, c)] = x[a];
                H[tri(a, c)] += x[a];
            }
        }
#pragma unroll
        for (int q = 0; q < kTri<N>; ++q) L[q] = H[q];
        const bool hok = chol<N>(L);
        ok = ok && hok;
#pragma unroll
        for (int c = 0; c < N; ++c) {
            double col[N], x[N];
#pragma unroll
            for (int a = 0; a < N; ++a) col[a] = Gi[a >= c ? tri(a, c) : tri(c, a)];
            chol_solve<N>(L, col, x);
            tr += x[c];
        }
    }
    double ld = 0.0;
    const bool pd = scaled_logdet<N>(H, &ld);
    ok = ok && pd;
    val[s] = ok ? -0.5 * (N * log(2.0 * M_PI) - ld) - 0.5 * N -
                      log_prior<N>(pr, act, theta + (size_t)s * kNT) + 0.5 * tr
                : quiet_nan();
    if (status) status[s] = ok ? EIG_OK : EIG_ENOTPD;
}

template <int N>
__global__ void __launch_bounds__(64) laplace_kernel(const double* __restrict__ H1, int nsample,
                               const eig_prior* __restrict__ prior,
                               const double* __restrict__ theta,
                               double* __restrict__ dkl, double* __restrict__ logdet,
                               int32_t* __restrict__ status) {
    const int s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= nsample) return;
    const Active<N> act(*prior);
    double h[kTri<N>];
#pragma unroll
    for (int i = 0; i < N; ++i)
#pragma unroll
        for (int j = 0; j <= i; ++j) h[tri(i, j)] = H1[(size_t)s * kNT * kNT + act.at(i, j)];
    double ld;
    bool ok;
    dkl[s] = dkl_of<N>(h, log_prior<N>(*prior, act, theta + (size_t)s * kNT), &ld, &ok);
    if (logdet) logdet[s] = ld;
    if (status) status[s] = ok ? EIG_OK : EIG_ENOTPD;
}

// out[r] = sum_s w[s] * x[r * n + s] for every row r (one block per row),
// summed in a fixed order: strided per-thread partials, then a tree.
__global__ void weighted_rows_kernel(const double* __restrict__ x, int n,
                                     const double* __restrict__ w,
                                     double* __restrict__ out) {
    const int r = blockIdx.x;
    __shared__ double part[256];
    double v = 0.0;
    for (int s = threadIdx.x; s < n; s += blockDim.x) v += w[s] * x[(size_t)r * n + s];
    part[threadIdx.x] = v;
    __syncthreads();
    for (int o = blockDim.x / 2; o > 0; o >>= 1) {
        if (threadIdx.x < o) part[threadIdx.x] += part[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[r] = part[0];
}

template <int N>
__global__ void __launch_bounds__(64) design_dkl_kernel(const double* __restrict__ H1r, int nsample,
                                  int ncand, const uint8_t* __restrict__ mask,
                                  const eig_prior* __restrict__ prior,
                                  const double* __restrict__ theta,
                                  double* __restrict__ work) {
    const int d = blockIdx.y;
    const int s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= nsample) return;
    const Active<N> act(*prior);
    double h[kTri<N>] = {};
    const uint8_t* md = mask + (size_t)d * ncand;
    for (int c = 0; c < ncand; ++c) {
        if (!md[c]) continue;
        const double* src = H1r + ((size_t)s * ncand + c) * kNT * kNT;
#pragma unroll
        for (int i = 0; i < N; ++i)
#pragma unroll
            for (int j = 0; j <= i; ++j) h[tri(i, j)] += src[act.at(i, j)];
    }
    double ld;
    bool ok;
    work[(size_t)d * nsample + s] =
        dkl_of<N>(h, log_prior<N>(*prior, act, theta + (size_t)s * kNT), &ld, &ok);
}

// The greedy search.  A step values every candidate not yet chosen on top of
// the chosen ones' summed Hessians, and the next launch picks: every wave
// finds the argmax of the step before for itself, which costs less than a
// launch of its own.  One block per candidate, one thread
// per sample (kGreedyBlock at a time); the weighted sum runs in a fixed order:
// 256 strided partials, then a tree.  The Hessians are first packed once, sample
// fastest, as the lower triangles of the inferred parameters: read as they come
// (392 B a pair, a cache line per lane and load) a step takes 48 us, not 15.
//
// Bound: latency, of a launch (4.5 us), of loads that wait for the pick and of
// some 950 FP64 instructions per sample on two to three waves per SIMD.
// Measured, 589 samples x 201 candidates: 15.2 us a step (105 us for the values
// alone and 46 for the pick when the matrices were indexed in scratch memory, one
// block added the pick's Hessians and values went by way of memory), 17 us to pack;
// 40 steps 6.15 -> 0.63 ms.
constexpr int kGreedyBlock = 1024;

// Argmax over candidates of finite or infinite value (chosen ones hold NaN),
// ties to the lowest index; -1 if there is none.
__device__ __forceinline__ bool better(double v2, int c2, double v1, int c1) {
    return c2 >= 0 && (c1 < 0 || v2 > v1 || (v2 == v1 && c2 < c1));
}
struct Best {
    double v = -INFINITY;
    int c = -1;
};
// Every wave for itself, which takes no barrier: a lane's share, then all lanes'.
__device__ __forceinline__ Best lane_best(const double* __restrict__ ival, int ncand) {
    Best b;
    for (int c = threadIdx.x & 63; c < ncand; c += 64) {
        const double v = ival[c];
        if (!isnan(v) && better(v, c, b.v, b.c)) b = {v, c};
    }
    return b;
}
__device__ __forceinline__ Best wave_best(Best b) {
    for (int o = 32; o > 0; o >>= 1) {
        const double v2 = __shfl_xor(b.v, o);
        const int c2 = __shfl_xor(b.c, o);
        if (better(v2, c2, b.v, b.c)) b = {v2, c2};
    }
    b.c = __builtin_amdgcn_readfirstlane(b.c);
    return b;
}

struct GreedyArgs {
    const double* H1r;
    const eig_prior* prior;
    const double* theta;
    const double* w;
    double* packed;        // [ncand][N (N + 1) / 2][nsample], or null
    double* lp;            // [nsample] h(theta_s)
    double* H;             // [28][nsample] sum of the chosen candidates' Hessians
    double* Hother;        // fused: the buffer that alternates with H
    double* ival;          // [ncand] I(chosen + {c})
    double* ival_other;    // fused: the one that alternates with it
    double* work;          // not fused: [ncand][nsample]
    int32_t* order;
    double* curve;
    int nsample, ncand;
};

// Records step k's pick (one block's business).
__device__ __forceinline__ void record_pick(const GreedyArgs& g, int k, Best b) {
    if (threadIdx.x) return;
    g.order[k] = b.c;
    g.curve[k] = b.c >= 0 ? b.v : quiet_nan();
}

// Whether one of the first n picks, as this lane reads them, is c.
__device__ __forceinline__ bool picked(const GreedyArgs& g, int n, int c) {
    bool hit = false;
    for (int q = threadIdx.x & 63; q < n; q += 64) hit = hit || g.order[q] == c;
    return hit;
}

template <int N>
__global__ void __launch_bounds__(kGreedyBlock)
greedy_start_kernel(GreedyArgs g) {
    const int s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= g.nsample) return;
    const Active<N> act(*g.prior);
    g.lp[s] = log_prior<N>(*g.prior, act, g.theta + (size_t)s * kNT);
    for (int j = 0; j < kTri<N>; ++j) g.H[(size_t)j * g.nsample + s] = 0.0;
}

// Element (i, j) of sample s's Hessian of candidate c.
template <int N, bool PACKED>
__device__ __forceinline__ double pair_element(const GreedyArgs& g, const Active<N>& act, int c,
                                               int s, int i, int j) {
    if (PACKED) return g.packed[((size_t)c * kTri<N> + tri(i, j)) * g.nsample + s];
    return g.H1r[((size_t)s * g.ncand + c) * kNT * kNT + act.at(i, j)];
}

// H1r to packed, 64 samples of one candidate per block.
template <int N>
__global__ void __launch_bounds__(256) greedy_pack_kernel(GreedyArgs g) {
    __shared__ double rows[64 * kNT * kNT];
    __shared__ int off[kTri<N>];
    const int t = threadIdx.x, s0 = blockIdx.x * 64, c = xcd_block(blockIdx.y, gridDim.y);
    const int n = min(64, g.nsample - s0);
    if (t == 0) {
        const Active<N> act(*g.prior);
#pragma unroll
        for (int i = 0; i < N; ++i)
#pragma unroll
            for (int j = 0; j <= i; ++j) off[tri(i, j)] = act.at(i, j);
    }
    for (int q = t; q < n * kNT * kNT; q += 256)
        rows[q] = g.H1r[((size_t)(s0 + q / (kNT * kNT)) * g.ncand + c) * (kNT * kNT) +
                        q % (kNT * kNT)];
    __syncthreads();
    const int l = t & 63;
    if (l >= n) return;
    for (int j = t >> 6; j < kTri<N>; j += 4)
        g.packed[((size_t)c * kTri<N> + j) * g.nsample + s0 + l] = rows[l * kNT * kNT + off[j]];
}

// Step k's pick, added to the running Hessians (one thread per sample).
template <int N, bool PACKED>
__global__ void __launch_bounds__(kGreedyBlock)
greedy_pick_kernel(GreedyArgs g, int k) {
    const Best best = wave_best(lane_best(g.ival, g.ncand));
    const int pick = best.c;
    if (blockIdx.x == 0) record_pick(g, k, best);
    const int s = blockIdx.x * blockDim.x + threadIdx.x;
    if (pick < 0 || s >= g.nsample) return;
    const Active<N> act(*g.prior);
#pragma unroll
    for (int i = 0; i < N; ++i)
#pragma unroll
        for (int j = 0; j <= i; ++j)
            g.H[(size_t)tri(i, j) * g.nsample + s] +=
                pair_element<N, PACKED>(g, act, pick, s, i, j);
}

// Step k's values, block (x, c): candidate c.  FUSED: the block first makes
// step k-1's pick and adds it to the running Hessians, and forms the
// candidate's weighted sum over all samples itself; one more block (c = ncand)
// keeps the pick and stores the running Hessians in the other buffer.  Else the
// values go to work.
template <int N, bool FUSED, bool PACKED>
__global__ void __launch_bounds__(kGreedyBlock) greedy_values_kernel(GreedyArgs g, int k) {
    const int t = threadIdx.x, ns = g.nsample;
    const int c = FUSED && blockIdx.y + 1 == gridDim.y ? g.ncand : xcd_block(blockIdx.y, g.ncand);
    const int s = blockIdx.x * blockDim.x + t;
    const Active<N> act(*g.prior);
    const double nan = quiet_nan();
    __shared__ double x[FUSED ? kGreedyBlock : 1], ws[FUSED ? kGreedyBlock : 1];
    // everything but what the pick selects is on its way while the wave picks
    Best best;
    if (FUSED && k > 0) best = lane_best(g.ival, g.ncand);
    const bool before = picked(g, FUSED ? k - 1 : k, c);
    double h[kTri<N>], lp = 0.0;
    if (s < ns && c < g.ncand) {
#pragma unroll
        for (int i = 0; i < N; ++i)
#pragma unroll
            for (int j = 0; j <= i; ++j) h[tri(i, j)] = pair_element<N, PACKED>(g, act, c, s, i, j);
        lp = g.lp[s];
        if (FUSED) ws[t] = g.w[s];
    }
    if (FUSED && k > 0) best = wave_best(best);
    const int pick = best.c;
    double* out = FUSED ? g.ival_other : g.ival;
    if (FUSED && c == g.ncand) {
        if (k == 0) return;
        record_pick(g, k - 1, best);
        if (s >= ns) return;
        double cur[kTri<N>];
#pragma unroll
        for (int j = 0; j < kTri<N>; ++j) cur[j] = g.H[(size_t)j * ns + s];
        if (pick >= 0) {
#pragma unroll
            for (int i = 0; i < N; ++i)
#pragma unroll
                for (int j = 0; j <= i; ++j)
                    cur[tri(i, j)] += pair_element<N, PACKED>(g, act, pick, s, i, j);
        }
#pragma unroll
        for (int j = 0; j < kTri<N>; ++j) g.Hother[(size_t)j * ns + s] = cur[j];
        return;
    }
    if (__any(before) || (FUSED && pick == c)) {  // chosen
        if (FUSED && t == 0) out[c] = nan;
        if (!FUSED && s < ns) g.work[(size_t)c * ns + s] = 0.0;
        return;
    }
    if (s < ns) {
        // half of the sums at a time, all loads of a half before the first
        // wait: pair by pair, as the compiler would have it, is 28 round trips,
        // some 4 us
        const int p = max(pick, 0);
        constexpr int kHalf = (kTri<N> + 1) / 2;
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            double cur[kHalf], add[kHalf];
#pragma unroll
            for (int i = 0; i < N; ++i)
#pragma unroll
                for (int j = 0; j <= i; ++j) {
                    const int q = tri(i, j) - half * kHalf;
                    if (q < 0 || q >= kHalf) continue;
                    cur[q] = g.H[(size_t)tri(i, j) * ns + s];
                    if (FUSED) add[q] = pair_element<N, PACKED>(g, act, p, s, i, j);
                }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int q = 0; q < kHalf && half * kHalf + q < kTri<N>; ++q) {
                if (FUSED) cur[q] = pick >= 0 ? cur[q] + add[q] : cur[q];
                h[half * kHalf + q] = cur[q] + h[half * kHalf + q];
            }
        }
        double ld;
        bool ok;
        const double v = dkl_of<N>(h, lp, &ld, &ok);
        if (FUSED)
            x[t] = v;
        else
            g.work[(size_t)c * ns + s] = v;
    }
    if (!FUSED) return;
    __syncthreads();
    __shared__ double part[256];
    const int np = min((int)blockDim.x, 256);
    double v = 0.0;
    if (t < np) {
        for (int u = t; u < ns; u += 256) v += ws[u] * x[u];
        part[t] = v;
    }
    for (int o = 128; o >= 64; o >>= 1) {
        __syncthreads();
        if (t < o && t + o < np) part[t] = v = v + part[t + o];
    }
    if (t >= 64) return;
    for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o);
    if (t == 0) out[c] = v;
}

// Rows of x as weighted_rows_kernel; NaN for a chosen candidate.
__global__ void greedy_rows_kernel(GreedyArgs g, int k) {
    const int c = blockIdx.x;
    __shared__ double part[256];
    double v = 0.0;
    const bool before = picked(g, k, c);
    for (int s = threadIdx.x; s < g.nsample; s += blockDim.x)
        v += g.w[s] * g.work[(size_t)c * g.nsample + s];
    part[threadIdx.x] = v;
    const bool chosen = __any(before);
    __syncthreads();
    for (int o = blockDim.x / 2; o > 0; o >>= 1) {
        if (threadIdx.x < o) part[threadIdx.x] += part[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) g.ival[c] = chosen ? quiet_nan() : part[0];
}

// The last step's pick.
__global__ void __launch_bounds__(kGreedyBlock) greedy_last_kernel(GreedyArgs g, int k) {
    record_pick(g, k, wave_best(lane_best(g.ival, g.ncand)));
}

// f(std::integral_constant<int, N>) for the number of parameters in a mask (0: all).
template <class F>
void for_active(int active, F f) {
    switch (active ? __builtin_popcount(active) : kNT) {
        case 1: f(std::integral_constant<int, 1>()); break;
        case 2: f(std::integral_constant<int, 2>()); break;
        case 3: f(std::integral_constant<int, 3>()); break;
        case 4: f(std::integral_constant<int, 4>()); break;
        case 5: f(std::integral_constant<int, 5>()); break;
        case 6: f(std::integral_constant<int, 6>()); break;
        default: f(std::integral_constant<int, kNT>()); break;
    }
}

}  // namespace

void launch_laplace(const double* H1, int nsample, int active, const eig_prior* prior_dev,
                    const double* theta, const double* w, double* dkl,
                    double* logdet, int32_t* status, double* eig, hipStream_t s) {
    if (nsample <= 0) return;
    for_active(active, [&](auto n) {
        laplace_kernel<n.value><<<(nsample + 63) / 64, 64, 0, s>>>(H1, nsample, prior_dev, theta,
                                                                   dkl, logdet, status);
    });
    weighted_rows_kernel<<<1, 256, 0, s>>>(dkl, nsample, w, eig);
}

void launch_theorem3(const double* H1, const double* H2, int nsample, int active,
                     const eig_prior* prior_dev, const double* theta_hat, const double* w,
                     double* val, int32_t* status, double* eig, hipStream_t s) {
    if (nsample <= 0) return;
    for_active(active, [&](auto n) {
        theorem3_kernel<n.value><<<(nsample + 63) / 64, 64, 0, s>>>(
            H1, H2, nsample, prior_dev, theta_hat, val, status);
    });
    if (eig) weighted_rows_kernel<<<1, 256, 0, s>>>(val, nsample, w, eig);
}

void launch_design_eval(const double* H1r, int nsample, int ncand,
                        const uint8_t* mask, int ndesign, int active, const eig_prior* prior_dev,
                        const double* theta, const double* w, double* work,
                        double* eig, hipStream_t s) {
    if (nsample <= 0 || ndesign <= 0) return;
    dim3 grid((nsample + 63) / 64, ndesign);
    for_active(active, [&](auto n) {
        design_dkl_kernel<n.value><<<grid, 64, 0, s>>>(H1r, nsample, ncand, mask, prior_dev,
                                                       theta, work);
    });
    weighted_rows_kernel<<<ndesign, 256, 0, s>>>(work, nsample, w, eig);
}

// A block holds all samples up to kGreedyBlock of them: then values, sums and
// the previous step's pick are one launch per step, where the second copies of
// the running Hessians and of the values fit the least scratch (from 9
// candidates or so).  More samples need more blocks per candidate to fill the
// device: three launches per step, the values by way of memory.  The packed
// copy is made where it fits the scratch and more than one step reads it.
void launch_greedy(const double* H1r, int nsample, int ncand, int active,
                   const eig_prior* prior_dev, const double* theta, const double* w,
                   double* scratch, size_t scratch_doubles, int kmax, int32_t* order,
                   double* curve, hipStream_t s) {
    const size_t ns = nsample, nc = ncand;
    GreedyArgs g{};
    g.H1r = H1r;
    g.prior = prior_dev;
    g.theta = theta;
    g.w = w;
    g.order = order;
    g.curve = curve;
    g.nsample = nsample;
    g.ncand = ncand;
    g.lp = scratch;
    g.H = g.lp + ns;
    g.ival = g.H + kTri<kNT> * ns;
    const bool fused = nsample <= kGreedyBlock &&
                       (1 + 2 * kTri<kNT>) * ns + 2 * nc <= greedy_scratch(nsample, ncand);
    if (fused) {
        g.ival_other = g.ival + nc;
        g.Hother = g.ival_other + nc;
    } else {
        g.work = g.ival + nc;
    }
    const size_t least = greedy_scratch(nsample, ncand);
    const bool pack = kmax > 1 && least + greedy_packed(nsample, ncand, active) <= scratch_doubles;
    if (pack) g.packed = scratch + least;
    const int block = nsample <= kGreedyBlock ? (nsample + 63) / 64 * 64 : 256;
    const int nblk = (nsample + block - 1) / block, nb64 = (nsample + 63) / 64;
    for_active(active, [&](auto n) {
        constexpr int N = n.value;
        auto search = [&](auto p) {
            constexpr bool PACKED = p.value;
            for (int k = 0; k < kmax; ++k) {
                if (fused) {
                    greedy_values_kernel<N, true, PACKED>
                        <<<dim3(1, ncand + 1), block, 0, s>>>(g, k);
                    if (k > 0) std::swap(g.H, g.Hother);
                    std::swap(g.ival, g.ival_other);
                    if (k == kmax - 1) greedy_last_kernel<<<1, 64, 0, s>>>(g, k);
                } else {
                    greedy_values_kernel<N, false, PACKED>
                        <<<dim3(nblk, ncand), block, 0, s>>>(g, k);
                    greedy_rows_kernel<<<ncand, 256, 0, s>>>(g, k);
                    greedy_pick_kernel<N, PACKED><<<nblk, block, 0, s>>>(g, k);
                }
            }
        };
        greedy_start_kernel<N><<<nb64, 64, 0, s>>>(g);
        if (pack) {
            greedy_pack_kernel<N><<<dim3(nb64, ncand), 256, 0, s>>>(g);
            search(std::true_type());
        } else {
            search(std::false_type());
        }
    });
}

}  // namespace eig
