// Depth-only media with rigid edges, K = 8 leapfrog steps per launch streamed
// through registers (variant 23, the temporal_blocking 4 family's default).
//
// One wave owns a strip of 128 columns (two per lane; or 64, one per lane) and
// a chunk of rows of one solve, and streams down the rows: when row i of u^m
// arrives, level j forms its row i - j (u^{m+j}) from rows i-j-1 .. i-j+1 of
// level j-1 and row i-j of level j-2, all in VGPRs, for j = 1 .. K.  A level
// keeps two rows and their x-differences (16 registers per lane with two
// columns), x-neighbours are DPP operands of the additions that use them, and
// the coefficients of a row are scalar operands.  Nothing passes through LDS
// but the forcing tables, and there is no barrier.  Levels m + K - 1 and m + K
// go to the other buffer pair (passes alternate between a solve's two pairs, so
// no wave overwrites what another still loads); the last pass stores nothing,
// and steps past the solve's last one are formed and dropped.
//
// The columns within K of a strip's side, and the rows within K of a chunk's
// ends, hold values whose halo went stale: neighbouring strips overlap by 2 K
// columns and a chunk starts K rows early and ends K late.  Rows off the plain
// path (the surface, the forcing window, past the last free row) branch to
// stream_special; the branch is uniform.
//
// Bound: memory and vector issue together.  On 3840 solves of 512^2 the fields
// move at 0.85 of the rate of a large copy, and the SIMDs issue vector instructions
// in 0.81 of the cycles (2.26 GHz under this load).  An update takes 24 vector
// instructions (13 per component, the depth differences shared between rows) times
// the overlap (1.13 at 512 columns) and the halo rows; past L2 a launch moves each
// node's two levels once in and once out, 4 B per update.  K = 8 is what 256 VGPRs
// hold, two waves per SIMD; measured on 240 solves of 512^2 in the Monte Carlo
// query: K = 4 336 ms, 6 244 ms, 8 211 ms.  On 960 solves of 512^2: 9.5e11
// updates/s against 4.9e11 for four steps with the tile in LDS (67 instructions
// per update, 8 B); 240 solves 8.0e11 against 4.8e11, 60 of 384^2 5.3e11
// against 4.0e11, 30 of 256^2 about the same (small_launch_variant says which runs).
//
// Two things the order of the code is for.  A row's coefficients are loaded
// when the previous level's work starts and waited for when it ends: loaded
// next to their use (as the compiler would have it) the same query took 253 ms
// instead of 211.  And a level is branch-free but for the one off the plain
// path: with its own range test and zero fill per level it took 272 ms.
#include "stream.h"

namespace eig {

namespace {

// What the edge relation takes of a row.
struct CeRow {
    float ap, as, l;
    double rp, rs;  // 1 / (1 + ap), 1 / (1 + as)
};
// (c: the coefficients' row, t: the side columns')
__device__ __forceinline__ CeRow scalar_ce(ScalarRow c, ScalarRow t) {
    const CAS double* r = (const CAS double*)t;
    return {c[kCeP], c[kCeS], c[kCeL], r[0], r[1]};
}

template <int K, int N>
struct StreamState {
    Pt<N> c[K], p[K], dc[K], dp[K];
};

// What a strip holds of the grid's sides.  Rigid: columns that stay zero or
// none.  Absorbing: column 0 (node 0 of a lane) and / or column nx-1 (node R of
// a lane, -1: not in the strip), which follow the edge relation.
template <bool EDGE>
struct RigidSides {
    static constexpr bool kAbs = false, kEdge = EDGE;
};
template <bool L, int R>
struct AbsorbingSides {
    static constexpr bool kAbs = true, kEdge = L || R >= 0, kLeft = L;
    static constexpr int kRight = R;
};

// The side columns of an absorbing strip (the relation of ce.h, ce_side):
// `below` and `above` are the column's rows r + 1 and r - 1 and half 1/2 (at the
// ends of a side column: the one-sided difference and 1).  x / (1 + a) is x
// times the FP64 reciprocal, rounded to FP32: the bits of the FP32 division.
// The product is off by 2^-52 of itself.  A quotient of two FP32 numbers that is
// not exactly where the rounding changes is at least 2^-48 of itself away,
// subnormal results included; exactly there it is only where a subnormal result's
// divisor is 2 (whose reciprocal is exact) or above 4, and 1 + a is below 2 for
// every stable time step.  It takes 3 instructions, a division 10.
template <int K, int N, class S>
__device__ __forceinline__ void absorbing_columns(const StreamTile<K, N>& t, const CeRow& ce,
                                                  float half, const Pt<N>& below,
                                                  const Pt<N>& above, const Pt<N>& c,
                                                  const Pt<N>& old, Pt<N>& nw) {
#pragma clang fp contract(off)
    float lu[N], ru[N], lv[N], rv[N];
    x_neighbours<N>(c.u, lu, ru);
    x_neighbours<N>(c.v, lv, rv);
    auto edge = [](float a, double r, float prev, float in, float tang) {
        return (float)(__builtin_fmaf(1.f - a, prev, 2.f * __builtin_fmaf(a, in, tang)) * r);
    };
    auto side = [&](auto q, float sg, float iu, float iv, bool here) {
        constexpr int Q = decltype(q)::value;
        const float dzu = half * (below.u[Q] - above.u[Q]), dzv = half * (below.v[Q] - above.v[Q]);
        const float wu = edge(ce.ap, ce.rp, old.u[Q], iu, sg * ce.l * dzv);
        const float wv = edge(ce.as, ce.rs, old.v[Q], iv, sg * ce.as * dzu);
        nw.u[Q] = here ? wu : nw.u[Q];
        nw.v[Q] = here ? wv : nw.v[Q];
    };
    if constexpr (S::kLeft) side(std::integral_constant<int, 0>(), 1.f, ru[0], rv[0], t.left);
    if constexpr (S::kRight >= 0) {
        constexpr int Q = S::kRight;
        side(std::integral_constant<int, Q>(), -1.f, lu[Q], lv[Q], t.right);
    }
}

// Level j's row r off the plain path: the surface row's own-row terms, the
// forcing, the grid's last row (rigid: zero; absorbing: the edge relation) and
// rows past it, the side columns, and the receivers.  a: the acceleration
// without the first two.
template <int K, int N, class S>
__device__ __forceinline__ void stream_special(const StreamTile<K, N>& t, int j, int r,
                                               ScalarRow crow, const LayerCoef& cf,
                                               const CeRow& ce, const Pt<N>& n, const Pt<N>& c,
                                               const Pt<N>& p, const Pt<N>& dc, const Pt<N>& up,
                                               float2 (&a)[N], Pt<N>& nw) {
    if (r < 0 || r >= t.nz - (S::kAbs ? 0 : 1)) {
#pragma unroll
        for (int q = 0; q < N; ++q) nw.u[q] = nw.v[q] = 0.f;
        return;
    }
    if constexpr (S::kAbs) {
        if (r == t.nz - 1) {
#pragma unroll
            for (int q = 0; q < N; ++q) {
                const float2 w = ce_bottom(crow[kCeP], crow[kCeS], crow[kCeL], dc.u[q], dc.v[q],
                                           make_float2(p.u[q], p.v[q]),
                                           make_float2(up.u[q], up.v[q]));
                nw.u[q] = w.x;
                nw.v[q] = w.y;
            }
            if constexpr (S::kEdge) absorbing_columns<K, N, S>(t, ce, 1.f, c, p, c, up, nw);
            return;
        }
    }
    const int col = lane_col(t);
    const int dk = r - t.sk0;
    const bool win = (unsigned)dk < (unsigned)kSrcW;
    if (r == 0 || win) {
#pragma unroll
        for (int q = 0; q < N; ++q) {
            if (r == 0) {
                a[q].x = __builtin_fmaf(cf.c[kCm0U], dc.v[q], a[q].x);
                a[q].y = __builtin_fmaf(cf.c[kCm0V], dc.u[q], a[q].y);
            }
            const int di = col + q - t.si0;
            if (win && (unsigned)di < (unsigned)kSrcW) {
                const float fsv = t.sw[kSwFco + dk] * t.sw[kSwSeries + j - 1];
                const float* w = t.sw + dk * kSrcW + di;
                a[q].x = __builtin_fmaf(fsv, w[0], a[q].x);
                a[q].y = __builtin_fmaf(fsv, w[kSrcW * kSrcW], a[q].y);
            }
            const float2 w = layered_new(a[q], c.u[q], c.v[q], up.u[q], up.v[q]);
            nw.u[q] = w.x;
            nw.v[q] = w.y;
        }
    }
    if constexpr (S::kAbs && S::kEdge) {
        if (r == 0)
            absorbing_columns<K, N, S>(t, ce, 1.f, n, c, c, up, nw);
        else
            absorbing_columns<K, N, S>(t, ce, 0.5f, n, p, c, up, nw);
    } else if constexpr (S::kEdge) {
        zero_rigid<K, N>(t, nw);
    }
    if (r == 0 && t.m + j <= t.nsteps) record_row<K, N>(t, j, nw);
}

// One row of the pipeline: level 0 takes row i (`n`, with u^{m-1} one row up
// in `up`), level j forms its row i - j from levels j-1 and j-2.  plain: every
// level is on a free row below the surface, off the forcing window.  S: the strip's
// side columns.  cf_next, ce_next: level 1's coefficients, for the next row on
// return.
template <int K, int N, class S>
__device__ __forceinline__ void stream_row(const StreamTile<K, N>& t, StreamState<K, N>& s, int i,
                                           bool plain, LayerCoef& cf_next, CeRow& ce_next, Pt<N> n,
                                           Pt<N> up) {
    // row i of the table; opaque, so that equal rows of two levels are loaded
    // twice rather than held in scalar registers between rows of the pipeline
    ScalarRow ci = (ScalarRow)((uintptr_t)t.coef + (intptr_t)i * (kCoefStride * sizeof(float)));
    __asm__ volatile("" : "+s"(ci));
    ScalarRow ti = (ScalarRow)((uintptr_t)(t.coef + ce_table(t.nz)) +
                               (intptr_t)i * (kCeStride * sizeof(float)));
    if constexpr (S::kAbs && S::kEdge) __asm__ volatile("" : "+s"(ti));
#pragma unroll
    for (int j = 1; j <= K; ++j) {
        const int r = i - j;
        const LayerCoef cf = cf_next;
        // the next level's row, or level 1's of the pipeline's next row: issued
        // once this level's has arrived (scalar loads return in any order, so
        // a wait for one is a wait for all) and before this level's work
        __asm__ volatile("" ::"s"(cf.c[0]));
        cf_next = scalar_coef(ci - (j < K ? (j + 1) * kCoefStride : 0));
        const CeRow ce = ce_next;
        if constexpr (S::kAbs && S::kEdge)
            ce_next = scalar_ce(ci - (j < K ? (j + 1) * kCoefStride : 0),
                                ti - (j < K ? (j + 1) * kCeStride : 0));
        __builtin_amdgcn_sched_barrier(0);
        const Pt<N> dn = x_diff<N>(n), c = s.c[j - 1], p = s.p[j - 1], sx = x_sum<N>(c);
        Pt<N> nw;
        float2 a[N];
#pragma unroll
        for (int q = 0; q < N; ++q) {
            NodeRow rm{}, rc{}, rn{};
            rm.u = p.u[q];
            rm.v = p.v[q];
            rm.dxu = s.dp[j - 1].u[q];
            rm.dxv = s.dp[j - 1].v[q];
            rc.u = c.u[q];
            rc.v = c.v[q];
            rc.sxu = sx.u[q];
            rc.sxv = sx.v[q];
            rn.u = n.u[q];
            rn.v = n.v[q];
            rn.dxu = dn.u[q];
            rn.dxv = dn.v[q];
            a[q] = layered_accel<false>(cf, rm, rc, rn);
            const float2 w = layered_new(a[q], c.u[q], c.v[q], up.u[q], up.v[q]);
            nw.u[q] = w.x;
            nw.v[q] = w.y;
        }
        if constexpr (S::kAbs && S::kEdge) {
            if (plain) absorbing_columns<K, N, S>(t, ce, 0.5f, n, p, c, up, nw);
        } else if constexpr (S::kEdge) {
            zero_rigid<K, N>(t, nw);
        }
        if (__builtin_expect(!plain, 0))
            stream_special<K, N, S>(t, j, r, ci - j * kCoefStride, cf, ce, n, c, p, s.dc[j - 1],
                                    up, a, nw);
        if (j == K && (unsigned)(r - t.kb) < (unsigned)t.nstore && t.st_ok) {
            Pt<N> w1 = c, w0 = nw;
            if constexpr (S::kAbs && N == 2) {
                if constexpr (S::kRight == 0) {  // the padding column beside nx-1 stays zero
                    w1.u[1] = t.right ? 0.f : w1.u[1];
                    w1.v[1] = t.right ? 0.f : w1.v[1];
                    w0.u[1] = t.right ? 0.f : w0.u[1];
                    w0.v[1] = t.right ? 0.f : w0.v[1];
                }
            }
            st_pt<N>(t.out1 + (size_t)r * t.pitch, t.col, w1);
            st_pt<N>(t.out0 + (size_t)r * t.pitch, t.col, w0);
        }
        up = p;
        s.p[j - 1] = c;
        s.c[j - 1] = n;
        s.dp[j - 1] = s.dc[j - 1];
        s.dc[j - 1] = dn;
        n = nw;
    }
}

template <int K, int N, class S>
__device__ __forceinline__ void stream_strip(const StreamEntry& e, const float* sw, int* rec) {
    StreamTile<K, N> t;
    tile_init<K, N>(t, e.d, e.m, e.pin, e.x0, e.kb, e.ke, sw, rec);
    StreamState<K, N> s{};
    const int i0 = max(e.kb - K, 0), i1 = e.ke + K;
    RowFeed<N> f;
    f.init(e.d, e.pin, i0, t.col);
    LayerCoef cf = scalar_coef((ScalarRow)((uintptr_t)t.coef) + ((ptrdiff_t)i0 - 1) * kCoefStride);
    CeRow ce{};
    if constexpr (S::kAbs && S::kEdge)
        ce = scalar_ce((ScalarRow)((uintptr_t)t.coef) + ((ptrdiff_t)i0 - 1) * kCoefStride,
                       (ScalarRow)((uintptr_t)(t.coef + ce_table(t.nz))) +
                           ((ptrdiff_t)i0 - 1) * kCeStride);
    for (int i = i0; i < i1; i += 3) {
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            stream_row<K, N, S>(t, s, i + q, plain_row(t, i + q), cf, ce, f.c[q], f.p[q]);
            f.template next<S::kAbs>(i + q, q);
        }
    }
}

template <int K>
__device__ __forceinline__ void load_tables(const StreamEntry& e, float* sw) {
    load_forcing<K>(e.d, e.m, sw);
    if (threadIdx.x < kSrcW)
        sw[kSwFco + threadIdx.x] =
            ld1(e.d->coef, (size_t)(e.d->src_k0 + threadIdx.x) * kCoefStride + kFco);
    __syncthreads();
}

template <int K>
__global__ void __launch_bounds__(64, 2)
stencil_layered_stream(const SolveDesc* __restrict__ descs, const int2* __restrict__ tiles,
                       int ntiles, int pass, int rows) {
    __shared__ float sw[kSwSeries + K];
    __shared__ int rec[128];
    const int b = xcd_block(blockIdx.x, gridDim.x);
    if (b >= ntiles) return;
    StreamEntry e;
    if (!stream_entry<K>(descs, tiles[b], pass, rows, e)) return;  // uniform
    load_tables<K>(e, sw);
    if (e.narrow)
        stream_strip<K, 1, RigidSides<true>>(e, sw, rec);
    else if (e.x0 == 0 || e.x0 + 128 > e.d->nx - 1)
        stream_strip<K, 2, RigidSides<true>>(e, sw, rec);
    else
        stream_strip<K, 2, RigidSides<false>>(e, sw, rec);
}

// The same with absorbing edges (variant 28): the side strips form their side
// columns in the same pass, the last row is a special row, and the halo is that
// of the rigid kernel (an edge node reads one node inside and two along the
// edge).  What a strip has of the sides is its template, so that the inner
// strips and each kind of side strip pay for what they hold only; the side
// columns take 16 instructions a side and level for both components, against
// 24 per update of all 128 columns.  Bound: vector issue.  K = 6: 8
// spills registers.  Against one step per launch (edge nodes in extra
// wavefronts; launch-bound up to some 60 solves of 252 x 90, field bytes above),
// us per step on 252 x 90: 1 solve 8.9 -> 4.4, 30 9.3 -> 6.2, 60 10.6 -> 9.4, 104
// 13.5 -> 13.0, 195 22.8 -> 13.9; 512 solves of 201 x 151 79 -> 31.  No measured
// load is faster with one step, so no rule keeps it.
template <int K>
__global__ void __launch_bounds__(64, 2)
stencil_absorbing_stream(const SolveDesc* __restrict__ descs, const int2* __restrict__ tiles,
                         int ntiles, int pass, int rows) {
    __shared__ float sw[kSwSeries + K];
    __shared__ int rec[128];
    const int b = xcd_block(blockIdx.x, gridDim.x);
    if (b >= ntiles) return;
    StreamEntry e;
    if (!stream_entry<K, true>(descs, tiles[b], pass, rows, e)) return;  // uniform
    load_tables<K>(e, sw);
    const int nx = e.d->nx;
    const bool left = e.x0 == 0, right = e.x0 + (e.narrow ? 64 : 128) > nx - 1;
    const bool odd = (nx - 1) & 1;  // column nx-1 is a lane's second node
    if (e.narrow) {
        if (left && right) stream_strip<K, 1, AbsorbingSides<true, 0>>(e, sw, rec);
        else if (left) stream_strip<K, 1, AbsorbingSides<true, -1>>(e, sw, rec);
        else if (right) stream_strip<K, 1, AbsorbingSides<false, 0>>(e, sw, rec);
        else stream_strip<K, 1, AbsorbingSides<false, -1>>(e, sw, rec);
    } else if (left && right) {
        if (odd) stream_strip<K, 2, AbsorbingSides<true, 1>>(e, sw, rec);
        else stream_strip<K, 2, AbsorbingSides<true, 0>>(e, sw, rec);
    } else if (left) {
        stream_strip<K, 2, AbsorbingSides<true, -1>>(e, sw, rec);
    } else if (right) {
        if (odd) stream_strip<K, 2, AbsorbingSides<false, 1>>(e, sw, rec);
        else stream_strip<K, 2, AbsorbingSides<false, 0>>(e, sw, rec);
    } else {
        stream_strip<K, 2, AbsorbingSides<false, -1>>(e, sw, rec);
    }
}

}  // namespace

void launch_layered_stream(const SolveDesc* descs, const int2* tiles, int ntiles, int pass,
                           int rows, int absorbing, hipStream_t s) {
    if (ntiles <= 0) return;
    if (absorbing)
        stencil_absorbing_stream<kAbsorbingStreamSteps><<<ntiles, 64, 0, s>>>(
            descs, tiles, ntiles, pass, rows);
    else
        stencil_layered_stream<kStreamSteps><<<ntiles, 64, 0, s>>>(descs, tiles, ntiles, pass,
                                                                   rows);
}

}  // namespace eig
