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
// Bound: vector issue.  An update takes 24 vector instructions (13 per
// component, the depth differences shared between rows) times the overlap
// (1.13 at 512 columns) and the halo rows; past L2 a launch moves each node's
// two levels once in and once out, 4 B per update.  K = 8 is what 256 VGPRs
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

// A row of a coefficient table through the scalar cache.
#if defined(__HIP_DEVICE_COMPILE__)
#define CAS __attribute__((address_space(4)))
#else
#define CAS
#endif
typedef const CAS float* ScalarRow;
__device__ __forceinline__ LayerCoef scalar_coef(ScalarRow c) {
    LayerCoef r;
#pragma unroll
    for (int j = 0; j < kFco; ++j) r.c[j] = c[j];
    return r;
}

// Levels 0..K-1 of a strip as seen between two rows: level j holds its row
// i - 1 - j in c and the row above in p, with their x-differences.
template <int K, int N>
struct StreamState {
    Pt<N> c[K], p[K], dc[K], dp[K];
};

// Level j's row r off the plain path: the surface row's own-row terms, the
// forcing, rows past the grid's and rigid columns (zero), and the receivers.
// a: the acceleration without the first two.
template <int K, int N, bool EDGE>
__device__ __forceinline__ void stream_special(const StreamTile<K, N>& t, int j, int r,
                                               const LayerCoef& cf, const Pt<N>& c,
                                               const Pt<N>& dc, const Pt<N>& up, float2 (&a)[N],
                                               Pt<N>& nw) {
    if (r < 0 || r >= t.nz - 1) {
#pragma unroll
        for (int q = 0; q < N; ++q) nw.u[q] = nw.v[q] = 0.f;
        return;
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
    if constexpr (EDGE) zero_rigid<K, N>(t, nw);
    if (r == 0 && t.m + j <= t.nsteps) record_row<K, N>(t, j, nw);
}

// One row of the pipeline: level 0 takes row i (`n`, with u^{m-1} one row up
// in `up`), level j forms its row i - j from levels j-1 and j-2.  plain: every
// level is on a free row below the surface, off the forcing window.  EDGE: the
// strip has a rigid column.  cf_next: level 1's coefficients, for the next row
// on return.
template <int K, int N, bool EDGE>
__device__ __forceinline__ void stream_row(const StreamTile<K, N>& t, StreamState<K, N>& s, int i,
                                           bool plain, LayerCoef& cf_next, Pt<N> n, Pt<N> up) {
    // row i of the table; opaque, so that equal rows of two levels are loaded
    // twice rather than held in scalar registers between rows of the pipeline
    ScalarRow ci = (ScalarRow)((uintptr_t)t.coef + (intptr_t)i * (kCoefStride * sizeof(float)));
    __asm__ volatile("" : "+s"(ci));
#pragma unroll
    for (int j = 1; j <= K; ++j) {
        const int r = i - j;
        const LayerCoef cf = cf_next;
        // the next level's row, or level 1's of the pipeline's next row: issued
        // once this level's has arrived (scalar loads return in any order, so
        // a wait for one is a wait for all) and before this level's work
        __asm__ volatile("" ::"s"(cf.c[0]));
        cf_next = scalar_coef(ci - (j < K ? (j + 1) * kCoefStride : 0));
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
        if constexpr (EDGE) zero_rigid<K, N>(t, nw);
        if (__builtin_expect(!plain, 0))
            stream_special<K, N, EDGE>(t, j, r, cf, c, s.dc[j - 1], up, a, nw);
        if (j == K && (unsigned)(r - t.kb) < (unsigned)t.nstore && t.st_ok) {
            st_pt<N>(t.out1 + (size_t)r * t.pitch, t.col, c);
            st_pt<N>(t.out0 + (size_t)r * t.pitch, t.col, nw);
        }
        up = p;
        s.p[j - 1] = c;
        s.c[j - 1] = n;
        s.dp[j - 1] = s.dc[j - 1];
        s.dc[j - 1] = dn;
        n = nw;
    }
}

template <int K, int N, bool EDGE>
__device__ __forceinline__ void stream_strip(const StreamEntry& e, const float* sw, int* rec) {
    StreamTile<K, N> t;
    tile_init<K, N>(t, e.d, e.m, e.pin, e.x0, e.kb, e.ke, sw, rec);
    StreamState<K, N> s{};
    const int i0 = max(e.kb - K, 0), i1 = e.ke + K;
    RowFeed<N> f;
    f.init(e.d, e.pin, i0, t.col);
    LayerCoef cf = scalar_coef((ScalarRow)((uintptr_t)t.coef) + ((ptrdiff_t)i0 - 1) * kCoefStride);
    for (int i = i0; i < i1; i += 3) {
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            stream_row<K, N, EDGE>(t, s, i + q, plain_row(t, i + q), cf, f.c[q], f.p[q]);
            f.next(i + q, q);
        }
    }
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
    load_forcing<K>(e.d, e.m, sw);
    if (threadIdx.x < kSrcW)
        sw[kSwFco + threadIdx.x] =
            ld1(e.d->coef, (size_t)(e.d->src_k0 + threadIdx.x) * kCoefStride + kFco);
    __syncthreads();
    if (e.narrow)
        stream_strip<K, 1, true>(e, sw, rec);
    else if (e.x0 == 0 || e.x0 + 128 > e.d->nx - 1)
        stream_strip<K, 2, true>(e, sw, rec);
    else
        stream_strip<K, 2, false>(e, sw, rec);
}

}  // namespace

void launch_layered_stream(const SolveDesc* descs, const int2* tiles, int ntiles, int pass,
                           int rows, hipStream_t s) {
    if (ntiles > 0)
        stencil_layered_stream<kStreamSteps><<<ntiles, 64, 0, s>>>(descs, tiles, ntiles, pass,
                                                                   rows);
}

}  // namespace eig
