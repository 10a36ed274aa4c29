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
// against 4.0e11, 30 of 256^2 about the same (lds_launch says which runs).
//
// Two things the order of the code is for.  A row's coefficients are loaded
// when the previous level's work starts and waited for when it ends: loaded
// next to their use (as the compiler would have it) the same query took 253 ms
// instead of 211.  And a level is branch-free but for the one off the plain
// path: with its own range test and zero fill per level it took 272 ms.
#include "internal.h"
#include "node_update.h"
#include "tile.h"

namespace eig {

namespace {

// A tile's forcing tables: the window's weights (two components), dt^2 / rho
// of its rows, and the series values of the K steps.
constexpr int kSwFco = 2 * kSrcW * kSrcW, kSwSeries = kSwFco + kSrcW;

// N neighbouring nodes of one row held by a lane.
template <int N>
struct Pt {
    float u[N], v[N];
};

// Values of the neighbouring lane; lanes 0 / 63 receive zero.
__device__ __forceinline__ float lane_left(float x) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x138, 0xf, 0xf, true));
}
__device__ __forceinline__ float lane_right(float x) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x130, 0xf, 0xf, true));
}

template <int N>
__device__ __forceinline__ void x_neighbours(const float (&w)[N], float (&l)[N], float (&r)[N]) {
    l[0] = lane_left(w[N - 1]);
    r[N - 1] = lane_right(w[0]);
#pragma unroll
    for (int n = 1; n < N; ++n) {
        l[n] = w[n - 1];
        r[n - 1] = w[n];
    }
}

template <int N>
__device__ __forceinline__ Pt<N> x_diff(const Pt<N>& w) {
    float l[N], r[N];
    Pt<N> d;
    x_neighbours<N>(w.u, l, r);
#pragma unroll
    for (int n = 0; n < N; ++n) d.u[n] = r[n] - l[n];
    x_neighbours<N>(w.v, l, r);
#pragma unroll
    for (int n = 0; n < N; ++n) d.v[n] = r[n] - l[n];
    return d;
}

template <int N>
__device__ __forceinline__ Pt<N> x_sum(const Pt<N>& w) {
    float l[N], r[N];
    Pt<N> d;
    x_neighbours<N>(w.u, l, r);
#pragma unroll
    for (int n = 0; n < N; ++n) d.u[n] = r[n] + l[n];
    x_neighbours<N>(w.v, l, r);
#pragma unroll
    for (int n = 0; n < N; ++n) d.v[n] = r[n] + l[n];
    return d;
}

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

template <int N>
__device__ __forceinline__ Pt<N> ld_pt(const float2* row, int col) {
    Pt<N> p;
    if constexpr (N == 2) {
        const float4 q = ld4(row, col);
        p.u[0] = q.x;
        p.v[0] = q.y;
        p.u[1] = q.z;
        p.v[1] = q.w;
    } else {
        const float2 q = ld2(row, col);
        p.u[0] = q.x;
        p.v[0] = q.y;
    }
    return p;
}
template <int N>
__device__ __forceinline__ void st_pt(float2* row, int col, const Pt<N>& p) {
    if constexpr (N == 2)
        st4(row, col, make_float4(p.u[0], p.v[0], p.u[1], p.v[1]));
    else
        st2(row, col, make_float2(p.u[0], p.v[0]));
}

// Levels 0..K-1 of a strip as seen between two rows: level j holds its row
// i - 1 - j in c and the row above in p, with their x-differences.
template <int K, int N>
struct StreamState {
    Pt<N> c[K], p[K], dc[K], dp[K];
};

template <int K, int N>
struct StreamTile {
    const SolveDesc* d;
    const float* coef;
    float2 *out0, *out1;       // levels m + K and m + K - 1
    float2* traces;
    int nz, pitch, m, nsteps, nrec;
    int kb, nstore;            // rows stored (none in the last pass)
    int col, cld;              // the lane's first column, clamped for loads
    bool st_ok;                // the lane stores its nodes
    bool free_col[N];          // columns 1..nx-2
    int rec[N];
    int sk0, si0;              // forcing window: first row and column
    const float* sw;           // forcing tables (LDS)
};

// Zero at the rigid columns.
template <int K, int N>
__device__ __forceinline__ void zero_rigid(const StreamTile<K, N>& t, Pt<N>& w) {
#pragma unroll
    for (int q = 0; q < N; ++q) {
        w.u[q] = t.free_col[q] ? w.u[q] : 0.f;
        w.v[q] = t.free_col[q] ? w.v[q] : 0.f;
    }
}

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
    // lane predicates are formed here, not kept in scalar registers
    int col = t.col;
    __asm__ volatile("" : "+v"(col));
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
    if (r == 0 && t.m + j <= t.nsteps) {
#pragma unroll
        for (int q = 0; q < N; ++q) {
            int rec = t.rec[q];
            __asm__ volatile("" : "+v"(rec));
            if (rec >= 0)
                st2(t.traces, (size_t)(t.m + j) * t.nrec + rec, make_float2(nw.u[q], nw.v[q]));
        }
    }
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
__device__ __forceinline__ void stream_strip(const SolveDesc* d, int m, int pin, int x0, int kb,
                                             int ke, const float* sw) {
    const int lane = threadIdx.x;
    StreamTile<K, N> t;
    t.d = d;
    t.coef = d->coef;
    t.nz = d->nz;
    t.pitch = d->pitch;
    t.m = m;
    t.nsteps = d->nsteps;
    t.nrec = d->nrec;
    t.traces = d->traces;
    t.kb = kb;
    const int nx = d->nx, nz = d->nz;
    constexpr int W = 64 * N;
    const int cs = x0 == 0 ? 0 : x0 + K, ce = x0 + W >= nx ? nx : x0 + W - K;
    t.col = x0 + N * lane;
    t.cld = min(t.col, t.pitch - N);
    t.st_ok = t.col >= cs && t.col < ce;
    t.sk0 = d->src_k0;
    t.si0 = d->src_i0;
    t.sw = sw;
#pragma unroll
    for (int q = 0; q < N; ++q) {
        const int c = t.col + q;
        t.free_col[q] = c >= 1 && c <= nx - 2;
        t.rec[q] = -1;
        if (kb == 0 && c >= 1 && c <= nx - 2 && c >= cs && c < ce) t.rec[q] = ldi(d->recmap, c);
    }
    const float2* b0 = pin ? d->buf2 : d->buf0;
    const float2* b1 = pin ? d->buf3 : d->buf1;
    float2* o0 = pin ? d->buf0 : d->buf2;
    float2* o1 = pin ? d->buf1 : d->buf3;
    t.out0 = o0;    // m is even: level m in slot 0, m - 1 in slot 1
    t.out1 = o1;
    t.nstore = m + K >= t.nsteps ? 0 : ke - kb;
    StreamState<K, N> s;
#pragma unroll
    for (int j = 0; j < K; ++j)
#pragma unroll
        for (int q = 0; q < N; ++q)
            s.c[j].u[q] = s.c[j].v[q] = s.p[j].u[q] = s.p[j].v[q] = s.dc[j].u[q] = s.dc[j].v[q] =
                s.dp[j].u[q] = s.dp[j].v[q] = 0.f;
    const int i0 = max(kb - K, 0), i1 = ke + K;
    // the next rows to load: cur's row i + 3 and prev's one above, both held at
    // the grid's last ones
    const size_t pitch = t.pitch;
    const float2* cur = b0 + (size_t)i0 * pitch;
    const float2* prev = b1 + (size_t)max(i0 - 1, 0) * pitch;
    Pt<N> ca = ld_pt<N>(cur, t.cld), pa = ld_pt<N>(prev, t.cld);
    prev = b1 + (size_t)i0 * pitch;
    Pt<N> cb = ld_pt<N>(cur + pitch, t.cld), pb = ld_pt<N>(prev, t.cld);
    Pt<N> cc = ld_pt<N>(cur + 2 * pitch, t.cld), pc = ld_pt<N>(prev + pitch, t.cld);
    cur += 2 * pitch;
    prev += pitch;
    auto load = [&](int i, Pt<N>& c, Pt<N>& p) {
        const size_t inc = i + 3 < nz ? pitch : 0;
        cur += inc;
        prev += inc;
        c = ld_pt<N>(cur, t.cld);
        p = ld_pt<N>(prev, t.cld);
    };
    // rows i whose K levels are all free ones below the surface
    const int f0 = K + 1, f1 = nz;
    // and off the forcing window where it meets this strip
    const bool win = t.si0 < x0 + W && t.si0 + kSrcW > x0;
    const int w0 = win ? t.sk0 + 1 : f1, w1 = win ? t.sk0 + kSrcW + K : f1;
    auto plain = [&](int i) { return i >= f0 && i < f1 && (i < w0 || i >= w1); };
    LayerCoef cf = scalar_coef((ScalarRow)((uintptr_t)t.coef) + ((ptrdiff_t)i0 - 1) * kCoefStride);
    for (int i = i0; i < i1; i += 3) {
        stream_row<K, N, EDGE>(t, s, i, plain(i), cf, ca, pa);
        load(i, ca, pa);
        stream_row<K, N, EDGE>(t, s, i + 1, plain(i + 1), cf, cb, pb);
        load(i + 1, cb, pb);
        stream_row<K, N, EDGE>(t, s, i + 2, plain(i + 2), cf, cc, pc);
        load(i + 2, cc, pc);
    }
}

template <int K>
__global__ void __launch_bounds__(64, 2)
stencil_layered_stream(const SolveDesc* __restrict__ descs, const int2* __restrict__ tiles,
                       int ntiles, int pass, int rows) {
    __shared__ float sw[kSwSeries + K];
    const int b = xcd_block(blockIdx.x, gridDim.x);
    if (b >= ntiles) return;
    const int2 te = tiles[b];
    const SolveDesc* d = descs + __builtin_amdgcn_readfirstlane(te.x);
    const unsigned sc = (unsigned)__builtin_amdgcn_readfirstlane(te.y);
    const int L = pass - d->start, m = K * L;
    if (L < 0 || m >= d->nsteps) return;
    const int x0 = (int)(sc >> 17) * 2;
    const int kb = (int)(sc & 0xffff) * rows, ke = min(kb + rows, d->nz - 1);
    for (int e = threadIdx.x; e < 2 * kSrcW * kSrcW; e += 64) sw[e] = ld1(d->srcw, e);
    if (threadIdx.x < kSrcW)
        sw[kSwFco + threadIdx.x] =
            ld1(d->coef, (size_t)(d->src_k0 + threadIdx.x) * kCoefStride + kFco);
    if (threadIdx.x < K)
        sw[kSwSeries + threadIdx.x] =
            m + (int)threadIdx.x < d->nsteps ? ld1(d->srcs, m + threadIdx.x) : 0.f;
    __syncthreads();
    if (sc & 0x10000)
        stream_strip<K, 1, true>(d, m, L & 1, x0, kb, ke, sw);
    else if (x0 == 0 || x0 + 128 > d->nx - 1)
        stream_strip<K, 2, true>(d, m, L & 1, x0, kb, ke, sw);
    else
        stream_strip<K, 2, false>(d, m, L & 1, x0, kb, ke, sw);
}

}  // namespace

void launch_layered_stream(const SolveDesc* descs, const int2* tiles, int ntiles, int pass,
                           int rows, hipStream_t s) {
    if (ntiles > 0)
        stencil_layered_stream<kStreamSteps><<<ntiles, 64, 0, s>>>(descs, tiles, ntiles, pass,
                                                                   rows);
}

}  // namespace eig
